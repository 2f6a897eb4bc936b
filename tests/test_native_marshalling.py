"""The native half of the binding (csrc/va_host.cpp) against the Python checks it stands for: same results to the bit, same
refusals.  A tensor subclass takes the Python way, a plain tensor the native one."""
import pytest
import torch

from paper_2605_08962_amd import binding


class Subclass(torch.Tensor):
    pass


def _refusal(f, *args, **kw):
    try:
        f(*args, **kw)
    except Exception as e:  # noqa: BLE001
        return type(e), str(e)
    return None


def _inputs(device, T=70, hq=2, hkv=1, d=64):
    gen = torch.Generator().manual_seed(3)
    mk = lambda h: torch.randn((T, h, d), generator=gen).to(torch.bfloat16).to(device)  # noqa: E731
    return mk(hq), mk(hkv), mk(hkv), torch.tensor([0, 30, T], dtype=torch.int32, device=device)


def test_tensors_on_the_cpu_are_refused_by_name():
    q, k, v, cu = _inputs("cpu")
    assert _refusal(binding.varlen_attn_fwd, q, k, v, cu, True, 0.1) == (
        ValueError, "q must be a contiguous torch.bfloat16 tensor on the GPU")
    assert _refusal(binding.varlen_attn_bwd, q, q, k, v, q, q, cu, True, 0.1) == (
        ValueError, "dout must be a contiguous torch.bfloat16 tensor on the GPU")
    assert _refusal(binding.varlen_attn_merge, q[None], q, None) == (
        ValueError, "o_parts must be a contiguous torch.bfloat16 tensor on the GPU")
    assert _refusal(binding.varlen_attn_fwd, 1, k, v, cu, True, 0.1)[0] is AttributeError


@pytest.mark.gpu
@pytest.mark.parametrize("given", [False, True])
def test_native_calls_give_what_the_python_way_gives(given):
    q, k, v, cu = _inputs("cuda")
    as_sub = lambda t: t.as_subclass(Subclass)  # noqa: E731
    side = torch.cuda.Stream()
    fo = {"out": torch.empty_like(q), "lse": torch.empty((2, 70), device="cuda")} if given else {}
    bo = {"dq": torch.empty_like(q), "dk": torch.empty_like(k), "dv": torch.empty_like(v)} if given else {}
    o, lse = binding.varlen_attn_fwd(q, k, v, cu, True, 0.1, max_seqlen=40, **fo)
    grads = binding.varlen_attn_bwd(q, q, k, v, o, lse, cu, True, 0.1, max_seqlen=40, **bo)
    if given:
        assert o is fo["out"] and lse is fo["lse"] and grads[0] is bo["dq"] and grads[2] is bo["dv"]
    o2, lse2 = binding.varlen_attn_fwd(as_sub(q), k, v, cu, True, 0.1, max_seqlen=40)
    grads2 = binding.varlen_attn_bwd(as_sub(q), q, k, v, o, lse, cu, True, 0.1, max_seqlen=40)
    torch.cuda.synchronize()
    o3, lse3 = binding.varlen_attn_fwd(q, k, v, cu, 1, 0.1, stream=side, max_seqlen=40)
    parts, lses = torch.stack([o, o]), torch.stack([lse, lse])
    merged = binding.varlen_attn_merge(parts, lses)
    merged2 = binding.varlen_attn_merge(as_sub(parts), lses)
    torch.cuda.synchronize()
    for a, b in [(o, o2), (lse, lse2), (o, o3), (lse, lse3), *zip(grads, grads2), *zip(merged, merged2)]:
        assert a.dtype == b.dtype and a.shape == b.shape and torch.equal(a, b.as_subclass(torch.Tensor))


@pytest.mark.gpu
def test_native_calls_refuse_what_the_python_way_refuses():
    q, k, v, cu = _inputs("cuda")
    sub = q.as_subclass(Subclass)
    for args, kw in [((k, v, cu.long(), True, 0.1), {}), ((k.float(), v, cu, True, 0.1), {}), ((k, v[:-1], cu, True, 0.1), {}),
                     ((k, v, cu, True, -1.0), {}), ((k, v, cu, True, float("nan")), {}), ((k, v, cu, True, 0.1), {"kv_splits": 9}),
                     ((k, v, cu, True, 0.1), {"max_seqlen": -1}), ((k[:, :, :32].contiguous(), v, cu, True, 0.1), {}),
                     ((k, v, cu, True, 0.1), {"workspace": torch.empty(16, dtype=torch.uint8, device="cuda"), "kv_splits": 1})]:
        want = _refusal(binding.varlen_attn_fwd, sub, *args, **kw)
        assert want is not None and _refusal(binding.varlen_attn_fwd, q, *args, **kw) == want
    assert _refusal(binding.varlen_attn_fwd, q[:, :, ::2], k, v, cu, True, 0.1)[0] is ValueError
    assert _refusal(binding.varlen_attn_merge, q[None], torch.zeros((1, 2, 69), device="cuda"))[1] == "lse_parts must be [P, Hq, T]"


@pytest.mark.gpu
def test_a_backward_whose_k_and_v_do_not_match_q_is_refused():
    q, k, v, cu = _inputs("cuda")
    o, lse = binding.varlen_attn_fwd(q, k, v, cu, True, 0.1)
    for k2, v2, l2, why in [(k[:-1], v[:-1], lse, "k and v must be"), (k[..., :32].contiguous(), v[..., :32].contiguous(), lse, "k and v must be"),
                            (k, v, lse[:, :-1].contiguous(), "lse must hold at least 140 elements")]:
        for first in (q, q.as_subclass(Subclass)):
            with pytest.raises(ValueError, match=why):
                binding.varlen_attn_bwd(first, q, k2, v2, o, l2, cu, True, 0.1)


@pytest.mark.gpu
def test_results_go_where_the_caller_says():
    """Buffers larger than the result or shaped otherwise, and pinned host memory (which only the Python half takes)."""
    q, k, v, cu = _inputs("cuda")
    o, lse = binding.varlen_attn_fwd(q, k, v, cu, True, 0.1)
    for out, l2 in [(torch.zeros((75, 2, 64), dtype=torch.bfloat16, device="cuda"), torch.zeros(150, device="cuda")),
                    (torch.zeros(70 * 128, dtype=torch.bfloat16).pin_memory(), torch.zeros(140).pin_memory())]:
        got = binding.varlen_attn_fwd(q, k, v, cu, True, 0.1, out=out, lse=l2)
        torch.cuda.synchronize()
        assert got[0] is out and got[1] is l2
        assert torch.equal(out.flatten()[:o.numel()].cuda(), o.flatten()) and torch.equal(l2[:140].cuda(), lse.flatten())
        assert not out.flatten()[o.numel():].any() and not l2[140:].any()
    with pytest.raises(ValueError, match="^out must be"):
        binding.varlen_attn_fwd(q, k, v, cu, True, 0.1, out=torch.empty((70, 2, 64), dtype=torch.bfloat16))


@pytest.mark.gpu
@pytest.mark.parametrize("as_handle", [False, True])
def test_what_a_call_on_another_stream_allocates_is_that_streams(as_handle):
    """Results and workspace lie in the pool of the stream the kernels run on (long enough a sample for chunks, whose fp32 parts
    make the workspace the largest piece), and the results are right."""
    T, hq = 3000, 2
    q, k, v, _ = _inputs("cuda", T=T)
    cu = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    o, lse = binding.varlen_attn_fwd(q, k, v, cu, True, 0.1, max_seqlen=T)
    grads = binding.varlen_attn_bwd(q, q, k, v, o, lse, cu, True, 0.1, max_seqlen=T)
    merged = binding.varlen_attn_merge(o[None], lse[None])
    torch.cuda.synchronize()
    side = torch.cuda.Stream()

    class Handle:
        cuda_stream = side.cuda_stream
    stream = Handle() if as_handle else side

    def pool():
        return [(s["address"], s["address"] + s["total_size"]) for s in torch.cuda.memory_snapshot() if s["stream"] == side.cuda_stream]
    p = binding.make_params(T, 1, hq, 1, 64, True, 0.1, max_seqlen=T)
    for call, want, scratch in [
            (lambda s: binding.varlen_attn_fwd(q, k, v, cu, True, 0.1, stream=s, max_seqlen=T), (o, lse), binding.fwd_workspace_bytes(p)),
            (lambda s: binding.varlen_attn_bwd(q, q, k, v, o, lse, cu, True, 0.1, stream=s, max_seqlen=T), grads,
             binding.bwd_workspace_bytes(p)),
            (lambda s: binding.varlen_attn_merge(o[None], lse[None], stream=s), merged, 0)]:
        torch.cuda.empty_cache()
        got = call(stream)
        segments = pool()
        assert sum(b - a for a, b in segments) >= scratch + sum(t.nbytes for t in got)
        assert all(any(a <= t.data_ptr() < b for a, b in segments) for t in got)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(got, want))
        del got

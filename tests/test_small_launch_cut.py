"""Launches whose walks are cut into chunks (csrc/va_small.h), forward and backward: in a recorded graph, from two host
threads, and with margins around every buffer they write."""
import pytest
import torch

from tests._util import assert_close
from tests.test_small_launch_contract import _cu, _qkv

pytestmark = pytest.mark.gpu


def test_recorded_cut_step_replays_on_new_sample_boundaries():
    """Forward and backward of a cut launch in a HIP graph: the cuts are made on the device, so replays on new lengths give
    the bits of the eager call, with eager work between the replays."""
    from paper_2605_08962_amd import binding
    T, Hq, Hkv, D, hint = 2600, 2, 1, 128, 2600
    x = _qkv(T, Hq, Hkv, D, 8) + [torch.randn((T, Hq, D), device="cuda").to(torch.bfloat16)]
    cu = _cu(2600, 0, 0)
    p = binding.make_params(T, 3, Hq, Hkv, D, True, D ** -0.5, 0, hint)
    ws = [torch.empty(f(p), dtype=torch.uint8, device="cuda") for f in (binding.fwd_workspace_bytes, binding.bwd_workspace_bytes)]
    assert ws[1].numel() > 2 * T * Hq * D * 4
    out = [torch.empty_like(x[0]), torch.empty((Hq, T), device="cuda")] + [torch.empty_like(t) for t in x[:3]]

    def call(x, cu, out, ws):
        q, k, v, do = x
        binding.varlen_attn_fwd(q, k, v, cu, True, D ** -0.5, out=out[0], lse=out[1], workspace=ws[0], max_seqlen=hint)
        binding.varlen_attn_bwd(do, q, k, v, out[0], out[1], cu, True, D ** -0.5, dq=out[2], dk=out[3], dv=out[4],
                                workspace=ws[1], max_seqlen=hint)

    call(x, cu, out, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(x, cu, out, ws)
    torch.cuda.synchronize()
    for lengths in ([2600, 0, 0], [1, 2598, 1], [900, 1000, 700], [0, 129, 2471]):
        print(f"case replay {lengths}", flush=True)
        new = [torch.randn_like(t) for t in x]
        for a, b in zip(x, new):
            a.copy_(b)
        cu.copy_(_cu(*lengths))
        for t in out:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        eager = [torch.empty_like(t) for t in out]
        call(new, _cu(*lengths), eager, [torch.empty_like(t) for t in ws])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, eager))


def test_two_threads_on_cut_launches():
    """Two host threads with streams, buffers and workspaces of their own get what serial calls give, bit for bit."""
    import threading
    from paper_2605_08962_amd import binding
    jobs = [(2049, 4, 1, 128, True), (1700, 2, 2, 80, False)]
    jobs = [(_qkv(T, Hq, Hkv, D, T) + [torch.randn((T, Hq, D), device="cuda").to(torch.bfloat16)], _cu(T), c, D)
            for T, Hq, Hkv, D, c in jobs]

    def run(i, stream, reps):
        (q, k, v, do), cu, causal, D = jobs[i]
        with torch.cuda.stream(stream):
            for _ in range(reps):
                o, lse = binding.varlen_attn_fwd(q, k, v, cu, causal, D ** -0.5, max_seqlen=q.shape[0])
                g = binding.varlen_attn_bwd(do, q, k, v, o, lse, cu, causal, D ** -0.5, max_seqlen=q.shape[0])
            stream.synchronize()
        return (o, lse) + g

    serial = [run(i, torch.cuda.current_stream(), 1) for i in range(2)]
    torch.cuda.synchronize()
    got, streams = [None, None], [torch.cuda.Stream(), torch.cuda.Stream()]

    def worker(i):
        got[i] = run(i, streams[i], 20)

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(a, b) for a, b in zip(got[i], serial[i])), f"thread {i}"


@pytest.mark.parametrize("lengths,Hq,Hkv,D,causal", [([2049], 4, 1, 128, True), ([1500, 0, 77], 2, 2, 80, False),
                                                     ([1601], 2, 1, 64, True), ([1700], 1, 1, 96, False)])
def test_margins_around_the_buffers_of_a_cut_step(lengths, Hq, Hkv, D, causal):
    """Every buffer the calls write sits between poisoned margins; the outputs are those of calls on buffers of their own."""
    from paper_2605_08962_amd import binding
    from tests.test_guard_bands import Guarded
    T, hint, sc = sum(lengths), max(lengths), D ** -0.5
    q, k, v = _qkv(T, Hq, Hkv, D, T)
    do, cu = torch.randn_like(q), _cu(*lengths)
    p = binding.make_params(T, len(lengths), Hq, Hkv, D, causal, sc, 0, hint)
    fw, bw = binding.fwd_workspace_bytes(p), binding.bwd_workspace_bytes(p)
    print(f"case {lengths} Hq={Hq} Hkv={Hkv} D={D} causal={causal} workspaces {fw} {bw}", flush=True)
    assert fw > 2 * T * Hq * D * 4 and bw > 2 * T * Hq * D * 4
    g = {"o": (q, torch.bfloat16), "lse": (torch.empty(Hq, T), torch.float32), "dq": (q, torch.bfloat16),
         "dk": (k, torch.bfloat16), "dv": (v, torch.bfloat16)}
    g = {n: (Guarded(t.numel() * (4 if dt == torch.float32 else 2)), t.shape, dt) for n, (t, dt) in g.items()}
    out = {n: b.view(dt, tuple(shape)) for n, (b, shape, dt) in g.items()}
    wsf, wsb = Guarded(fw), Guarded(bw)
    binding.varlen_attn_fwd(q, k, v, cu, causal, sc, out=out["o"], lse=out["lse"], workspace=wsf.bytes_view(), max_seqlen=hint)
    binding.varlen_attn_bwd(do, q, k, v, out["o"], out["lse"], cu, causal, sc, dq=out["dq"], dk=out["dk"], dv=out["dv"],
                            workspace=wsb.bytes_view(), max_seqlen=hint)
    torch.cuda.synchronize()
    assert all(b.intact() for b in (wsf, wsb, *(b for b, _, _ in g.values())))
    ref = binding.varlen_attn_fwd(q, k, v, cu, causal, sc, max_seqlen=hint)
    ref += binding.varlen_attn_bwd(do, q, k, v, *ref, cu, causal, sc, max_seqlen=hint)
    assert all(torch.equal(a, b) for a, b in zip(out.values(), ref))


@pytest.mark.parametrize("D", [64, 80, 96, 128])
@pytest.mark.parametrize("Hq,tiles", [(2, 128), (4, 256), (4, 260)])  # up to 256 16 rows to a workgroup of the merge, beyond 32
def test_merge_on_both_sides_of_its_rows(D, Hq, tiles):
    """Every row of a cut forward, long samples and short ones beside them, against attention in 64 bits."""
    from paper_2605_08962_amd import binding
    lengths = [3500] + [1 + 37 * i % 130 for i in range(tiles // Hq - 48)]
    lengths.insert(1, 46 * 128 + 77 - sum(lengths))
    T, sc, hint = sum(lengths), D ** -0.5, 3500
    assert (T // 128 + len(lengths)) * Hq == tiles and 1000 < lengths[1] < 3500
    q, k, v = _qkv(T, Hq, 1, D, T + D)
    o, lse = binding.varlen_attn_fwd(q, k, v, _cu(*lengths), False, sc, max_seqlen=hint)
    assert not torch.equal(o, binding.varlen_attn_fwd(q, k, v, _cu(*lengths), False, sc, max_seqlen=hint, kv_splits=1)[0])
    q, k, v, o, lse = (x.double().cpu() for x in (q, k, v, o, lse))
    at = 0
    for n in lengths:
        s = sc * q[at:at + n].transpose(0, 1) @ k[at:at + n, 0].T
        assert float((lse[:, at:at + n] - torch.logsumexp(s, -1)).abs().max()) <= 1e-3
        want = (torch.softmax(s, -1) @ v[at:at + n, 0]).transpose(0, 1)
        assert_close(f"O of the sample at {at}", o[at:at + n].numpy(), want.numpy(), allow_output_rounding=True)
        at += n

"""What holds for launches that do not fill the chip whichever way their walks are cut (csrc/va_small.h): the contract of
the entry points, on small inputs that take that path."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _qkv(T, Hq, Hkv, D, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn((T, h, D), generator=gen, device="cuda").to(torch.bfloat16) for h in (Hq, Hkv, Hkv)]


def _cu(*lengths):
    return torch.tensor([0, *lengths], dtype=torch.int32, device="cuda").cumsum(0, dtype=torch.int32)


@pytest.mark.parametrize("D,causal", [(64, False), (80, True), (96, False), (128, True)])
def test_rows_whose_scores_are_all_minus_infinity(D, causal):
    """Scores of -inf (an infinite query against keys of one sign) leave a row without weight: O = 0 and LSE = -inf, cut
    into chunks as uncut, and no trace in the other rows."""
    from paper_2605_08962_amd import binding
    T, rows = 1500, [0, 77, 1200, 1499]
    print(f"case D={D} causal={causal} T={T}", flush=True)
    q, k, v = _qkv(T, 2, 2, D, D)
    k[:, :, 0] = -1.0
    q[rows] = 0.0
    clean = q.clone()
    q[rows, :, 0] = float("inf")
    p = binding.make_params(T, 1, 2, 2, D, causal, D ** -0.5)
    assert binding.fwd_workspace_bytes(p) > T * 2 * D * 8             # cut: room for two parts and more
    others = [i for i in range(T) if i not in rows]
    for splits in (0, 1):
        o, lse = binding.varlen_attn_fwd(q, k, v, _cu(T), causal, D ** -0.5, kv_splits=splits)
        ro, rlse = binding.varlen_attn_fwd(clean, k, v, _cu(T), causal, D ** -0.5, kv_splits=splits)
        assert bool((o[rows] == 0).all()) and bool((lse[:, rows] == float("-inf")).all()), f"kv_splits {splits}"
        assert torch.equal(o[others], ro[others]) and torch.equal(lse[:, others], rlse[:, others])


def _guarded(nbytes):
    """A workspace of nbytes between two poisoned margins, and whether they are still whole."""
    buf = torch.full((4096 + nbytes + 4096 + 16,), 0xA5, dtype=torch.uint8, device="cuda")
    return buf[4096:4096 + nbytes], lambda: bool((buf[:4096] == 0xA5).all()) and bool((buf[4096 + nbytes:] == 0xA5).all())


@pytest.mark.parametrize("lengths,Hq,Hkv,D,causal", [([2049], 4, 1, 128, True), ([1500], 2, 2, 80, False),
                                                     ([1300, 0, 1, 1100], 2, 1, 64, True), ([1700], 2, 2, 96, False),
                                                     ([1300] + [200] * 70, 1, 1, 64, False)])  # (by the work list)
def test_smaller_workspaces_get_fewer_chunks(lengths, Hq, Hkv, D, causal):
    """A workspace that does not hold all chunks (kept from a larger batch, sized without the hint) is worked with; one
    that only holds what an uncut call needs gives that call's bits; one below that is refused; nothing is written past it."""
    from paper_2605_08962_amd import binding
    T, hint, sc = sum(lengths), max(lengths), D ** -0.5
    q, k, v = _qkv(T, Hq, Hkv, D, 3 * D)
    do, cu = torch.randn_like(q), _cu(*lengths)
    size = lambda f, splits: f(binding.make_params(T, len(lengths), Hq, Hkv, D, causal, sc, splits, hint))
    near = lambda a, b: float((a.float() - b.float()).norm()) <= 5e-3 * float(b.float().norm())
    uncut = binding.varlen_attn_fwd(q, k, v, cu, causal, sc, kv_splits=1)
    uncut_g = binding.varlen_attn_bwd(do, q, k, v, *uncut, cu, causal, sc)
    for what, sizes in (("fwd", binding.fwd_workspace_bytes), ("bwd", binding.bwd_workspace_bytes)):
        full, least = size(sizes, 0), size(sizes, 1)
        part = {"fwd": Hq * T * (4 * D + 4), "bwd": Hq * T * D * 4}[what]
        assert full >= least + 2 * part or (what == "bwd" and len(lengths) > 64 and full == least)
        for n in sorted({n for n in (full, full - 1, least + 3 * part, least + 2 * part, least + part, least) if least <= n}):
            print(f"case {what} {lengths} Hq={Hq} Hkv={Hkv} D={D} causal={causal} workspace {n} of {full}", flush=True)
            ws, intact = _guarded(n)
            if what == "fwd":
                got, ref = binding.varlen_attn_fwd(q, k, v, cu, causal, sc, workspace=ws, max_seqlen=hint), uncut
            else:
                got, ref = binding.varlen_attn_bwd(do, q, k, v, *uncut, cu, causal, sc, workspace=ws, max_seqlen=hint), uncut_g
            assert intact() and all(near(a, b) for a, b in zip(got, ref))
            if n == least:
                assert all(torch.equal(a, b) for a, b in zip(got, ref))
        with pytest.raises(binding.VarlenAttnError):
            ws = torch.empty(least - 1, dtype=torch.uint8, device="cuda")
            if what == "fwd":
                binding.varlen_attn_fwd(q, k, v, cu, causal, sc, workspace=ws, max_seqlen=hint)
            else:
                binding.varlen_attn_bwd(do, q, k, v, *uncut, cu, causal, sc, workspace=ws, max_seqlen=hint)


@pytest.mark.parametrize("lengths,Hq,Hkv,D", [([8191], 4, 1, 128), ([2000], 2, 2, 64), ([6000, 5, 3000], 3, 3, 96)])
@pytest.mark.parametrize("hinted", [False, True])
def test_static_scratch_gives_the_bits_of_a_workspace_of_its_size(lengths, Hq, Hkv, D, hinted):
    from paper_2605_08962_amd import binding
    T, hint, sc = sum(lengths), max(lengths) if hinted else 0, D ** -0.5
    q, k, v = _qkv(T, Hq, Hkv, D, T)
    cu = _cu(*lengths)
    need = binding.fwd_workspace_bytes(binding.make_params(T, len(lengths), Hq, Hkv, D, True, sc, 0, hint))
    print(f"case {lengths} Hq={Hq} Hkv={Hkv} D={D} hint={hint} preferred workspace {need}", flush=True)
    n = binding.STATIC_SCRATCH_BYTES
    ref = binding.varlen_attn_fwd(q, k, v, cu, True, sc, workspace=torch.empty(n, dtype=torch.uint8, device="cuda"),
                                  max_seqlen=hint)
    got = [torch.full_like(t, float("nan")) for t in ref]
    binding.varlen_attn_fwd_static_scratch(q, k, v, cu, True, sc, *got, max_seqlen=hint)
    assert all(torch.equal(a, b) for a, b in zip(got, ref))
    own = binding.varlen_attn_fwd(q, k, v, cu, True, sc, max_seqlen=hint)
    for a, b in zip(got, own):
        assert torch.equal(a, b) if need <= n else float((a.float() - b.float()).norm()) <= 5e-3 * float(b.float().norm())


@pytest.mark.parametrize("lengths,causal", [([16, 16, 1300, 1, 0], False), ([1100, 2, 63, 64], True), ([400] * 4, False)])
@pytest.mark.parametrize("D", [64, 128])
def test_uneven_batches_without_the_hint(lengths, causal, D):
    """Several samples of unknown lengths: the device cuts by the lengths it finds, and not at all where none is long."""
    from paper_2605_08962_amd import binding
    T, sc = sum(lengths), D ** -0.5
    print(f"case {lengths} D={D} causal={causal}", flush=True)
    q, k, v = _qkv(T, 2, 1, D, T + D)
    assert binding.fwd_workspace_bytes(binding.make_params(T, len(lengths), 2, 1, D, causal, sc)) > 2 * T * 2 * D * 4
    got = binding.varlen_attn_fwd(q, k, v, _cu(*lengths), causal, sc)
    ref = binding.varlen_attn_fwd(q, k, v, _cu(*lengths), causal, sc, kv_splits=1)
    for a, b in zip(got, ref):
        assert float((a.float() - b.float()).norm()) <= 5e-3 * float(b.float().norm())
        assert max(lengths) > 512 or torch.equal(a, b)


@pytest.mark.parametrize("lengths,Hq,Hkv", [([100] * 30 + [900], 8, 8), ([300] * 9 + [0, 1, 700, 129], 8, 4),
                                            ([5, 64] * 31 + [0, 400], 4, 4)])
@pytest.mark.parametrize("D,causal", [(64, True), (80, False), (96, True), (128, False)])
def test_order_of_the_samples_does_not_show(lengths, Hq, Hkv, D, causal):
    """dK/dV may have more workgroups than the chip holds and takes the longest samples first then (the first batch at
    head_dim 96 and 128).  The batch turned round gives the same bits, and so does each sample by itself."""
    from paper_2605_08962_amd import binding
    T, sc = sum(lengths), D ** -0.5
    assert len(lengths) <= 64 and 256 < (T // 128 + len(lengths)) * Hq
    print(f"case B={len(lengths)} T={T} Hq={Hq} Hkv={Hkv} D={D} causal={causal}", flush=True)
    x = _qkv(T, Hq, Hkv, D, T + D)
    x.append(torch.randn_like(x[0]))

    def call(q, k, v, do, lens):
        o, lse = binding.varlen_attn_fwd(q, k, v, _cu(*lens), causal, sc, kv_splits=0, max_seqlen=max(max(lens), 1))
        return (o, lse.t()) + binding.varlen_attn_bwd(do, q, k, v, o, lse, _cu(*lens), causal, sc)

    got = [t.split(lengths) for t in call(*x, lengths)]
    turned = [t.flip(0) if t.dim() == 1 else torch.cat(t.split(lengths)[::-1]) for t in x]
    back = [t.split(lengths[::-1])[::-1] for t in call(*turned, lengths[::-1])]
    for s in (lengths.index(max(lengths)), 0, len(lengths) - 1):
        alone = call(*[t.split(lengths)[s].contiguous() for t in x], [lengths[s]]) if lengths[s] else None
        for i in range(5):
            # (the forward's keys may be cut by what else is in the launch: only the gradients and short samples' outputs)
            assert torch.equal(got[i][s], back[i][s]), f"sample {s}, output {i}: order"
            if alone and max(lengths) <= 512:
                assert torch.equal(got[i][s], alone[i]), f"sample {s}, output {i}: alone"


@pytest.mark.parametrize("lengths,Hq,Hkv,D,causal", [([2049], 4, 2, 128, True), ([1300, 3, 1700], 2, 2, 64, False),
                                                     ([1100, 700], 2, 1, 80, True), ([1500], 3, 3, 96, False)])
def test_hints_above_1024_right_or_wrong(lengths, Hq, Hkv, D, causal):
    """With kv_splits = 1 the gradients are the same bits whatever the hint; cut by a hint that is exact, too large or too
    small they agree with the oracle like the uncut ones, and the forward's outputs do."""
    import oracle
    from paper_2605_08962_amd import binding, workloads as W
    from tests._util import LSE_ABS, assert_close, assert_gradients_close, to_f64, upload
    w = W.make_custom(lengths, Hq, Hkv, D, causal, seed=5200 + D, with_dout=True)
    d, T = upload(w), sum(lengths)
    x = (d["q"], d["k"], d["v"])
    plain = binding.varlen_attn_fwd(*x, d["cu"], causal, w.scale, kv_splits=1)
    ref = binding.varlen_attn_bwd(d["dout"], *x, *plain, d["cu"], causal, w.scale)
    ro, rlse = oracle.fwd(w.f32("q"), w.f32("k"), w.f32("v"), w.cu_seqlens, causal, w.scale)
    for hint in (max(lengths), 1025, 1 << 20, T):
        print(f"case {lengths} Hq={Hq} Hkv={Hkv} D={D} causal={causal} hint={hint}", flush=True)
        got = binding.varlen_attn_bwd(d["dout"], *x, *plain, d["cu"], causal, w.scale, max_seqlen=hint, kv_splits=1)
        assert all(torch.equal(a, b) for a, b in zip(got, ref))
        p = binding.make_params(T, len(lengths), Hq, Hkv, D, causal, w.scale, 0, hint)
        p1 = binding.make_params(T, len(lengths), Hq, Hkv, D, causal, w.scale, 1, hint)
        assert binding.bwd_workspace_bytes(p) > binding.bwd_workspace_bytes(p1)        # the automatic choice cuts
        o, lse = binding.varlen_attn_fwd(*x, d["cu"], causal, w.scale, max_seqlen=hint)
        assert_close("O", to_f64(o), ro, allow_output_rounding=True)
        assert float(abs(to_f64(lse) - rlse).max()) <= LSE_ABS
        got = binding.varlen_attn_bwd(d["dout"], *x, *plain, d["cu"], causal, w.scale, max_seqlen=hint)
        assert_gradients_close(f"hint {hint}", tuple(to_f64(t) for t in got), w.f32("q"), w.f32("k"), w.f32("v"),
                               w.f32("dout"), w.cu_seqlens, causal, w.scale, to_f64(plain[0]), allow_output_rounding=True)


@pytest.mark.parametrize("L,B,H,D,causal", [(640, 12, 5, 64, False), (640, 12, 5, 80, True), (640, 12, 3, 96, False),
                                               (600, 14, 3, 128, False)])
def test_even_batches_without_the_hint_are_not_cut_where_their_tiles_fill_the_chip(L, B, H, D, causal):
    """No walk is longer than the work there is for a CU anyway: the bits of the uncut call."""
    from paper_2605_08962_amd import binding
    lengths = [L] * B
    T, sc = sum(lengths), D ** -0.5
    print(f"case {lengths} D={D} causal={causal}", flush=True)
    q, k, v = _qkv(T, H, H, D, D)
    assert binding.fwd_workspace_bytes(binding.make_params(T, len(lengths), H, H, D, causal, sc)) > 2 * T * H * D * 4
    got = binding.varlen_attn_fwd(q, k, v, _cu(*lengths), causal, sc)
    ref = binding.varlen_attn_fwd(q, k, v, _cu(*lengths), causal, sc, kv_splits=1)
    assert all(torch.equal(a, b) for a, b in zip(got, ref))

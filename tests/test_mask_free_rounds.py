"""The mask-free loop's rounds of written-out steps: every remainder of the six-step round, with and without a ragged end,
and a running maximum that has to move at any step of a round (each later key tile's scores exceed all earlier ones by more
than the 2^30 that a step takes on trust).  Against the same attention in 64 bits.  And the backward over the same lengths: its
first steps, which only their own tiles' loads are waited for; dK/dV in slices (head_dim 64, 80 and 96 beside the forward's cases,
which have too few tiles for anything else), and whole: steady steps and, at head_dim 64, rounds of the stages, with a second
head of the group behind them, from the work list, in small launches uncut, and in chunks.

Bounds: the suite's (O 1e-2 and 5e-3 relative RMS, LSE 1e-3).  Where the maximum moves, scores reach hundreds and LSE is held to
an fp32 ulp of its size times the handful of operations that form it, 1e-3 + 4e-7 * max |LSE|."""
import numpy as np
import pytest
import torch

from tests._util import assert_close, assert_gradients_close, to_f64

pytestmark = pytest.mark.gpu


def _reference(q, k, v, lens, causal, scale):
    o, lse, at = torch.zeros_like(q), torch.zeros(q.shape[1], q.shape[0], dtype=q.dtype), 0
    for n in lens:
        for h in range(q.shape[1]):
            s = scale * q[at:at + n, h] @ k[at:at + n, 0].T
            if causal:
                s = s.masked_fill(~torch.tril(torch.ones(n, n, dtype=torch.bool)), float("-inf"))
            lse[h, at:at + n] = torch.logsumexp(s, -1)
            o[at:at + n, h] = torch.softmax(s, -1) @ v[at:at + n, 0]
        at += n
    return o, lse


@pytest.mark.parametrize("D", [64, 80, 96, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("hint,splits", [(0, 1), (1000, 1), (0, 0)])  # general, lean and small form
def test_every_remainder_of_a_round(D, causal, hint, splits):
    from paper_2605_08962_amd import binding
    gen = torch.Generator().manual_seed(D)
    lens = [512, 513, 576, 640, 703, 704, 768, 832, 895, 896, 960]  # 8..15 tiles of 64 keys, whole and ragged
    if hint == 0 and splits == 1:
        lens.append(1153)
    T, scale = sum(lens), D ** -0.5
    q, k, v = (torch.randn(T, h, D, generator=gen).to(torch.bfloat16) for h in (2, 1, 1))
    do = torch.randn(T, 2, D, generator=gen).to(torch.bfloat16)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32).cuda()
    o, lse = binding.varlen_attn_fwd(q.cuda(), k.cuda(), v.cuda(), cu, causal, scale, max_seqlen=hint, kv_splits=splits)
    grads = binding.varlen_attn_bwd(do.cuda(), q.cuda(), k.cuda(), v.cuda(), o, lse, cu, causal, scale, kv_splits=splits)
    ro, rl = _reference(q.double(), k.double(), v.double(), lens, causal, scale)
    assert_close("O", to_f64(o), ro.numpy(), allow_output_rounding=causal)
    assert float((lse.double().cpu() - rl).abs().max()) <= 1e-3
    assert_gradients_close(f"D={D}", [to_f64(g) for g in grads], *(x.float().numpy() for x in (q, k, v, do)), cu.cpu().numpy(),
                           causal, scale, to_f64(o), allow_output_rounding=True)


@pytest.mark.parametrize("D", [64, 80, 96, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("form", ["list", "whole", "cut"])
def test_every_remainder_of_the_backwards_rounds(D, causal, form):
    from paper_2605_08962_amd import binding
    gen = torch.Generator().manual_seed(20 + D)
    lens = [512, 513, 576, 640, 703, 704, 768, 832, 895, 896, 960, 1153]  # 8..19 steps of 64 queries
    if form == "list":
        lens += [2] * 54  # more than 64 samples
    hq, hkv = (4, 1) if form == "cut" else (4, 2)
    T, scale, hint = sum(lens), D ** -0.5, 1153 if form == "cut" else 0
    p = binding.make_params(T, len(lens), hq, hkv, D, causal, scale, max_seqlen=hint)
    tiles, blocks = binding.max_work_items(p, 1), (D + 31) // 32
    if form == "whole":
        assert tiles * hkv * blocks > 256 and tiles * hq <= 512  # no slices, and a small launch
    q, k, v, do = (torch.randn(T, h, D, generator=gen).to(torch.bfloat16) for h in (hq, hkv, hkv, hq))
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32).cuda()
    o, lse = binding.varlen_attn_fwd(q.cuda(), k.cuda(), v.cuda(), cu, causal, scale)
    args = do.cuda(), q.cuda(), k.cuda(), v.cuda(), o, lse, cu, causal, scale
    grads = binding.varlen_attn_bwd(*args, max_seqlen=hint)
    if form == "cut":  # (sums of chunks are not the bits of whole walks)
        whole = binding.varlen_attn_bwd(*args, max_seqlen=hint, kv_splits=1)
        assert not torch.equal(grads[1], whole[1]) and not torch.equal(grads[2], whole[2])
    assert_gradients_close(f"D={D} {form}", [to_f64(g) for g in grads], *(x.float().numpy() for x in (q, k, v, do)), cu.cpu().numpy(),
                           causal, scale, to_f64(o), allow_output_rounding=True)


@pytest.mark.parametrize("D", [64, 80, 96, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("first", [1, 2, 3, 4, 5, 6])
def test_the_maximum_moves_at_any_step_of_a_round(D, causal, first):
    """From key tile `first` on, every third tile of 64 keys lies 40 (2^57) above everything before it."""
    from paper_2605_08962_amd import binding
    gen = torch.Generator().manual_seed(10 * D + first)
    n, scale = 64 * 14 + 9, D ** -0.5
    q, k, v = (torch.randn(n, h, D, generator=gen) for h in (2, 1, 1))
    q[:, :, 0] = 8.0  # one channel carries the steps
    k[:, :, 0] = 0.0
    for step, tile in enumerate(range(first, 14, 3)):
        k[64 * tile:, :, 0] = 40.0 * (step + 1) / (8.0 * scale)
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    cu = torch.tensor([0, n], dtype=torch.int32).cuda()
    ro, rl = _reference(q.double(), k.double(), v.double(), [n], causal, scale)
    for hint, splits in ((0, 1), (1000, 1), (0, 0)):
        o, lse = binding.varlen_attn_fwd(q.cuda(), k.cuda(), v.cuda(), cu, causal, scale, max_seqlen=hint, kv_splits=splits)
        assert_close(f"O, hint {hint}, kv_splits {splits}", to_f64(o), ro.numpy(), allow_output_rounding=True)
        assert float((lse.double().cpu() - rl).abs().max()) <= 1e-3 + 4e-7 * float(rl.abs().max())

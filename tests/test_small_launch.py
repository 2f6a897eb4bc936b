"""GPU parity of launches that do not fill the chip: tiles found from cu_seqlens without a work list, walks cut into
chunks whose fp32 results a second kernel combines (csrc/va_small.h).  Against the fp64 oracle at the stated bounds, at
the edges of the path: one tile and its neighbours, samples that end just past a tile or a step, empty samples, 64
samples (one per lane) and 65 (the work list again), and cuts that fall inside a query head of a GQA group."""
import pytest
import torch

from paper_2605_08962_amd import workloads as W
from tests._util import LSE_ABS, assert_close, assert_gradients_close, to_f64, upload

pytestmark = pytest.mark.gpu

CASES = [  # lengths, Hq, Hkv, D, causal
    ([1], 1, 1, 64, False), ([128, 0, 129], 2, 1, 128, True), ([127, 1, 64, 65, 0], 2, 2, 96, False),
    ([1500], 2, 2, 64, False), ([1601], 2, 2, 80, True), ([2049], 1, 1, 128, False), ([1793, 0, 1, 130], 4, 1, 128, True),
    ([1090, 1025], 2, 1, 96, True), ([1100, 700], 4, 2, 80, False), ([2000], 3, 1, 64, True),
    ([1100] + [3] * 63, 1, 1, 64, True), ([1100] + [3] * 64, 1, 1, 64, True),
]


@pytest.mark.parametrize("lengths,Hq,Hkv,D,causal", CASES)
def test_small_launch_matches_oracle(lengths, Hq, Hkv, D, causal):
    import numpy as np
    import oracle
    from paper_2605_08962_amd import binding
    w = W.make_custom(lengths, Hq, Hkv, D, causal, seed=900 + len(lengths) + D, with_dout=True)
    hint = max(lengths)
    print(f"case B={len(lengths)} T={w.total_tokens} Hq={Hq} Hkv={Hkv} D={D} causal={causal} max_seqlen={hint}", flush=True)
    d = upload(w)
    o, lse = binding.varlen_attn_fwd(d["q"], d["k"], d["v"], d["cu"], causal, w.scale, max_seqlen=hint)
    ro, rlse = oracle.fwd(w.f32("q"), w.f32("k"), w.f32("v"), w.cu_seqlens, causal, w.scale)
    assert_close("O", to_f64(o), ro, allow_output_rounding=True)
    assert float(np.abs(to_f64(lse) - rlse).max()) <= LSE_ABS
    grads = [binding.varlen_attn_bwd(d["dout"], d["q"], d["k"], d["v"], o, lse, d["cu"], causal, w.scale, max_seqlen=h)
             for h in (hint, hint, 0)]
    torch.cuda.synchronize()
    # the same call twice gives the same bits; with and without the cut agree as two roundings of one sum do
    assert all(torch.equal(a, b) for a, b in zip(grads[0], grads[1]))
    for a, b in zip(grads[0], grads[2]):
        assert float((a.float() - b.float()).norm()) <= 5e-3 * float(b.float().norm()) + 1e-6
    assert_gradients_close(f"small {D}", tuple(to_f64(t) for t in grads[0]), w.f32("q"), w.f32("k"), w.f32("v"),
                           w.f32("dout"), w.cu_seqlens, causal, w.scale, to_f64(o), allow_output_rounding=True)


def test_backward_is_cut_only_where_the_caller_names_long_samples():
    from paper_2605_08962_amd import binding
    size = lambda T, B, hint: binding.bwd_workspace_bytes(binding.make_params(T, B, 4, 1, 128, True, 0.1, 0, hint))
    assert size(8192, 1, 8192) > size(8192, 1, 0) == size(8192, 1, 1024)
    assert size(8192, 65, 8192) == size(8192, 65, 0)              # more samples than lanes
    assert size(60000, 1, 60000) == size(60000, 1, 0)             # fills the chip

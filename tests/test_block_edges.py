"""GPU parity at the edges of what a wave computes: samples that end at, before and behind the 32-row halves of a step,
the waves of a 128-row tile and the tiles themselves, in batches that go by the work list, with and without the hint
that selects the lean forward, against the fp64 oracle at the stated bounds; heads on both sides of the rule for the
order of short samples."""
import pytest
import torch

from paper_2605_08962_amd import workloads as W
from tests._util import LSE_ABS, assert_close, assert_gradients_close, to_f64, upload

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 129, 159, 160, 161, 192, 193, 224, 225, 256, 257]


@pytest.mark.parametrize("Hq,Hkv", [(2, 1), (8, 8)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [64, 80, 96, 128])
def test_samples_ending_at_block_edges(D, causal, Hq, Hkv):
    import numpy as np
    import oracle
    from paper_2605_08962_amd import binding
    lengths = EDGES + [2] * (70 - len(EDGES))  # more than 64 samples: the work list
    w = W.make_custom(lengths, Hq, Hkv, D, causal, seed=4100 + D + causal, with_dout=True)
    print(f"case D={D} causal={causal} Hq={Hq} Hkv={Hkv} T={w.total_tokens}", flush=True)
    d = upload(w)
    runs = []
    for hint in (0, max(lengths)):  # (kv_splits = 1: the hint may split the keys of so small a batch otherwise)
        o, lse = binding.varlen_attn_fwd(d["q"], d["k"], d["v"], d["cu"], causal, w.scale, kv_splits=1, max_seqlen=hint)
        runs.append((o, lse) + binding.varlen_attn_bwd(d["dout"], d["q"], d["k"], d["v"], o, lse, d["cu"], causal, w.scale,
                                                       max_seqlen=hint))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*runs))
    o, lse, *grads = runs[0]
    ro, rlse = oracle.fwd(w.f32("q"), w.f32("k"), w.f32("v"), w.cu_seqlens, causal, w.scale)
    assert_close("O", to_f64(o), ro, allow_output_rounding=True)
    assert float(np.abs(to_f64(lse) - rlse).max()) <= LSE_ABS
    assert_gradients_close(f"edges {D}", tuple(to_f64(t) for t in grads), w.f32("q"), w.f32("k"), w.f32("v"), w.f32("dout"),
                           w.cu_seqlens, causal, w.scale, to_f64(o), allow_output_rounding=True)

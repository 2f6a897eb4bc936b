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

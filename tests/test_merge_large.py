"""Merges of more than 256 MB, parts and result together, read and write past the caches: the same bits, row for row, as the
small merge of any stretch of tokens, empty parts (NaN behind an LSE of -inf) included; on both sides of the limit, for
every number of parts with a kernel of its own and one beyond, at every head_dim."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,T,H,D,past", [
    (3, 65536, 8, 64, False), (3, 65537, 8, 64, True), (1, 105001, 5, 128, True), (2, 111900, 5, 80, True),
    (4, 34953, 8, 96, True), (4, 178572, 3, 64, True), (5, 29200, 8, 96, True), (6, 48001, 5, 80, True),
    (7, 65537, 2, 128, True), (8, 29130, 8, 64, True), (9, 34960, 3, 128, True), (9, 34952, 3, 128, False)])
def test_large_merge_equals_the_merges_of_its_stretches(P, T, H, D, past):
    from paper_2605_08962_amd import binding
    assert ((P + 1) * T * H * D * 2 > 256 << 20) == past
    print(f"case large merge P={P} T={T} H={H} D={D}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(P * T)
    o = torch.randn((P, T, H, D), generator=gen, device="cuda").to(torch.bfloat16)
    lse = torch.randn((P, H, T), generator=gen, device="cuda") * 3
    empty = torch.rand((P, H, T), generator=gen, device="cuda") < 0.2
    empty[:, :, :3] = True
    lse[empty] = float("-inf")
    o[empty.transpose(1, 2)] = float("nan")
    got_o, got_lse = binding.varlen_attn_merge(o, lse)
    for lo, hi in ((0, 1000), (T // 2, T // 2 + 77), (T - 1001, T)):
        ref_o, ref_lse = binding.varlen_attn_merge(o[:, lo:hi].contiguous(), lse[:, :, lo:hi].contiguous())
        assert torch.equal(got_o[lo:hi], ref_o) and torch.equal(got_lse[:, lo:hi], ref_lse)
    assert not got_o.isnan().any() and bool((got_o[:3] == 0).all())

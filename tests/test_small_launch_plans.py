"""What launches that do not fill the chip are planned to take, as far as it shows in the workspace sizes (CPU)."""
import pytest

from paper_2605_08962_amd import binding


@pytest.mark.parametrize("T,Hq,Hkv,D,causal", [(8191, 4, 1, 128, True), (16383, 2, 2, 128, True), (16383, 1, 1, 128, True),
                                               (20000, 4, 1, 64, True), (8192, 2, 2, 80, False)])
def test_one_sample_is_cut_the_same_with_and_without_the_hint(T, Hq, Hkv, D, causal):
    """The length of a single sample is known to be total_tokens: max_seqlen adds nothing."""
    size = lambda hint: binding.fwd_workspace_bytes(binding.make_params(T, 1, Hq, Hkv, D, causal, 0.1, 0, hint))
    assert size(0) == size(T) > 2 * T * Hq * D * 4


@pytest.mark.parametrize("lengths,H,D,cut", [([8192] + [16] * 20, 2, 64, True), ([8192] + [16] * 20, 2, 128, True),
                                             ([8192] + [16] * 10, 2, 64, True), ([8192] + [64] * 16, 2, 64, True),
                                             ([1200] + [16] * 40, 2, 64, False), ([129, 64, 37, 16], 2, 64, False)])
def test_one_long_sample_among_short_ones_is_cut_without_the_hint(lengths, H, D, cut):
    """Room for two parts and more although the average is short; not where it is under 256 tokens."""
    T = sum(lengths)
    size = binding.fwd_workspace_bytes(binding.make_params(T, len(lengths), H, H, D, False, 0.1))
    assert (size > 2 * T * H * D * 4) == cut

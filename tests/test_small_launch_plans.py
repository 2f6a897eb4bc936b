"""What launches that do not fill the chip are planned to take, as far as it shows in the workspace sizes (CPU)."""
import pytest

from paper_2605_08962_amd import binding


@pytest.mark.parametrize("T,Hq,Hkv,D,causal", [(8191, 4, 1, 128, True), (16383, 2, 2, 128, True), (16383, 1, 1, 128, True),
                                               (20000, 4, 1, 64, True), (8192, 2, 2, 80, False)])
def test_one_sample_is_cut_the_same_with_and_without_the_hint(T, Hq, Hkv, D, causal):
    """The length of a single sample is known to be total_tokens: max_seqlen adds nothing."""
    size = lambda hint: binding.fwd_workspace_bytes(binding.make_params(T, 1, Hq, Hkv, D, causal, 0.1, 0, hint))
    assert size(0) == size(T) > 2 * T * Hq * D * 4

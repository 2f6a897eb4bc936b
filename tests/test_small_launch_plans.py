"""What launches that do not fill the chip are planned to take, as far as it shows in the workspace sizes, and in which order (CPU)."""
import os
import subprocess

import pytest

from paper_2605_08962_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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


def test_samples_are_taken_longest_first(tmp_path):
    exe = str(tmp_path / "length_order_check")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-o", exe, os.path.join(ROOT, "tests", "length_order_check.hip")], check=True,
                   capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "length order ok" in r.stdout, r.stdout

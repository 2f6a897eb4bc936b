"""What launches that do not fill the chip are planned to take, as far as it shows in the workspace sizes, and in which order (CPU)."""
import os
import re
import struct
import subprocess
import tempfile

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


def _kernel_scratch_bytes():
    """{mangled kernel name: bytes of scratch memory per lane} from the metadata of the built library's device code."""
    lib = open(os.path.join(ROOT, "paper_2605_08962_amd", "libvarlen_attn.so"), "rb").read()
    magic, out, at = b"__CLANG_OFFLOAD_BUNDLE__", {}, 0
    while (at := lib.find(magic, at)) >= 0:
        n, pos = struct.unpack_from("<Q", lib, at + 24)[0], at + 32
        for _ in range(n):
            ofs, size, idlen = struct.unpack_from("<QQQ", lib, pos)
            if b"gfx950" in lib[pos + 24:pos + 24 + idlen]:
                with tempfile.NamedTemporaryFile(suffix=".elf") as f:
                    f.write(lib[at + ofs:at + ofs + size])
                    f.flush()
                    notes = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", f.name], check=True,
                                           capture_output=True, text=True).stdout
                for name, rest in re.findall(r"\.name:\s+(_ZN2va\w+)\n((?:.*\n)*?.*\.private_segment_fixed_size:\s+\d+)", notes):
                    out[name] = int(rest.rsplit(":", 1)[1])
            pos += 24 + idlen
        at += len(magic)
    return out


def test_dq_of_small_launches_keeps_everything_in_registers():
    """Scratch loads in the loop wait for every tile load in flight.  The kernels' last template argument: small launches."""
    scratch = {n: b for n, b in _kernel_scratch_bytes().items() if re.search(r"dq_kernel(_direct)?ILi\d+ELb[01]ELb1E", n)}
    assert len(scratch) == 8 and not any(scratch.values()), scratch


@pytest.mark.parametrize("T,B,H,D,causal,hint,cut", [
    (39540, 30, 1, 128, True, 1318, False), (20061, 9, 2, 128, True, 2229, False),   # the chip is full of them uncut
    (9415, 9, 4, 96, False, 9199, True), (3126, 2, 4, 80, False, 1563, True), (1343, 1, 8, 64, False, 1343, True),
    (4096, 1, 2, 128, True, 4096, True)])
def test_backward_is_cut_where_that_pays(T, B, H, D, causal, hint, cut):
    size = lambda splits: binding.bwd_workspace_bytes(binding.make_params(T, B, H, H, D, causal, 0.1, splits, hint))
    assert (size(0) > size(1)) == cut


@pytest.mark.parametrize("T,B,H,D,by_list", [(6141, 3, 8, 80, True), (30294, 9, 3, 64, True), (30000, 10, 2, 96, True),
                                             (10770, 2, 2, 64, False), (5083, 17, 2, 96, False), (6141, 3, 2, 128, False)])
def test_causal_batches_of_long_samples_keep_the_order_of_the_list(T, B, H, D, by_list):
    """Causal forward with many tiles to a CU: as the work list has it, not cut; elsewhere the plan cuts."""
    size = lambda splits: binding.fwd_workspace_bytes(binding.make_params(T, B, H, H, D, True, 0.1, splits))
    assert (size(0) == size(1)) == by_list

"""The order in which workgroups take a batch of short samples: a permutation of (item, head) for every shape (CPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_short_sample_order_is_a_permutation(tmp_path):
    exe = str(tmp_path / "work_order_check")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-o", exe, os.path.join(ROOT, "tests", "work_order_check.hip")], check=True,
                   capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "work order ok" in r.stdout, r.stdout

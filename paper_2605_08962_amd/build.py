"""Builds libvarlen_attn.so from csrc/ with hipcc for gfx950 (cross-compiles without a GPU), and the native half of the Python
binding with g++ against torch."""
import glob
import hashlib
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libvarlen_attn.so")
HOST_SOURCES = [os.path.join(CSRC, "va_host.cpp"), os.path.join(HERE, "..", "include", "varlen_attn.h")]
# (source, object name, extra flags).  va_bwd.hip is built in parts, each under the instruction-scheduling strategy that
# measured best for its kernels among the default, iterative-ilp, iterative-minreg, iterative-maxocc, max-ilp and
# max-memory-clause (64 ViT samples, 16 heads, unless said otherwise; the forward does best with the default):
#   dQ iterative-ilp: LLM batch at head_dim 128 7 % faster than the default, 64 without the mask even, causal 1.3-3 %; head_dim
#     96 1.6 %; 80 29.6 against 31.6 ms (65536 tokens and 256 short samples).
#   dK/dV at 128, causal: iterative-ilp 7 % (iterative-maxocc: batches of 64..1024 tokens 1058 against 985 us); without the
#     mask iterative-maxocc 10.58 -> 10.23 ms, 8 x 8192 tokens 7.61 -> 7.30 ms.
#   dK/dV at 96: iterative-maxocc, 8.92 -> 8.41 ms.  At 80: iterative-minreg, 1 % (iterative-ilp: 8 % slower).
# dK/dV at 96 and 128 are also told to let MFMAs write S and dP into ordinary vector registers: they run one wave per SIMD on
# more than 256 registers, and the default puts every MFMA result into the accumulation half of the register file, from
# where the vector ALU needs a copy per register (64 per step; 5 % of the time at 128, 9.52 -> 8.41 ms at 96).
_SCHED = "-amdgpu-sched-strategy="
_VGPR_FORM = ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
SOURCES = [("va_api.hip", "va_api.o", []), ("va_sched.hip", "va_sched.o", []), ("va_fwd.hip", "va_fwd.o", []),
           ("va_bwd.hip", "va_bwd.o", ["-DVA_BWD_PART=0"]),
           ("va_bwd.hip", "va_bwd_dkdv128c.o", ["-DVA_BWD_PART=1", "-mllvm", _SCHED + "iterative-ilp", *_VGPR_FORM]),
           ("va_bwd.hip", "va_bwd_dq.o", ["-DVA_BWD_PART=2", "-mllvm", _SCHED + "iterative-ilp"]),
           ("va_bwd.hip", "va_bwd_dkdv80.o", ["-DVA_BWD_PART=3", "-mllvm", _SCHED + "iterative-minreg"]),
           ("va_bwd.hip", "va_bwd_dkdv128.o", ["-DVA_BWD_PART=4", "-mllvm", _SCHED + "iterative-maxocc", *_VGPR_FORM]),
           ("va_partition.hip", "va_partition.o", []), ("va_merge.hip", "va_merge.o", [])]
# -packed-fp32-ops is switched off on purpose: hipcc must not form v_pk_*_f32 from float code.
# -fno-honor-nans: the kernels never produce NaN from finite inputs (masked scores use a finite
# sentinel), and without it every fmaxf of an MFMA result costs an extra canonicalising v_max.
# -Wno-inline-asm: the direct-to-LDS load statements name M0 as clobbered (they overwrite it); clang remarks
# on every one of them that M0 is a reserved register it will not save, which is exactly what is meant.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
         "-fno-honor-nans",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(item):
    src, objname, extra = item
    obj = os.path.join(CSRC, "_build", objname)
    cmd = ["hipcc", *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(ln for ln in r.stderr.splitlines() if "packed-fp32-ops" not in ln)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def compile_host(source, target):
    """A CPython module from `source` against the installed torch."""
    import torch
    t = os.path.dirname(torch.__file__)
    inc = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include",
           sysconfig.get_paths()["include"]]  # (system headers: warnings are of our own source)
    # (under its own name only when whole: another process may be loading the old one)
    tmp = f"{target}.{os.getpid()}"
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Wextra", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                    f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(f"-isystem{d}" for d in inc),
                    source, "-o", tmp, "-L" + os.path.join(t, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"],
                   check=True)
    os.replace(tmp, target)
    return target


def host_path():
    """Where the native half of the binding belongs.  It reaches into torch's and CPython's objects, so its name says what it was
    built from and for: one that does not match what runs is never loaded."""
    import torch
    h = hashlib.sha256()
    for path in HOST_SOURCES:
        with open(path, "rb") as f:
            h.update(f.read())
    return os.path.join(HERE, f"_varlen_attn_host.{sysconfig.get_config_var('SOABI')}.torch-{torch.__version__}."
                              f"{h.hexdigest()[:12]}.so")


def build_host():
    """The native half of the binding, in place of an older one for the same torch and interpreter; returns its path."""
    path = compile_host(HOST_SOURCES[0], host_path())
    for old in glob.glob(glob.escape(path[:-len("123456789012.so")]) + "?" * 12 + ".so"):
        if old != path:
            os.remove(old)
    return path


def build():
    os.makedirs(os.path.join(CSRC, "_build"), exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        host = ex.submit(build_host)
        objs = list(ex.map(_compile, SOURCES))
        host.result()
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
    return LIB


if __name__ == "__main__":
    print(build())

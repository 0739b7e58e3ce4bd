"""Compile the HIP sources under csrc/ into paper_2006_06762_amd/libanr.so for gfx950, and the binding's extension module.

Run as ``python -m paper_2006_06762_amd.build`` (hipcc cross-compiles without a GPU).
"""
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libanr.so")
NATIVE = os.path.join(HERE, "_native.so")       # the binding's extension module (csrc/binding_native.cpp)

SOURCES = ["api.cpp", "gemm.hip", "tbg.hip", "conv_direct.hip", "conv_igemm.hip", "conv_gather.hip", "conv_pieces.hip", "conv_pointwise.hip", "conv_stem.hip", "dwconv.hip", "nrm.hip", "static_scratch.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
    # packed fp32 instructions are kept off on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# Per-file flags.  The convolution and GEMM kernels keep their MFMA accumulators in ordinary vector
# registers instead of the accumulation registers: prologues and epilogues then need no copies
# between the two register files.  Measured: 0.25-0.35 us per launch on the three benchmark
# convolutions, 1-2 % on the general convolution kernels, 6-10 % on GEMMs of 512^3 x 16 and
# 2048^3; no gain on the attention kernels, which are left alone.
FILE_FLAGS = {
    "conv_igemm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
    "conv_gather.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
    "conv_pieces.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
    "conv_stem.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
    "gemm.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
}


def _compile(src, verbose, extra):
    out = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc"] + FLAGS + FILE_FLAGS.get(src, []) + list(extra) + ["-c", os.path.join(CSRC, src), "-o", out]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass warns that it does not know the packed-fp32 feature: harmless
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, res.stderr))
    if verbose and err.strip():
        print(err, flush=True)
    return out


def _build_native(verbose):
    import torch
    at = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-isystem", os.path.join(at, "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "binding_native.cpp"),
           "-o", NATIVE, "-L", os.path.join(at, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


def build(verbose: bool = False, extra=()) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        native = ex.submit(_build_native, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose, extra), SOURCES))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    native.result()
    return LIB


def _stale() -> bool:
    """True when the library or the extension module is missing or older than any source they are built from."""
    if not all(os.path.exists(f) for f in (LIB, NATIVE)):
        return True
    built = min(os.path.getmtime(f) for f in (LIB, NATIVE))
    srcs = [os.path.join(CSRC, f) for f in os.listdir(CSRC)]
    inc = os.path.join(ROOT, "include")
    srcs += [os.path.join(inc, f) for f in os.listdir(inc)]
    return any(os.path.getmtime(f) > built for f in srcs if os.path.isfile(f))


def ensure_built(verbose: bool = False) -> str:
    """Build the library unless a built one is there that is newer than every file under
    csrc/ and include/ (tests, the smoke run and the benchmark load what is built)."""
    if not _stale():
        return LIB
    if not shutil.which("hipcc"):
        if os.path.exists(LIB) and os.path.exists(NATIVE):
            return LIB      # a box without the compiler runs what was shipped
        raise RuntimeError("libanr.so or _native.so is missing and hipcc is not on PATH")
    return build(verbose=verbose)


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))

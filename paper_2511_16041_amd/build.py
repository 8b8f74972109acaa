"""Build libatb.so (HIP kernels + C ABI) for gfx950 with hipcc, and the binding's extension module with g++, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libatb.so")
EXT = os.path.join(HERE, "_launch.so")           # the binding's extension module (csrc/atb_binding.cpp)
OBJ_DIR = os.path.join(HERE, "_build")
# accumulators stay in ordinary vector registers: with up to 470 of a wave's 512 in use the compiler otherwise parks other
# values in the accumulation half and moves the accumulators out and in again around every panel (208 moves to 64 MFMAs)
SKINNY_FLAGS = ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
# loops of the 128-row tiles begin on a line of the instruction cache: the same instructions some bytes further on cost the 64,128,64,128
# tile with B in BFP16 4 % (706 x 4992 x 3880 50.4 -> 52.5 us); the other forms of these tiles are level (the 64 x 64 tiles lose 2 % by it)
ALIGNED = ["-falign-loops=64"]
# (source, object name, extra flags): the GEMM instance table is cut into three groups that compile side by side
SOURCES = [("atb_gemm.hip", "atb_gemm_g0", ["-DATB_GROUP=0"]), ("atb_gemm.hip", "atb_gemm_g1", ["-DATB_GROUP=1"] + ALIGNED),
           ("atb_gemm.hip", "atb_gemm_g2", ["-DATB_GROUP=2"]), ("atb_skinny.hip", "atb_skinny", SKINNY_FLAGS), ("atb_bfp16.hip", "atb_bfp16", []), ("atb_probe.hip", "atb_probe", []),
           ("atb_model.cpp", "atb_model", []), ("atb_api.cpp", "atb_api", [])]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    # packed fp32 VALU forms are kept out of the generated code on this machine pool
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-attributes",
]


def _compile(item, extra, verbose: bool) -> str:
    src, name, flags = item
    obj = os.path.join(OBJ_DIR, name + ".o")
    lang = ["-x", "hip"]
    cmd = [HIPCC] + COMMON + list(flags) + list(extra) + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return obj


def build_binding(verbose: bool = False) -> str:
    """The extension module that checks operands and launches; host code only, against torch's headers and libraries."""
    import sysconfig
    import torch
    from torch.utils.cpp_extension import include_paths
    includes = include_paths() + [sysconfig.get_paths()["include"], "/opt/rocm/include"]
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    for d in includes:
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, "atb_binding.cpp"), "-o", EXT, "-L" + libs, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return EXT


def build(verbose: bool = False, extra=()) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    build_binding(verbose)
    with ThreadPoolExecutor(max_workers=6) as ex:
        objs = list(ex.map(lambda s: _compile(s, extra, verbose), SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return OUT


def build_microbench(verbose: bool = False) -> str:
    """The unit-cost micro-benchmark behind the constants of atb_model_microkernel (a developer
    tool, a stand-alone executable; nothing loads it)."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    exe = os.path.join(OBJ_DIR, "unit_costs")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wno-unused-command-line-argument", "-o", exe, os.path.join(CSRC, "microbench", "unit_costs.hip")]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return exe


def _stale() -> bool:
    """True if the library or the extension module is missing or older than any of the sources (or this file)."""
    if not os.path.exists(OUT) or not os.path.exists(EXT):
        return True
    built = min(os.path.getmtime(OUT), os.path.getmtime(EXT))
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if os.path.isfile(os.path.join(CSRC, f))]
    deps += [os.path.join(ROOT, "include", "atb.h"), os.path.abspath(__file__)]
    return any(os.path.getmtime(d) > built for d in deps)


def ensure_built() -> str:
    """Path of the library; builds it first if it is missing or a source is newer than it.  (A stale
    library that cannot be rebuilt because there is no compiler is an error, not a silent fallback.)"""
    if _stale():
        build()
    return OUT


if __name__ == "__main__":
    extra = [a for a in sys.argv[1:] if a != "--microbench"]
    print(build(verbose=True, extra=extra))
    if "--microbench" in sys.argv:
        print(build_microbench(verbose=True))

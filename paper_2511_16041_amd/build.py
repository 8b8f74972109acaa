"""Build libatb.so (HIP kernels + C ABI) for gfx950 with hipcc, and the binding's extension module with g++, in-tree.  The library needs
neither torch nor Python's headers; only the extension module does."""
from __future__ import annotations

import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libatb.so")
BINDING_SOURCE = "atb_binding.cpp"
OBJ_DIR = os.path.join(HERE, "_build")
# accumulators stay whole where they are carried round a loop: taken apart (as the compiler does with vectors that begin as constants), each
# of their registers is moved once per round (212 moves to 64 MFMAs in atb_rows; in atb_skinny 0.99 to 1.05 x: 500 x 4096 x 4096 B^T 34.0 -> 32.9 us)
WHOLE_PHIS = ["-mllvm", "-amdgpu-codegenprepare-break-large-phis=0"]
# accumulators stay in ordinary vector registers: with up to 470 of a wave's 512 in use the compiler otherwise parks other
# values in the accumulation half and moves the accumulators out and in again around every panel (208 moves to 64 MFMAs)
SKINNY_FLAGS = ["-mllvm", "-amdgpu-mfma-vgpr-form=1"] + WHOLE_PHIS
# loops of the 128-row tiles begin on a line of the instruction cache: the same instructions some bytes further on cost the 64,128,64,128
# tile with B in BFP16 4 % (706 x 4992 x 3880 50.4 -> 52.5 us); the other forms of these tiles are level (the 64 x 64 tiles lose 2 % by it)
ALIGNED = ["-falign-loops=64"]
# (source, object name, extra flags): the GEMM instance table is cut into three groups that compile side by side
SOURCES = [("atb_gemm.hip", "atb_gemm_g0", ["-DATB_GROUP=0"]), ("atb_gemm.hip", "atb_gemm_g1", ["-DATB_GROUP=1"] + ALIGNED),
           ("atb_gemm.hip", "atb_gemm_g2", ["-DATB_GROUP=2"]), ("atb_skinny.hip", "atb_skinny", SKINNY_FLAGS), ("atb_rows.hip", "atb_rows", WHOLE_PHIS), ("atb_bfp16.hip", "atb_bfp16", []), ("atb_probe.hip", "atb_probe", []),
           ("atb_model.cpp", "atb_model", []), ("atb_api.cpp", "atb_api", [])]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    # packed fp32 VALU forms are kept out of the generated code: some of them have given wrong results
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


def binding_path() -> str:
    """The extension module.  Its name holds the Python and the torch that it is built against, so that another of either builds its own."""
    import torch
    return os.path.join(HERE, f"_launch.{sysconfig.get_config_var('SOABI')}.torch-{torch.__version__}.so")


def build_binding(verbose: bool = False) -> str:
    """The extension module that checks operands and launches; host code only, against torch's headers and libraries."""
    import torch
    from torch.utils.cpp_extension import include_paths
    out = binding_path()
    part = f"{out}.{os.getpid()}"                  # several processes may build it at once; each puts a whole file in place
    rocm = os.path.dirname(os.path.dirname(shutil.which(HIPCC) or HIPCC))
    includes = include_paths() + [sysconfig.get_paths()["include"], os.path.join(rocm, "include")]
    includes += [d for d in include_paths("cuda") if d not in includes]          # torch's ROCm, where HIPCC is not inside one
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    for d in includes:
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, BINDING_SOURCE), "-o", part, "-L" + libs, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(part, out)
    return out


def build_library(verbose: bool = False, extra=()) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=6) as ex:
        objs = list(ex.map(lambda s: _compile(s, extra, verbose), SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return OUT


def build(verbose: bool = False, extra=()) -> str:
    """The library, and the extension module where there is a torch to build it against."""
    build_library(verbose, extra)
    if importlib.util.find_spec("torch") is not None:
        build_binding(verbose)
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


def _older(out: str, sources) -> bool:
    """True if a built file is missing or older than any of its sources (or this file)."""
    return not os.path.exists(out) or any(os.path.getmtime(d) > os.path.getmtime(out) for d in [*sources, os.path.abspath(__file__)])


def _stale() -> bool:
    """True if the library is missing or older than any of its sources (or this file)."""
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f != BINDING_SOURCE and os.path.isfile(os.path.join(CSRC, f))]
    return _older(OUT, deps + [os.path.join(ROOT, "include", "atb.h")])


def ensure_built() -> str:
    """Path of the library; builds it first if it is missing or a source is newer than it.  (A stale
    library that cannot be rebuilt because there is no compiler is an error, not a silent fallback.)"""
    if _stale():
        build_library()
    return OUT


def ensure_binding() -> str:
    """Path of the extension module, likewise."""
    out = binding_path()
    if _older(out, [os.path.join(CSRC, BINDING_SOURCE)]):
        build_binding()
    return out


if __name__ == "__main__":
    extra = [a for a in sys.argv[1:] if a != "--microbench"]
    print(build(verbose=True, extra=extra))
    if "--microbench" in sys.argv:
        print(build_microbench(verbose=True))

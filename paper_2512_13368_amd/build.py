"""Builds libblossom.so in-tree with hipcc for gfx950 (cross-compiles without a GPU), and the binding's host module."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libblossom.so")
FASTCALL = os.path.join(HERE, "_fastcall.so")
OBJ_DIR = os.path.join(HERE, "_build")

# per-file extra flags; select.hip decides integers from fp32 arithmetic and must not be
# contracted into fused operations the source does not spell out
SOURCES = {
    "api.hip": [],
    "select.hip": ["-ffp-contract=off"],
    "select_pos.hip": ["-ffp-contract=off"],
    "generic.hip": [],
    # accumulators of the matrix instructions stay in VGPRs: the online softmax rescales them
    # with VALU instructions, and AGPR placement costs a register copy per element per tile
    # (the forward kernel also reuses its bf16 staging rows as fp32 exchange space between wavefronts)
    "mfma_fwd.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1", "-fno-strict-aliasing"],
    "mfma_fwd4.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1", "-fno-strict-aliasing"],
    "mfma_f32.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
    "mfma_f32_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],  # (the same source, bf16 storage)
    "mfma_bwd.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
    "probe.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
    "out_proj.hip": ["-fno-strict-aliasing"],
}

COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc() -> str:
    for c in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.isabs(c) and not os.path.exists(c):
            continue
        return c
    return "hipcc"


def fastcall_command(obj: str) -> list[str]:
    """Compiles csrc/fastcall.cpp: host code only, against the headers of the installed torch and Python."""
    import sysconfig

    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    return [_hipcc(), "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem", inc, "-isystem",
            sysconfig.get_paths()["include"], "-isystem", "/opt/rocm/include", "-c", os.path.join(CSRC, "fastcall.cpp"), "-o", obj]


def _run(cmd: list[str], what: str, verbose: bool = False) -> None:
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{r.stdout}\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr)


def build_fastcall() -> str:
    """Compiles and links the binding's host module: needs torch and the library, which does not need it."""
    import torch
    os.makedirs(OBJ_DIR, exist_ok=True)
    obj = os.path.join(OBJ_DIR, "fastcall.o")
    _run(fastcall_command(obj), "compilation of fastcall.cpp")
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    _run([_hipcc(), "-shared", "-fPIC", "-o", FASTCALL, obj, "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
          "-L" + os.path.dirname(LIB), "-lblossom", "-Wl,-rpath,$ORIGIN"], "link of _fastcall.so")
    return FASTCALL


def build_library(verbose: bool = False) -> str:
    """Compiles and links libblossom.so, the C ABI: HIP sources alone."""
    os.makedirs(OBJ_DIR, exist_ok=True)

    def compile_one(item):
        src, extra = item
        obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
        _run([_hipcc(), *COMMON, *extra, "-c", os.path.join(CSRC, src), "-o", obj], f"hipcc on {src}", verbose)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES.items()))
    _run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], "link of libblossom.so")
    return LIB


def build_all(verbose: bool = False) -> None:
    """The library first: a host module that does not build leaves it in place."""
    print(build_library(verbose))
    print(build_fastcall())


if __name__ == "__main__":
    build_all(verbose=True)

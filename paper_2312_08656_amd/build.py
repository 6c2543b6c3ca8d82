"""Builds libmaxk.so for gfx950 with hipcc, and the marshalling of torch tensors with the host compiler, in-tree (next to this file)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

HERE = Path(__file__).resolve().parent
CSRC = HERE / "csrc"
LIB = HERE / "libmaxk.so"
TORCH_CALLS = HERE / "_torch_calls.so"
SOURCES = ["graph.hip", "topk.hip", "spgemm_fwd.hip", "spgemm_fwd_f32.hip", "spgemm_fwd_bf16.hip", "spgemm_fwd_f16.hip",
           "sspmm_bwd.hip", "sspmm_bwd_f32.hip", "sspmm_bwd_bf16.hip", "sspmm_bwd_f16.hip", "sspmm_bwd_tiled.hip", "sspmm_bwd_regs.hip",
           "sspmm_bwd_regs_f32.hip", "sspmm_bwd_regs_bf16.hip", "sspmm_bwd_regs_f16.hip", "spmm.hip"]

# -packed-fp32-ops off: the compiler must not form packed fp32 instructions from float code
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-Wno-unused-result",
]


def build_torch_calls(verbose: bool = False) -> None:
    """The marshalling of torch tensors (host code): an extension module next to this file."""
    import sysconfig

    import torch

    home = Path(torch.__file__).resolve().parent
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = TORCH_CALLS.with_suffix(".so.tmp%d" % os.getpid())
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", "-DTORCH_EXTENSION_NAME=_torch_calls",
           f"-I{home}/include", f"-I{home}/include/torch/csrc/api/include", f"-I{rocm}/include", f"-I{sysconfig.get_paths()['include']}",
           str(CSRC / "torch_calls.cpp"), f"-L{home}/lib", "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", "-ltorch_hip", "-o", str(tmp)]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        subprocess.check_call(cmd)
        os.replace(tmp, TORCH_CALLS)
    finally:
        tmp.unlink(missing_ok=True)


def try_torch_calls(verbose: bool = False) -> bool:
    """build_torch_calls where the host has a compiler and torch's headers; without the module every call is marshalled in Python."""
    try:
        build_torch_calls(verbose)
        return True
    except (OSError, subprocess.CalledProcessError) as e:
        TORCH_CALLS.unlink(missing_ok=True)  # (one of another build may not fit this library)
        print(f"{TORCH_CALLS.name} not built, calls are marshalled in Python: {e}", file=sys.stderr, flush=True)
        return False


def build(verbose: bool = False) -> Path:
    """Compile every translation unit and link the shared library (always rebuilds)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    extra = os.environ.get("MAXK_HIPCC_EXTRA", "").split()  # e.g. -DMAXK_FWD_COPY_PAD=4 for an experiment build
    objdir = HERE / "_build"
    objdir.mkdir(exist_ok=True)

    def compile_one(src: str) -> Path:
        obj = objdir / (src + ".o")
        cmd = [hipcc, *HIPCC_FLAGS, *extra, "-c", str(CSRC / src), "-o", str(obj)]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 4)) as ex:
        calls = ex.submit(try_torch_calls, verbose)
        objs = list(ex.map(compile_one, SOURCES))
        calls.result()
    tmp = LIB.with_suffix(".so.tmp%d" % os.getpid())
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *map(str, objs), "-o", str(tmp)]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

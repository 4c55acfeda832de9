"""Builds libsk.so (HIP, gfx950 only) in-tree with hipcc.

    python -m paper_2601_15473_amd.build

Cross-compiles without a GPU.  Objects go to csrc/_build/ (not committed); the
library lands in lib/ next to this file, where the ctypes binding looks for it.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "lib", "libsk.so")
OUT_TORCH = os.path.join(HERE, "lib", "_sktorch.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCES = ["sk_api.hip", "sk_bf16_gemm.hip", "sk_bf16_gemm256.hip", "sk_bf16_few_rows.hip",
           "sk_f32_gemm.hip", "sk_chain.hip", "sk_bwd_narrow.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU forms are kept off on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


# Per-source extras.  The chain kernels read every accumulator exactly once in their
# epilogues, so MFMA results go straight to VGPRs there (the option crashes this
# compiler on the 256x256 GEMM, whose accumulators need the AGPR file anyway).
EXTRA = {"sk_chain.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def _compile(src: str, obj: str) -> None:
    cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines()
                    if "packed-fp32-ops" not in l and "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")


def build_torch(verbose: bool = True) -> str:
    """The PyTorch layers' native functions: host code against torch's headers, linked to libsk.so beside it."""
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    include = os.path.join(root, "include")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unknown-pragmas",
           "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1", f'-DSK_TORCH_VERSION="{torch.__version__}"', f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           "-isystem", include, "-isystem", os.path.join(include, "torch", "csrc", "api", "include"),
           "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "sk_torch.cpp"), OUT, "-L" + os.path.join(root, "lib"),
           "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python", "-Wl,-rpath,$ORIGIN", "-o", OUT_TORCH]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on sk_torch.cpp:\n" + r.stderr)
    if r.stderr.strip():
        sys.stderr.write(r.stderr)
    if verbose:
        print(f"built {OUT_TORCH}")
    return OUT_TORCH


def build(verbose: bool = True) -> str:
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    bdir = os.path.join(CSRC, "_build")
    os.makedirs(bdir, exist_ok=True)
    objs = [os.path.join(bdir, s.replace(".hip", ".o")) for s in SOURCES]
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        list(ex.map(_compile, SOURCES, objs))
    # (a name of its own: what links to it finds the file beside itself, not the path it was built at)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-soname,libsk.so", *objs, "-o", OUT],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print(f"built {OUT}")
    try:
        import torch  # noqa: F401
    except ImportError:   # (libsk.so serves callers without PyTorch)
        print(f"no PyTorch here: {OUT_TORCH} not built")
    else:
        build_torch(verbose)
    return OUT


if __name__ == "__main__":
    build()

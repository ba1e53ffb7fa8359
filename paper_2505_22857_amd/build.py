"""Build of the HIP library ``libngpu_lm.so`` for gfx950 with hipcc, and of the
binding's per-call module ``_fastcall.so`` against the installed torch."""

from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libngpu_lm.so")
FAST_PATH = os.path.join(HERE, "_fastcall.so")
SOURCES = ["api.cpp", "trie_build.cpp", "arpa.cpp", "advance.hip", "fused_step.hip", "decode.hip", "topk.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",                      # no contraction beyond the explicit fmaf
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    path = os.path.join(rocm, "bin", "hipcc")
    return path if os.path.exists(path) else "hipcc"


def build(out: str = LIB_PATH, extra=(), verbose: bool = False) -> str:
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    cmd = [hipcc(), *HIPCC_FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           "-o", out + ".tmp", *srcs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(out + ".tmp", out)
    return out


def build_fastcall(out: str = FAST_PATH, verbose: bool = False) -> str:
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DNGPU_TORCH_VERSION="{torch.__version__}"',
           *[x for p in include_paths("cuda") for x in ("-isystem", p)],
           "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"),
           os.path.join(CSRC, "fastcall.cpp"), *[f"-L{p}" for p in library_paths("cuda") if os.path.isdir(p)],
           "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-o", out + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(out + ".tmp", out)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_fastcall(verbose=True))

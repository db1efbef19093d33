"""Build libmage.so (the C-ABI HIP library, hipcc for gfx950) and _marshal.so (the Python binding's argument
marshalling, host compiler) in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmage.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
SOURCES = ["mage_api.hip", "attn_bf16.hip", "sparse_bf16.hip", "sparse_batch_bf16.hip", "sparse_few_bf16.hip", "attn_f32.hip", "reduce.hip", "topk.hip", "quest.hip", "diag.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xarch_host", "-fPIC", "-shared",   # position-independent code for the host side only (the device code objects need none)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU ops
    # no NaN ever enters the arithmetic (masked scores are -inf, never inf - inf), so max/min need no
    # quieting canonicalisation; infinities stay honoured
    "-fno-honor-nans", "-mno-amdgpu-ieee",
    "-Wall", "-Wno-unused-function",
]


def marshal_command() -> list[str]:
    import torch
    root = os.path.dirname(torch.__file__)
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM", "-w",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-I", os.path.join(root, "include"), "-I", os.path.join(root, "include", "torch", "csrc", "api", "include"),
            "-I", "/opt/rocm/include", "-I", sysconfig.get_paths()["include"],
            "-o", MARSHAL, os.path.join(CSRC, "marshal.cpp"),
            "-L", HERE, "-lmage", "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip",
            "-Wl,-rpath,$ORIGIN"]


def build(verbose: bool = False, extra: list[str] | None = None) -> str:
    _run(["hipcc", *FLAGS, *(extra or []), "-o", LIB, *[os.path.join(CSRC, s) for s in SOURCES]], verbose)
    _run(marshal_command(), verbose)
    return LIB


def _run(cmd: list[str], verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + out)
    if verbose and out.strip():
        print(out, flush=True)


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))

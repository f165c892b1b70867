"""Compile libckv.so (gfx950, hipcc) and the torch binding _ckv_binding.so in-tree.
`python -m paper_2506_11418_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libckv.so")
BINDING = os.path.join(HERE, "_ckv_binding.so")
SOURCES = ["ckv_host.hip", "k1_match.hip", "k2_select.hip", "k3_merge.hip", "k4_attn.hip", "k4_attn_f32.hip", "k5_round.hip", "k6_paged.hip", "k7_mfma_ceiling.hip", "ckv_noalloc.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 code generation
    "-Wall", "-Wno-unused-function", "-Wno-unknown-pragmas",
]


def build_library(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{res.stdout}\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return LIB


def build_binding(verbose: bool = True) -> str:
    """csrc/binding.cpp: host code against torch's tensor headers; torch's libraries are loaded when it is imported."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", os.path.join(ROOT, "include")]
    for d in [*cpp_extension.include_paths(), sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, "binding.cpp"), "-o", BINDING]
    for d in cpp_extension.library_paths():
        cmd += ["-L", d]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed ({res.returncode}):\n{res.stdout}\n{res.stderr}")
    return BINDING


if __name__ == "__main__":
    print(build_library())
    print(build_binding())

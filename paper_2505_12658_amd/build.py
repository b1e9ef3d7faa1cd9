"""Builds the HIP library and its Python binding in-tree:
  hipcc --offload-arch=gfx950 -> paper_2505_12658_amd/libhydra_attn.so    (the C ABI and the kernels)
  g++                         -> paper_2505_12658_amd/_hydra_torch.so     (torch tensors -> C ABI, host code only)

hipcc cross-compiles without a GPU.  Run as `python -m paper_2505_12658_amd.build`.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "hydra_api.hip")
LIB = os.path.join(HERE, "libhydra_attn.so")
BINDING_SRC = os.path.join(HERE, "csrc", "torch_binding.cpp")
BINDING = os.path.join(HERE, "_hydra_torch.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    # packed fp32 VALU forms are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-shared",
    "-fPIC",
]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass warns that it does not know the device-only target feature
    out = "\n".join(line for line in res.stdout.splitlines() if "packed-fp32-ops" not in line)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + out)
    if verbose and out.strip():
        print(out)


def _binding_command():
    import torch

    root = os.path.join(os.path.dirname(torch.__file__))
    include, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
            "-isystem", sysconfig.get_paths()["include"], "-isystem", include, "-isystem", os.path.join(include, "torch", "csrc", "api", "include"),
            "-isystem", "/opt/rocm/include", BINDING_SRC, "-o", BINDING,
            f"-L{lib}", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python"]


def build(verbose: bool = False) -> str:
    _run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + HIPCC_FLAGS + [SRC, "-o", LIB], verbose)
    _run(_binding_command(), verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)

"""Builds libdfa.so (the HIP kernels and the C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_PKG, "csrc")
INCLUDE = os.path.join(os.path.dirname(_PKG), "include")
LIB_PATH = os.path.join(_PKG, "libdfa.so")
# named for the interpreter it is built with: another one does not find it, and says so, instead of failing inside it
TORCH_MODULE_PATH = os.path.join(_PKG, "_dfa_torch" + sysconfig.get_config_var("EXT_SUFFIX"))

SOURCES = ["dfa_api.hip", "dfa_fwd_bf16.hip", "dfa_fwd_short.hip", "dfa_fwd_f32.hip", "dfa_bwd.hip", "dfa_bwd_bf16.hip", "dfa_bwd_short.hip", "dfa_linear_bf16.hip", "dfa_dense.hip", "dfa_aux.hip", "dfa_probe.hip", "dfa_plan.cpp"]


def hipcc_command(out: str = LIB_PATH, extra=()):
    return ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
            # keep the compiler from forming packed-fp32 instructions
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wno-unused-command-line-argument",
            # the LDS-copy asm names m0 as clobbered; clang notes that it treats m0 as reserved anyway
            "-Wno-inline-asm",
            "-I", INCLUDE, *extra, "-o", out] + [os.path.join(CSRC, s) for s in SOURCES]


def torch_module_command(out: str = TORCH_MODULE_PATH):
    """g++ command of the module that takes torch tensors to libdfa.so (host code only)."""
    import torch
    root = os.path.dirname(torch.__file__)
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-I", INCLUDE, "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
            "-isystem", sysconfig.get_paths()["include"], "-isystem", "/opt/rocm/include", os.path.join(CSRC, "dfa_torch.cpp"), "-o", out,
            "-L", os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def build(verbose: bool = False) -> str:
    """Compiles every source into libdfa.so and the torch module beside it, both at once; raises on failure."""
    jobs = [(what, cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
            for what, cmd in (("libdfa.so", hipcc_command()), ("the torch module", torch_module_command()))]
    results = [(what, cmd, job.communicate()[0], job.returncode) for what, cmd, job in jobs]
    for what, cmd, output, code in results:
        if verbose or code != 0:
            print(" ".join(cmd))
            print(output)
    failed = [what for what, _, _, code in results if code != 0]
    if failed:
        raise RuntimeError(f"building {' and '.join(failed)} failed")
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))

"""Builds libintfa.so (hand-written HIP for gfx950) with hipcc and the binding's host module with the host compiler, in-tree."""
from __future__ import annotations

import os
import subprocess

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(_HERE), "include")
LIB = os.path.join(_HERE, "libintfa.so")
SOURCES = ["intfa_attention.hip", "intfa_attention_fewq.hip", "intfa_attention_half.hip", "intfa_quantize.hip"]

# Packed-fp32 instructions are switched off on purpose (the flag is a device-side feature; the host
# pass warns that it does not know it, which is harmless).  No fast-math: the quantizer is bit-exact.
# Loops start at multiples of 32 bytes: where the 4 KB body of the fused kernel's key loop lies relative to the
# instruction fetch is worth 4 % (32 heads x 8192 x 128 causal, start moved in steps of 4 bytes: 348 - 363 us, with a
# period of 32 bytes; 350 at a multiple), and without the flag every change in front of a loop moves it.
# It helps two workgroups that share a CU (32 x 8192 x 128 without the mask, half-INT8 942 -> 918 us; INT8 64 x 4096 339 -> 334) and costs one
# that is alone on it, i.e. calls whose last wave leaves most CUs half empty (half-INT8 36 x 4096 308 -> 319, INT8 12 x 8192 269 -> 275 - 283).
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-ffp-contract=off", "-falign-loops=32", "-Wall", "-Wno-unused-command-line-argument"]


# The binding's plain calls (host code only): a CPython module on torch's C++ interface.
HOST_SRC = os.path.join(CSRC, "intfa_host.cpp")
HOST_LIB = os.path.join(_HERE, "_intfa_host.so")


def _host_command():
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")))
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DINTFA_TORCH_VERSION="{torch.__version__}"', "-I", INCLUDE, "-isystem", os.path.join(root, "include"),
            "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"], "-Wall", HOST_SRC, "-o", HOST_LIB,
            "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_hip", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def build(verbose: bool = False, extra_flags=()) -> str:
    """libintfa.so and, beside it, the host module."""
    host_cmd = _host_command()
    if verbose:
        print(" ".join(host_cmd), flush=True)
    host = subprocess.Popen(host_cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *extra_flags, "-I", INCLUDE, "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(ln for ln in res.stdout.splitlines() if "packed-fp32-ops" not in ln)
    host_out = host.communicate()[0]
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if host.returncode != 0:
        raise RuntimeError(f"{host_cmd[0]} failed:\n" + host_out)
    if verbose and (out + host_out).strip():
        print(out + host_out)
    return LIB


MICROBENCH_SRC = os.path.join(CSRC, "microbench", "issue_model.hip")
MICROBENCH_BIN = os.path.join(_HERE, "issue_model_microbench.bin")


def build_microbench(verbose: bool = False) -> str:
    """The stand-alone issue-model micro-benchmark (register-only probes of the MFMA / vector ALU / exp pipes)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-Wall", "-Wno-unused-command-line-argument", MICROBENCH_SRC, "-o", MICROBENCH_BIN]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(ln for ln in res.stdout.splitlines() if "packed-fp32-ops" not in ln)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    return MICROBENCH_BIN


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_microbench(verbose=True))

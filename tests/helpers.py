"""Shared test helpers: build quantized Algorithm-1 inputs from the seeded workloads using the
ORACLE's quantizer (never the HIP path's), so expected values depend on oracle/ alone."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

import oracle
import workloads


def quantized_inputs(w, heads=None, scaled=False):
    """Real Q, K, V of workload `w` -> dict with int8 tensors and scales [heads, ...].
    scaled=True folds 1/sqrt(d) into s_Q (exact by the linearity remark of Section 3.2)."""
    Q = workloads.tensor(w, "Q", heads)
    K = workloads.tensor(w, "K", heads)
    V = workloads.tensor(w, "V", heads)
    Qq, sQ = oracle.quantize_tokenwise(Q)
    Kq, sK = oracle.quantize_tokenwise(K)
    Vq, sV = oracle.quantize_headwise(V)
    if scaled:
        sQ = (sQ * np.float32(1.0 / np.sqrt(w.d))).astype(np.float32)
    return {"Q": Q, "K": K, "V": V, "Qq": Qq, "Kq": Kq, "Vq": Vq, "sQ": sQ, "sK": sK, "sV": sV}


def dequant(q, s):
    return q.astype(np.float64) * np.asarray(s, np.float64)[..., None]


def random_int8_problem(rng, heads, N, d, score_sigma=1.0):
    """Random int8 Q, K, V with scales chosen so that scores have standard deviation ~score_sigma."""
    Qq = rng.integers(-127, 128, (heads, N, d), dtype=np.int8)
    Kq = rng.integers(-127, 128, (heads, N, d), dtype=np.int8)
    Vq = rng.integers(-127, 128, (heads, N, d), dtype=np.int8)
    base = score_sigma / (73.3 * 73.3 * np.sqrt(d))      # std of uniform int8 ~ 73.3
    sQ = (rng.uniform(0.5, 1.5, (heads, N)) * np.sqrt(base)).astype(np.float32)
    sK = (rng.uniform(0.5, 1.5, (heads, N)) * np.sqrt(base)).astype(np.float32)
    sV = rng.uniform(0.005, 0.02, heads).astype(np.float32)
    return Qq, Kq, Vq, sQ, sK, sV


_RULES = r"""
#include "intfa_internal.h"
#include "intfa_device.h"
extern "C" int route(int heads, int Nq, int Nk, int d, int causal, int vblock) { return ifa_fwd_kernel(heads, Nq, Nk, d, causal, vblock); }
extern "C" int few_half(int heads, int Nq, int Nk, int d) { return ifa_few_queries(heads, Nq, Nk, d, true); }
extern "C" int unsplit(int heads, int Nq, int Nk, int d) { return ifa_unsplit_queries(heads, Nq, Nk, d); }
extern "C" int wavefronts(int heads, int Nq, int Nk, int d, int causal, int half) {
    if (half) return ifa_half_wavefronts(heads, Nq, Nk, d, causal, ifa_dev::head_group_for(causal, 3L * Nk * d, 0));
    return ifa_fused_wavefronts(heads, Nq, Nk, d, causal, ifa_dev::head_group_for(causal, 2L * Nk * d, (Nq + 127) / 128));
}
"""


@functools.lru_cache(maxsize=None)
def library_rules():
    """The library's own dispatch rules, compiled for the host: tests say which kernel they reach without a line of their own."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    with tempfile.TemporaryDirectory() as tmp:
        src, lib = os.path.join(tmp, "rules.hip"), os.path.join(tmp, "rules.so")
        with open(src, "w") as f:
            f.write(_RULES)
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(root, "include"), "-I",
                        os.path.join(root, "paper_2409_16997_amd", "csrc"), src, "-o", lib], check=True, stdout=subprocess.DEVNULL)
        return ctypes.CDLL(lib)


def route(heads, Nq, Nk, d, causal=None, half=False, vblock=False):
    """Which kernel a plain attention call runs: "fused", "few" (twelve wavefronts per 32 queries, half-INT8 eight), "packed" or "pair" (two groups of 32
    queries).  `causal` decides nothing for half-INT8; `vblock`: per-block V scales."""
    if half:
        return "few" if library_rules().few_half(heads, Nq, Nk, d) else "fused"
    assert causal is not None
    return ("fused", "pair", "packed", "few")[library_rules().route(heads, Nq, Nk, d, int(causal), int(vblock))]


def unsplit(heads, Nq, Nk, d):
    """Whether a call of the key-split entry points runs the kernel of the plain call."""
    return bool(library_rules().unsplit(heads, Nq, Nk, d))


def wavefronts(heads, Nq, Nk, d, causal, half=False):
    """Wavefronts per SIMD of the fused kernel (half-INT8: of its own) for a call that runs it."""
    assert route(heads, Nq, Nk, d, causal, half) == "fused"
    return library_rules().wavefronts(heads, Nq, Nk, d, int(causal), int(half))


def copies_for(kernel, heads, Nq, Nk, d, causal=None, half=False):
    """How many copies of these heads make a call that runs `kernel`, "fused" or "pair"; None if no number does."""
    first = -(-(513 if kernel == "fused" else 257) // (heads * -(-Nq // 32)))
    return next((c for c in range(first, 4 * first + 1) if route(heads * c, Nq, Nk, d, causal, half) == kernel), None)


def copies_for_the_fused_kernel(heads, Nq, Nk, d, causal=None, half=False):
    return copies_for("fused", heads, Nq, Nk, d, causal, half)


def many(copies, *arrays):
    """`copies` copies of the heads of each array, one after the other."""
    return [np.concatenate([a] * copies) for a in arrays]


def first_copy(O, copies):
    """What the first copy of the heads got, as a host array; every copy must have got the same."""
    o = O.reshape(copies, -1)
    assert bool((o == o[:1]).all()), "copies of a head differ"
    return o[0].cpu().numpy()

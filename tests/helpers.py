"""Shared test helpers: build quantized Algorithm-1 inputs from the seeded workloads using the
ORACLE's quantizer (never the HIP path's), so expected values depend on oracle/ alone."""
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


def route(heads, Nq, Nk, d, causal=None, half=False):
    """Which kernel a plain attention call runs: "fused", "few" (twelve wavefronts per 32 queries, half-INT8 eight), "packed" or "pair" (two groups of 32
    queries).  `causal` decides nothing for half-INT8.  tests/test_routes.py holds this to the library's own rule."""
    groups = heads * -(-Nq // 32)
    if not half:
        assert causal is not None
        if Nq > 32 and groups > 256:
            wgs, uneven = heads * -(-Nq // 64), causal and 2 * Nq >= Nk
            if wgs <= 256:
                pair = Nk >= (512 if d == 128 else 384) and not (uneven and Nk >= 2048 and (heads == 1 or wgs <= 192))
            else:
                line = 4 * wgs - 100 if d == 128 else 3 * wgs - 200
                if wgs <= 512:
                    pair = causal and 4 * Nq >= Nk >= line and (uneven or Nk >= (3000 if d == 128 else 2048))
                else:
                    pair = uneven and Nk >= 2048 and heads * Nk <= 56 << 10 and (heads <= 8 and wgs <= 768 or wgs <= 576 and Nk >= (4000 if d == 128 else 3000))
            if pair:
                return "pair"
        if Nk <= 128 if groups <= 256 else d == 64 and (Nk <= (768 if groups <= 1024 else 1152) if Nq <= 32 else
                                                        Nq <= 64 and groups <= 512 and 128 <= Nk < 384):
            return "packed"
    short_keys = {(True, 128): 256, (True, 64): 64, (False, 128): 384, (False, 64): 0}[half, d]
    if groups <= 5 << 20 and (groups <= 256 or (Nk > short_keys if Nq <= 32 else groups <= 512 and Nk >= 2048)):
        return "few"
    return "fused"


def unsplit(heads, Nq, Nk, d):
    """Whether a call of the key-split entry points runs the kernel of the plain call.  tests/test_routes.py holds this to the library's own rule."""
    if heads <= (64 if d == 128 else 128) and (Nq == 1 or Nq <= 8 and Nk > 384):      # the decode kernel's
        return Nk <= 3000 + 75 * heads or heads >= 108 if Nq == 1 else Nk <= 2000 + (86 + 4 * Nq) * heads or heads >= 120 - 3 * Nq
    if Nq <= 8:
        E, S, H = (2048, 1536, 134 - 5 * Nq) if d == 128 else (1024, 1536, 146 - 7 * Nq)
    else:
        E, S, H = 1024, 2304, (104 if d == 128 else 122) - Nq
    return Nk <= 2048 or heads * (Nk + E) >= H * (Nk - S)


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

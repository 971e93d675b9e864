"""The work this library is used for, as cases that can be timed: each goes from the activations (or the quantized cache)
a caller holds to the attention output, through the public Python entry points of paper_2409_16997_amd.

Two kinds of call:
  prefill  Nq queries that come with their own keys and values (Nq = Nk), real activations in: Section 3.2's quantizers,
           then the attention call.  The quantized K and V are the cache the caller keeps, so they are outputs too.
  cached   Nq new queries (a decode step, a few draft tokens, a chunk of a long prompt) against Nk keys that already sit
           quantized in the cache, under the mask the last Nq positions: quantize the new Q, then the attention call.
           The cache and, for the key-split call, its workspace are what the program keeps between steps.
`variant` is the scheme for P and V: "full" (INT8, one V scale per head), "vblock" (INT8, one V scale per 128 keys),
"half" (fp16 weights and V), "hadamard" (full, on Hadamard-rotated Q and K).  `call` says which attention entry point a
cached call goes through: "fwd" (int_flash_attn_fwd or its half form), "splitk" (the program's own workspace) or
"static" (the built-in one).
"""
import math

import torch

import paper_2409_16997_amd as ifa

DTYPES = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"fp32": 4, "fp16": 2, "bf16": 2}


def _case(name, kind, B, H, Nq, Nk, d, causal, dtype, variant="full", call="fwd", dist="normal"):
    c = {"kind": kind, "B": B, "H": H, "Nq": Nq, "Nk": Nk, "d": d, "causal": causal, "dtype": dtype, "variant": variant,
         "call": call, "dist": dist}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one short head, fp32 in and out: the smallest call, launches and host work only
        _case("one_head_128", "prefill", 1, 1, 128, 128, 64, False, "fp32"),
        # an encoder layer: short sequences, d = 64, no mask
        _case("encoder_1024", "prefill", 4, 16, 1024, 1024, 64, False, "fp16"),
        # the headline prefill of a decoder layer
        _case("prefill_4096", "prefill", 4, 32, 4096, 4096, 128, True, "fp16"),
        # a batch of long documents without a mask, outlier channels: the largest call
        _case("documents_8192", "prefill", 8, 32, 8192, 8192, 128, False, "fp16", dist="uniform_outlier"),
        # one very long heavy-tailed prompt, which is what the per-block V scales are for
        _case("long_vblock_16384", "prefill", 1, 32, 16384, 16384, 128, True, "fp16", "vblock", dist="student_t3"),
        # prompts of an everyday length that is a multiple of nothing, bf16, head count not a multiple of the 8 XCDs
        _case("ragged_bf16_1777", "prefill", 3, 12, 1777, 1777, 128, True, "bf16"),
        # the headline prefill in the half-INT8 variant
        _case("half_4096", "prefill", 4, 32, 4096, 4096, 128, True, "fp16", "half"),
        # the next chunk of a long prompt against the cache
        _case("chunk_512_of_8192", "cached", 1, 32, 512, 8192, 128, True, "fp16"),
        # a decode step of a batch, long context, key-split call
        _case("decode_batch_16384", "cached", 4, 32, 1, 16384, 128, True, "fp16", call="splitk"),
        # a decode step of one sequence through the plain attention call
        _case("decode_one_4099", "cached", 1, 32, 1, 4099, 128, True, "fp16"),
        # verification of 16 draft tokens of one sequence, key-split call on the built-in workspace
        _case("draft_16_of_8192", "cached", 1, 32, 16, 8192, 128, True, "bf16", call="static"),
        # a decode step of a batch in the half-INT8 variant
        _case("decode_half_4096", "cached", 4, 32, 1, 4096, 128, True, "fp16", "half"),
    ]


def _log(rng, lo, hi):
    """An integer between lo and hi, even over the logarithm."""
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


MOST_OPS = 8.0e12            # below documents_8192
MOST_BYTES = 2.0e9
MOST_STATIC = (32, 8192)     # heads and keys that the built-in workspace holds at up to 32 queries per head


def draw(rng):
    """Another case of the same ranges: any length (most of them ragged), 1 to 256 heads, both head sizes, every scheme."""
    while True:
        d, dtype = rng.choice([64, 128, 128]), rng.choice(["fp16", "fp16", "bf16", "fp32"])
        B, H = rng.choice([1, 1, 2, 3, 4, 8]), rng.choice([1, 4, 8, 12, 16, 32, 32])
        dist = rng.choice(["normal", "normal", "uniform_outlier", "student_t3"])
        if rng.random() < 0.5:
            N = _log(rng, 128, 16384)
            if rng.random() < 0.3:
                N = max(128, N // 128 * 128)
            variant = rng.choice(["full", "full", "full", "vblock", "half", "hadamard"])
            if variant == "half":
                dtype = "fp16"
            c = _case(None, "prefill", B, H, N, N, d, rng.random() < 0.6, dtype, variant, dist=dist)
        else:
            variant = rng.choice(["full", "full", "full", "half", "vblock"])
            Nk = _log(rng, 256, 32768)
            Nq = rng.choice([1, 1, 1, rng.randint(2, 8), rng.randint(9, 32), _log(rng, 33, 2048)])
            call = rng.choice(["fwd", "splitk", "splitk", "static"]) if variant == "full" and Nq <= 32 else "fwd"
            if Nq > Nk or (call == "static" and (B * H > MOST_STATIC[0] or Nk > MOST_STATIC[1])):
                continue
            c = _case(None, "cached", B, H, Nq, Nk, d, True, dtype if dtype != "fp32" else "fp16", variant, call, dist)
            if variant == "half":
                c["dtype"] = "fp16"
        w = work(c)
        if w["flops"] <= MOST_OPS and w["bytes"] <= MOST_BYTES:
            return c


def _activations(shape, case, g):
    dev = g.device
    if case["dist"] == "normal":
        x = torch.randn(shape, device=dev, generator=g, dtype=torch.float32)
    elif case["dist"] == "uniform_outlier":          # U(-0.5, 0.5), four of the channels twenty times as large
        x = torch.rand(shape, device=dev, generator=g, dtype=torch.float32).sub_(0.5)
        x[..., torch.randperm(shape[-1], device=dev, generator=g)[:4]] *= 20.0
    else:                                            # Student-t with 3 degrees of freedom, unit variance
        x = torch.randn(shape, device=dev, generator=g, dtype=torch.float32)
        chi2 = torch.randn(shape, device=dev, generator=g, dtype=torch.float32).square_()
        for _ in range(2):
            chi2.add_(torch.randn(shape, device=dev, generator=g, dtype=torch.float32).square_())
        x.mul_(chi2.rsqrt_().clamp_(max=1e3))
    return x.to(DTYPES[case["dtype"]])


def _block(case):
    return ifa.block_cols(case["d"], case["causal"])


def _quantize_v(V, case):
    """(codes, scale) of V as the attention call of this variant takes it; the half variant keeps V."""
    if case["variant"] == "half":
        return V, None
    return ifa.quantize_blockwise(V, _block(case)) if case["variant"] == "vblock" else ifa.quantize_headwise(V)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, H, Nq, Nk, d = (case[k] for k in ("B", "H", "Nq", "Nk", "d"))
    Q, K, V = (_activations((B, H, n, d), case, g) for n in (Nq, Nk, Nk))
    s = {"case": case, "Q": Q, "fold": d ** -0.5}
    if case["kind"] == "prefill":
        s.update(K=K, V=V)
        return s
    s["k8"], s["sk"] = ifa.quantize_tokenwise(K)     # the cache
    s["v"], s["sv"] = _quantize_v(V, case)
    if case["call"] == "splitk":
        s["workspace"] = torch.empty(ifa.splitk_workspace_bytes(B, H, Nq, Nk, d), dtype=torch.uint8, device="cuda")
    elif case["call"] == "static":
        ifa.lib().ifa_static_workspace_bytes()
        s["workspace"] = "static"
    return s


def run(s):
    case, fold = s["case"], s["fold"]
    causal, out_dtype, variant = case["causal"], DTYPES[case["dtype"]], case["variant"]
    if case["kind"] == "cached":
        q8, sq = ifa.quantize_tokenwise(s["Q"], scale_mul=fold)
        if variant == "half":
            return ifa.int_flash_attn_fwd_half(q8, s["k8"], s["v"], sq, s["sk"], causal=causal, out_dtype=out_dtype)
        if case["call"] == "fwd":
            return ifa.int_flash_attn_fwd(q8, s["k8"], s["v"], sq, s["sk"], s["sv"], causal=causal, out_dtype=out_dtype)
        return ifa.int_flash_attn_fwd_splitk(q8, s["k8"], s["v"], sq, s["sk"], s["sv"], causal=causal, out_dtype=out_dtype,
                                             workspace=s["workspace"])
    Q, K, V = s["Q"], s["K"], s["V"]
    if variant == "full":
        q8, k8, v8, sq, sk, sv = ifa.quantize_qkv(Q, K, V, s_Q_mul=fold)
    else:
        rotated = variant == "hadamard"              # rotating both multiplies Q K^T by d, on top of the 1/sqrt(d)
        q8, k8, sq, sk = ifa.quantize_qk(Q, K, s_Q_mul=fold / case["d"] if rotated else fold, hadamard=rotated)
        v8, sv = _quantize_v(V, case)
    if variant == "half":
        return {"O": ifa.int_flash_attn_fwd_half(q8, k8, v8, sq, sk, causal=causal, out_dtype=out_dtype), "k8": k8, "sk": sk}
    O = ifa.int_flash_attn_fwd(q8, k8, v8, sq, sk, sv, causal=causal, out_dtype=out_dtype)
    return {"O": O, "k8": k8, "v8": v8, "sk": sk, "sv": sv}


def work(case):
    B, H, Nq, Nk, d = (case[k] for k in ("B", "H", "Nq", "Nk", "d"))
    heads, es = B * H, BYTES[case["dtype"]]
    scores = sum(Nk - Nq + i + 1 for i in range(Nq)) if case["causal"] else Nq * Nk
    half, v_scales = case["variant"] == "half", -(-Nk // 128) if case["variant"] == "vblock" else 1
    if case["kind"] == "prefill":                    # Q, K, V in; K and V codes with their scales and O out
        per_head = 3 * Nk * d * es + Nk * d + 4 * Nk + (0 if half else Nk * d + 4 * v_scales) + Nq * d * es
    else:                                            # Q and the cache in, O out
        per_head = 2 * Nq * d * es + Nk * d + 4 * Nk + (2 * Nk * d if half else Nk * d + 4 * v_scales)
    return {"bytes": heads * per_head, "flops": 4.0 * heads * scores * d}


def tolerance(case):
    """Four times the largest difference seen between O and the CPU oracle, which takes exp in 64 bits, over the listed and
    fourteen drawn cases (two seeds, up to two heads each).  What differs is a P within fp32 noise of a half-integer that
    one side rounds up and the other down (a 127th of one weight: most on rows with few keys), and the last bit of O.
    Seen: INT8 weights 2.1e-4 with fp16 or fp32 output and 5.7e-4 with bf16, largest single difference 0.057 of the rms;
    fp16 weights 6.2e-5 and 0.002.  Codes are exact."""
    if case["variant"] == "half":
        return {"rel": 2.5e-4, "max": 0.01, "differ": 0.0}
    return {"rel": 2.3e-3 if case["dtype"] == "bf16" else 8.5e-4, "max": 0.2, "differ": 0.0}

"""The few-query kernels and the fused kernel on the two sides of the dispatcher's rule: the same rows, bit for bit.

A call with many heads runs the fused kernel; the same problem on a few of the heads (or on the last few queries) runs a
few-query kernel.  All perform Algorithm 1 with the same operations on the same operands, so torch.equal is the bar; one
head of each shape is also held to the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from helpers import route, unsplit

pytestmark = pytest.mark.gpu

# (heads, N): more than 512 groups of 32 queries each, so that the whole call is not a few-query kernel's (but the fused one's or, under the mask, the two-group one's).  Lengths at the edges
# of the 128-key block, of the few-query kernel's group of two blocks and of its 32 queries.
SHAPES = [(180, 65), (140, 127), (132, 128), (110, 129), (90, 191), (80, 255), (80, 256), (64, 257), (60, 384), (48, 385), (40, 513), (17, 1100), (30, 1100)]


def problem(heads, N, d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    q8, k8, v8 = (torch.randint(-127, 128, (1, heads, N, d), generator=g, device="cuda", dtype=torch.int8) for _ in range(3))
    base = (2.0 / (73.3 * 73.3 * d ** 0.5)) ** 0.5
    sq, sk = (base * (0.5 + torch.rand((1, heads, N), generator=g, device="cuda")) for _ in range(2))
    return q8, k8, v8, sq, sk


@pytest.mark.parametrize("vblock", [False, True])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,N", SHAPES)
def test_both_kernels_give_the_same_rows(heads, N, d, causal, vblock):
    import paper_2409_16997_amd as ifa
    assert route(heads, N, N, d, causal) in ("fused", "pair") and route(5, N, N, d, causal) == ("packed" if N <= 128 else "few")
    q8, k8, v8, sq, sk = problem(heads, N, d, heads + N)
    Bc = ifa.block_cols(d, causal)
    g = torch.Generator(device="cuda").manual_seed(N)
    sv = 0.005 + 0.02 * torch.rand((1, heads) + ((-(-N // Bc),) if vblock else ()), generator=g, device="cuda")
    call = lambda q, k, v, a, b, c: ifa.int_flash_attn_fwd(q, k, v, a, b, c, causal=causal, out_dtype=torch.float32)
    full = call(q8, k8, v8, sq, sk, sv)
    cut = [t[:, 1:6].contiguous() for t in (q8, k8, v8, sq, sk, sv)]
    assert torch.equal(call(*cut), full[:, 1:6])
    for nq in (1, 31, 32):                                       # the last rows only, all heads
        if causal or nq == 31:
            few = call(q8[:, :, N - nq:].contiguous(), k8, v8, sq[:, :, N - nq:].contiguous(), sk, sv)
            if vblock and causal:
                # a row may share its group with one that sees a block it does not see itself: with one V scale per block
                # its output then goes through one more change of unit, s_a * rcp(s_b) on the way and s_b for s_a at the end
                # (four roundings and a 1-ulp reciprocal: below 2^-21 of the value)
                assert bool(((few - full[:, :, N - nq:]).abs() <= 2.0 ** -21 * full[:, :, N - nq:].abs()).all())
            else:
                assert torch.equal(few, full[:, :, N - nq:])
    n = lambda t: t[0, :1].cpu().numpy()
    res = oracle.compare_up_to_ties(full[0, 0].cpu().numpy(), n(q8), n(k8), n(v8), n(sq), n(sk), n(sv), causal, Bc)
    assert float(res["err"].max()) <= 1e-3 * float(res["scale"])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,N", SHAPES + [(300, 33), (100, 192), (80, 193)])
def test_half_int8_kernels_agree(heads, N, d, causal):
    # the same weights, and both sums in the same order: the same bits
    import paper_2409_16997_amd as ifa
    q8, k8, v8, sq, sk = problem(heads, N, d, heads + N)
    v = v8.to(torch.float16) / 64
    call = lambda q, k, x, a, b: ifa.int_flash_attn_fwd_half(q, k, x, a, b, causal=causal, out_dtype=torch.float32)
    full = call(q8, k8, v, sq, sk)
    assert route(heads, N, N, d, half=True) == "fused" and route(4, N, N, d, half=True) == "few"
    cut = [t[:, 1:5].contiguous() for t in (q8, k8, v, sq, sk)]
    assert torch.equal(call(*cut), full[:, 1:5])
    for nq in (1, 31, 32):
        few = call(q8[:, :, N - nq:].contiguous(), k8, v, sq[:, :, N - nq:].contiguous(), sk)
        assert torch.equal(few, full[:, :, N - nq:]), nq
    n = lambda t: t[0, :1].cpu().numpy()
    ref = oracle.int_flash_attn_fwd_half(n(q8), n(k8), n(v), n(sq), n(sk), causal, ifa.block_cols_half(d, causal))["O"]
    few = call(*[t[:, :1].contiguous() for t in (q8, k8, v, sq, sk)])[0, 0].cpu().numpy()
    assert np.abs(few - ref).max() <= 1e-3 * np.abs(ref).max()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,Nq", [(128, 1), (128, 8), (128, 9), (128, 32), (64, 1), (64, 4), (64, 8), (64, 9), (64, 32)])
def test_key_split_entry_point_on_both_sides_of_its_rule(d, Nq, causal):
    # With many heads, and up to 2048 keys, the entry point runs the kernel of the plain call: the same result, bit for bit.
    # Otherwise the split passes run, which add up O in another order (a few ulp of the
    # largest value; in the last case the last run of key blocks is masked for the early queries).
    import paper_2409_16997_amd as ifa
    cases = [(3, 2048), (3, 2049), (2, 4098)]
    for Nk in (2305, 4096, 4099, 8193) + ((16385,) if Nq in (9, 32) else ()):
        many = next(H for H in range(1, 200) if unsplit(H, Nq, Nk, d))
        cases += [(many, Nk), (max(many - 1, 1), Nk)]
    seen = set()
    for H, Nk in cases:
        q8, k8, v8, sq, sk = problem(H, Nk, d, H + Nk)
        q8, sq = q8[:, :, Nk - Nq:].contiguous(), sq[:, :, Nk - Nq:].contiguous()
        sv = 0.005 + 0.02 * torch.rand((1, H), device="cuda", generator=torch.Generator(device="cuda").manual_seed(Nk))
        ref = ifa.int_flash_attn_fwd(q8, k8, v8, sq, sk, sv, causal=causal, out_dtype=torch.float32)
        need = ifa.splitk_workspace_bytes(1, H, Nq, Nk, d)
        ws = torch.full((need // 4,), float("nan"), device="cuda").view(torch.uint8)
        out = ifa.int_flash_attn_fwd_splitk(q8, k8, v8, sq, sk, sv, causal=causal, out_dtype=torch.float32, workspace=ws)
        same = unsplit(H, Nq, Nk, d)
        seen.add((Nk > 2048, same))
        assert bool(torch.isnan(ws.view(torch.float32)).all()) == same, (H, Nk)          # the passes ran, or not
        if same:
            assert torch.equal(out, ref), (H, Nk)
        else:
            assert float((out - ref).abs().max()) <= 4e-6 * float(ref.abs().max()), (H, Nk)
    assert seen == {(False, True), (True, True), (True, False)}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [128, 161, 200])
def test_half_int8_rows_stay_clear_of_values_they_do_not_see(N, d):
    # V is the caller's fp16 and may hold infinities.  Rows of a 32-query group that see no key of a 32-key tile do not depend on
    # what V holds there, on either kernel (inside the tile that the diagonal crosses 0 * inf is a NaN on both).
    import paper_2409_16997_amd as ifa
    heads = 600                                                  # the whole call: the fused kernel
    q8, k8, v8, sq, sk = problem(heads, N, d, N)
    v = v8.to(torch.float16) / 64
    for key, value in ((40, float("inf")), (97, float("nan")), (N - 1, float("-inf"))):
        bad = v.clone()
        bad[:, :, key] = value
        call = lambda n, x: ifa.int_flash_attn_fwd_half(q8[:, :n].contiguous(), k8[:, :n].contiguous(), x[:, :n].contiguous(), sq[:, :n].contiguous(),
                                                        sk[:, :n].contiguous(), causal=True, out_dtype=torch.float32)
        first = key // 32 * 32                                   # the first row of the first group that sees the tile
        for n in (heads, 2):
            assert torch.equal(call(n, bad)[:, :, :first], call(n, v)[:, :, :first]), (n, key)


@pytest.mark.parametrize("variant,heads", [("full", 6_000_000), ("splitk", 6_000_000), ("half", 9_000_000)])
def test_more_heads_than_one_few_query_launch_holds(variant, heads):
    # 768 (half-INT8: 512) threads per head are more than 2^32 in one launch: such a call takes a kernel with 256
    import paper_2409_16997_amd as ifa
    few, Nk, d = 1000, 2, 64
    q8, k8, v8, sq, sk = problem(few, Nk, d, 5)
    q8, sq = q8[:, :, 1:].contiguous(), sq[:, :, 1:].contiguous()
    v = v8.to(torch.float16) / 64 if variant == "half" else v8
    sv = () if variant == "half" else (0.005 + 0.02 * torch.rand((1, few), device="cuda"),)
    fn = {"full": ifa.int_flash_attn_fwd, "splitk": ifa.int_flash_attn_fwd_splitk, "half": ifa.int_flash_attn_fwd_half}[variant]
    call = lambda *a: fn(*a, causal=True, out_dtype=torch.float32)
    ref = call(q8, k8, v, sq, sk, *sv)
    out = call(*[t.repeat((1, heads // few) + (1,) * (t.dim() - 2)) for t in (q8, k8, v, sq, sk) + sv]).view(heads // few, few, d)
    # (the key-split passes add O up in another order)
    assert float((out - ref.view(1, few, d)).abs().max()) <= 2.0 ** -21 * float(ref.abs().max())


@pytest.mark.parametrize("vblock", [False, True])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,Nk", [(64, 1), (64, 66), (64, 128), (64, 129), (64, 257), (64, 383), (64, 384), (64, 768), (64, 769), (64, 1023), (64, 1024), (64, 1025), (64, 1152), (64, 1153), (64, 1280), (64, 1281), (64, 2047), (64, 2048),
                                  (128, 1), (128, 66), (128, 128), (128, 129), (128, 384), (128, 385), (128, 700)])
def test_few_queries_of_more_heads_than_cus(d, Nk, causal, vblock):
    # More than 256 groups of 32 queries: up to 32 queries per head the packed kernel (d = 64) or the fused one (d = 128) takes short
    # key sequences, the twelve-wavefront kernel the rest; d = 64 and 33 to 64 queries the packed kernel between 128 and 383 keys, the two-group one beyond.
    # One to 256 groups and at most 128 keys: the packed kernel.  All against the rows of a call with more than 64 queries and more
    # than 512 groups, which is the fused kernel's.
    import paper_2409_16997_amd as ifa
    Bc = ifa.block_cols(d, causal)
    N = max(Nk, 129) if not causal else Nk                       # queries of that call (more than keys only without the mask)
    heads = 530 if Nk <= 128 or Nk in (1024, 1025) else 1030 if Nk in (1152, 1153) else 300
    q8, k8, v8, sq, sk = problem(heads, max(N, Nk), d, Nk)
    k8, v8, sk = (t[:, :, :Nk].contiguous() for t in (k8, v8, sk))
    g = torch.Generator(device="cuda").manual_seed(Nk)
    sv = 0.005 + 0.02 * torch.rand((1, heads) + ((-(-Nk // Bc),) if vblock else ()), generator=g, device="cuda")
    call = lambda q, a, n: ifa.int_flash_attn_fwd(q[:, :n].contiguous(), k8[:, :n], v8[:, :n], a[:, :n].contiguous(), sk[:, :n], sv[:, :n],
                                                  causal=causal, out_dtype=torch.float32)
    assert route(heads, N, Nk, d, causal) == ("packed" if d == 64 and N <= 64 else "fused")
    full, reached = call(q8, sq, heads), set()
    for n, nq in ((heads, 1), (heads, 8), (heads, 32), (257, 32), (257, 31), (256, 32), (256, 33), (140, 64), (140, 40), (7, 1), (3, 33), (2, 128)):
        if nq > N:
            continue
        reached.add((nq > 32, route(n, nq, Nk, d, causal)))
        out, ref = call(q8[:, :, N - nq:], sq[:, :, N - nq:], n), full[:, :n, N - nq:]
        if vblock and causal:                                    # as above
            assert bool(((out - ref).abs() <= 2.0 ** -21 * ref.abs()).all()), (n, nq)
        else:
            assert torch.equal(out, ref), (n, nq)
    if d == 64 and Nk > 128:
        assert (True, "packed" if Nk < 384 else "pair") in reached and (False, "packed" if Nk <= 768 or Nk == 1152 else "few") in reached
    h = lambda t, n=1: t[0, :n].cpu().numpy()
    res = oracle.compare_up_to_ties(h(full)[0], h(q8), h(k8), h(v8), h(sq), h(sk), h(sv), causal, Bc)
    assert float(res["err"].max()) <= 1e-3 * float(res["scale"])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,Nk", [(64, 64), (64, 65), (128, 256), (128, 257)])
def test_few_queries_of_more_heads_than_cus_half_int8(d, Nk, causal):
    import paper_2409_16997_amd as ifa
    heads = 300
    q8, k8, v8, sq, sk = problem(heads, Nk, d, Nk)
    v = v8.to(torch.float16) / 64
    call = lambda q, a, n: ifa.int_flash_attn_fwd_half(q[:, :n].contiguous(), k8[:, :n], v[:, :n], a[:, :n].contiguous(), sk[:, :n], causal=causal,
                                                       out_dtype=torch.float32)
    full = call(q8, sq, heads)
    for n, nq in ((heads, 1), (heads, 32), (257, 31), (256, 32)):
        assert torch.equal(call(q8[:, :, Nk - nq:], sq[:, :, Nk - nq:], n), full[:, :n, Nk - nq:]), (n, nq)


# One query per head and more than 64 MB of K and V: the copies carry the non-temporal hint (INT8: one workgroup per head; half-INT8: two up
# to 128 heads at d = 128).
@pytest.mark.parametrize("variant,heads,Nk,d", [("full", 65, 4200, 128), ("full", 136, 2050, 128), ("full", 140, 4100, 64),
                                                ("half", 100, 2100, 128), ("half", 130, 1500, 128), ("half", 120, 3100, 64), ("half", 300, 1300, 64)])
def test_long_caches_are_read_past_the_caches(variant, heads, Nk, d):
    import paper_2409_16997_amd as ifa
    half = variant == "half"
    assert heads * Nk * d * (3 if half else 2) > 64 << 20 and route(heads, 1, Nk, d, True, half) == "few"
    q8, k8, v8, sq, sk = problem(heads, Nk, d, heads)
    q8, sq = q8[:, :, 1:2].contiguous(), sq[:, :, 1:2].contiguous()
    sv = 0.005 + 0.02 * torch.rand((1, heads), device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    pick = [0, heads // 2, heads - 1]
    n = lambda t: t[0, pick].cpu().numpy()
    if half:
        v = v8.to(torch.float16) / 64
        O = ifa.int_flash_attn_fwd_half(q8, k8, v, sq, sk, causal=True, out_dtype=torch.float32)
        ref = oracle.int_flash_attn_fwd_half(n(q8), n(k8), n(v), n(sq), n(sk), True, ifa.block_cols_half(d, True))["O"].reshape(-1, d)
        assert np.abs(n(O).reshape(-1, d) - ref).max() <= 1e-3 * np.abs(ref).max()
        few = ifa.int_flash_attn_fwd_half(*[t[:, :8].contiguous() for t in (q8, k8, v, sq, sk)], causal=True, out_dtype=torch.float32)
    else:
        O = ifa.int_flash_attn_fwd(q8, k8, v8, sq, sk, sv, causal=True, out_dtype=torch.float32)
        res = oracle.compare_up_to_ties(n(O).reshape(-1, d), n(q8), n(k8), n(v8), n(sq), n(sk), n(sv), True, ifa.block_cols(d, True))
        assert float(res["err"].max()) <= 1e-3 * float(res["scale"])
        few = ifa.int_flash_attn_fwd(*[t[:, :8].contiguous() for t in (q8, k8, v8, sq, sk, sv)], causal=True, out_dtype=torch.float32)
    assert torch.equal(few, O[:, :8])                            # without the hint: the same bits

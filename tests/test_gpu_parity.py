"""GPU parity: the HIP path through the C ABI against the CPU oracle, element by element, on the same
seeded inputs.  Bit-exact for the quantizers and the int32 GEMM accumulators; for O the bar is
max|O_gpu - O_oracle| <= 1e-3 * max|O_oracle| on EVERY row, where O_oracle is the oracle's output for a valid
resolution of line 11's rounding: P entries whose fp32 argument lies within evaluation noise of a half-integer may
round either way (the hardware exp2 against the oracle's correctly rounded exp is enough to decide them
differently), and ONE such entry moves a row of O by up to |V_j - O_i| s_V / l -- percents of max|O| for a sharp
row.  A row that misses the oracle's default resolution must therefore match the oracle re-run with some of its
flagged entries rounded the other way (oracle.compare_up_to_ties); rows without flagged entries have no such way
out.  The number of rows that needed it is printed."""
import math

import numpy as np
import pytest

import oracle
import workloads
from helpers import copies_for_the_fused_kernel, first_copy, many, quantized_inputs, random_int8_problem, route, unsplit

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-3
# Window, in units of the exponent argument, inside which a different but equally valid fp32 evaluation
# order (scales folded with log2 e, fused multiply-add, hardware exp2) may move 127*exp(S - m) across a
# rounding boundary: a few roundings of relative size 2^-24 on |S| and |m|, plus the exp2 unit's error.
TIE_REL = 8 * 2.0 ** -24
TIE_ABS = 2e-6


@pytest.fixture(scope="module")
def ifa():
    import paper_2409_16997_amd as m
    m.lib()                      # raises if the HIP library is not built: there is no fallback
    assert torch.cuda.is_available()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def bf16_round(x):               # fp32 -> bf16 (round half to even) -> fp32, on the host
    u = np.ascontiguousarray(x, np.float32).view(np.uint32).astype(np.uint64)
    u = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16
    return u.astype(np.uint32).view(np.float32)


# ------------------------------------------------------------------ quantizers: bit-exact

@pytest.mark.parametrize("dtype", ["float32", "float16", "bfloat16"])
@pytest.mark.parametrize("rows,d", [(1, 64), (37, 128), (128, 64), (4099, 128), (1000, 32), (513, 256), (70, 512)])
def test_quantize_tokenwise_bit_exact(ifa, dtype, rows, d):
    rng = np.random.default_rng(rows * 1000 + d)
    x = (rng.standard_t(3, (rows, d)) * rng.uniform(1e-3, 30, (rows, 1))).astype(np.float32)
    x[rows // 2] = 0.0                                        # an all-zero token
    if rows > 3:
        x[1] = np.round(x[1])                                 # exact ties after scaling are likely here
        x[2, :] = 0.0; x[2, 5] = -1.0                         # single non-zero
    xt = torch.from_numpy(x).to(getattr(torch, dtype)).cuda()
    xq, s = ifa.quantize_tokenwise(xt)
    ref_q, ref_s = oracle.quantize_tokenwise(xt.float().cpu().numpy())    # widening is exact
    assert np.array_equal(xq.cpu().numpy(), ref_q)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), ref_s.view(np.uint32))


@pytest.mark.parametrize("dtype", ["float32", "float16"])
@pytest.mark.parametrize("global_scale", [False, True])
def test_quantize_headwise_bit_exact(ifa, dtype, global_scale):
    rng = np.random.default_rng(7)
    x = rng.standard_normal((2, 3, 384, 64)).astype(np.float32) * rng.uniform(0.1, 5, (2, 3, 1, 1)).astype(np.float32)
    x[1, 1] = 0.0                                             # an all-zero head
    xt = torch.from_numpy(x).to(getattr(torch, dtype)).cuda()
    xq, s = ifa.quantize_headwise(xt, global_scale=global_scale)
    ref_q, ref_s = oracle.quantize_headwise(xt.float().cpu().numpy().reshape(6, 384, 64), global_scale=global_scale)
    assert np.array_equal(xq.cpu().numpy().reshape(6, 384, 64), ref_q)
    assert np.array_equal(s.cpu().numpy().reshape(6).view(np.uint32), ref_s.view(np.uint32))


def test_quantize_tokenwise_scale_mul(ifa):
    # scale_mul multiplies the stored scale once in fp32 and leaves the codes alone
    rng = np.random.default_rng(8)
    x = rng.standard_normal((300, 128)).astype(np.float16)
    c = 1.0 / math.sqrt(128)
    q, s = ifa.quantize_tokenwise(dev(x), scale_mul=c)
    rq, rs = oracle.quantize_tokenwise(x)
    assert np.array_equal(q.cpu().numpy(), rq)
    assert np.array_equal(s.cpu().numpy(), (rs * np.float32(c)).astype(np.float32))


@pytest.mark.parametrize("dtype", ["float32", "float16", "bfloat16"])
@pytest.mark.parametrize("rows,d", [(5, 32), (131, 64), (1000, 128), (77, 256), (40, 512)])
def test_quantize_tokenwise_hadamard_bit_exact(ifa, dtype, rows, d):
    rng = np.random.default_rng(rows + d)
    x = rng.standard_normal((rows, d)).astype(np.float32)
    x[:, rng.choice(d, 3, replace=False)] *= 25.0             # outlier channels, the case the rotation is for
    x[rows // 2] = 0.0
    xt = torch.from_numpy(x).to(getattr(torch, dtype)).cuda()
    c = d ** -0.5
    q, s = ifa.quantize_tokenwise(xt, scale_mul=c, hadamard=True)
    rq, rs = oracle.quantize_tokenwise_hadamard(xt.float().cpu().numpy(), c)
    assert np.array_equal(q.cpu().numpy(), rq)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), rs.view(np.uint32))


def test_hadamard_rotated_attention_on_outlier_channels(ifa):
    # rotate Q and K before quantizing, feed the unchanged attention kernel; parity against the oracle on the
    # rotated inputs, and accuracy against fp64 attention of the original activations
    w = workloads.custom("t", 1, 4, 1024, 128, False, dist="uniform_outlier", seed=5)
    Q, K, V = (workloads.tensor(w, t) for t in "QKV")
    sh = (1, 4, 1024, 128)
    d = w.d
    ref = oracle.attention_fp64(Q, K, V, causal=False, scale=d ** -0.5)
    Vq, sV = oracle.quantize_headwise(V)
    res = {}
    for rot in (False, True):
        if rot:
            Qq, sQ = oracle.quantize_tokenwise_hadamard(Q, (d ** -0.5) * (d ** -0.5))   # rotation and softmax scale
            Kq, sK = oracle.quantize_tokenwise_hadamard(K, d ** -0.5)
        else:
            Qq, sQ = oracle.quantize_tokenwise(Q); sQ = (sQ * np.float32(d ** -0.5)).astype(np.float32)
            Kq, sK = oracle.quantize_tokenwise(K)
        O = ifa.int_flash_attn_fwd(dev(Qq.reshape(sh)), dev(Kq.reshape(sh)), dev(Vq.reshape(sh)), dev(sQ.reshape(1, 4, -1)),
                                   dev(sK.reshape(1, 4, -1)), dev(sV.reshape(1, 4)), causal=False, out_dtype=torch.float32)
        torch.cuda.synchronize()
        O = O.cpu().numpy().reshape(-1, d)
        check_against_oracle(ifa, O, Qq, Kq, Vq, sQ, sK, sV, False, label=f"outlier channels, hadamard={rot}")
        res[rot] = np.abs(O - ref).sum() / np.abs(ref).sum()
    print(f"[MRE outlier channels N=1024] plain {res[False]:.4%}   Hadamard-rotated Q,K {res[True]:.4%}", flush=True)
    assert res[True] < res[False]


def test_quantize_workload_heads_bit_exact(ifa):
    for name in ("c1", "c2", "c4", "c5"):
        w = workloads.WORKLOADS[name]
        heads = [0, w.heads - 1] if w.heads > 1 else [0]
        for t in ("Q", "V"):
            x = workloads.tensor(w, t, heads)
            xt = dev(x)
            q, s = ifa.quantize_tokenwise(xt)
            rq, rs = oracle.quantize_tokenwise(x)
            assert np.array_equal(q.cpu().numpy(), rq) and np.array_equal(s.cpu().numpy(), rs)
            q, s = ifa.quantize_headwise(xt)
            rq, rs = oracle.quantize_headwise(x)
            assert np.array_equal(q.cpu().numpy(), rq) and np.array_equal(s.cpu().numpy(), rs)


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,H,N,d", [(2, 3, 384, 64), (1, 5, 200, 128), (1, 2, 37, 32), (4, 10, 37, 64), (2, 16, 8, 64), (1, 33, 1000, 128), (8, 8, 5, 128)])
def test_quantize_qkv_equals_the_three_separate_calls(ifa, dtype, B, H, N, d):
    # the fused preparation against the separate entry points, bit for bit, twice in a row into the same buffers (the
    # second call must not see what the first one left in the codes).  V goes whole heads in the launch of Q and K, or in parts that leave
    # their maxima in V's codes for a second launch (40 heads of 37 x 64 whole, 33 of 1000 x 128 in parts).
    g = torch.Generator(device="cuda").manual_seed(B * 1000 + N + d)
    Q, K, V = (torch.randn((B, H, N, d), generator=g, device="cuda", dtype=torch.float32).to(dtype) for _ in range(3))
    V[0, 0] = 0                                            # an all-zero head: scale 1, codes 0
    fold = 1.0 / math.sqrt(d)
    rq, rsq = ifa.quantize_tokenwise(Q, scale_mul=fold)
    rk, rsk = ifa.quantize_tokenwise(K)
    rv, rsv = ifa.quantize_headwise(V)
    out = ifa.quantize_qkv(Q, K, V, s_Q_mul=fold)
    for _ in range(2):
        got = ifa.quantize_qkv(Q, K, V * 0.5 if _ == 0 else V, s_Q_mul=fold, out=out)   # first pass leaves other absmax values behind
    torch.cuda.synchronize()
    for a, b in zip(got, (rq, rk, rv, rsq, rsk, rsv)):
        assert torch.equal(a, b)
    assert float(rsv[0, 0]) == 1.0 and not bool(rv[0, 0].any())


@pytest.mark.parametrize("hadamard", [False, True])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("shape", [(2, 3, 77, 64), (4, 8, 500, 128), (1, 1, 1, 32)])
def test_quantize_qk_equals_the_two_separate_calls(ifa, shape, dtype, hadamard):
    # Q and K in one launch against the single-tensor entry points (themselves bit-exact against the oracle above),
    # bit for bit, with and without the Hadamard rotation; the second call writes into the first call's buffers
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    Q, K = (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dtype) for _ in range(2))
    K[0, 0, 0] = 0                                         # an all-zero row: scale 1, codes 0
    fold = 1.0 / math.sqrt(shape[-1])
    rq, rsq = ifa.quantize_tokenwise(Q, scale_mul=fold, hadamard=hadamard)
    rk, rsk = ifa.quantize_tokenwise(K, hadamard=hadamard)
    out = ifa.quantize_qk(Q * 0.25, K * 2.0, s_Q_mul=1.0, hadamard=hadamard)
    got = ifa.quantize_qk(Q, K, s_Q_mul=fold, hadamard=hadamard, out=out)
    torch.cuda.synchronize()
    for a, b in zip(got, (rq, rk, rsq, rsk)):
        assert torch.equal(a, b)


# ------------------------------------------------------------------ int32 accumulators: bit-exact

def _oracle_block_pv(P, V, Bc):
    """P_j V_j per key block with the oracle's integer GEMM: [N / Bc, N, d] int32."""
    N = P.shape[0]
    out = []
    for j in range(N // Bc):
        Pj = np.zeros_like(P)
        Pj[:, j * Bc:(j + 1) * Bc] = P[:, j * Bc:(j + 1) * Bc]
        out.append(oracle.pv_i32(Pj, V))
    return np.stack(out)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N,d", [(128, 64), (128, 128), (384, 128), (256, 64), (640, 128)])
def test_int32_accumulators_of_the_production_kernel_bit_exact(ifa, N, d, causal):
    # The fused kernel itself (its test instantiation stores what sits in its accumulators): the int32 result of
    # line 9, the packed P of line 11 and the int32 result of line 13 per key block, against the oracle's integer
    # GEMMs -- bit for bit.  P is compared with the oracle's own P outside the entries it flags as near-ties.
    rng = np.random.default_rng(N + d + causal)
    Q = rng.integers(-127, 128, (N, d), dtype=np.int8)
    K = rng.integers(-127, 128, (N, d), dtype=np.int8)
    V = rng.integers(-127, 128, (N, d), dtype=np.int8)
    Q[0] = 127; K[1] = 127; K[2] = -128; Q[3] = -128; V[:, 7] = -128       # extremes of the accumulator range of line 9
    base = 1.0 / (73.3 * 73.3 * math.sqrt(d))
    sQ = (rng.uniform(0.5, 1.5, N) * math.sqrt(base)).astype(np.float32)
    sK = (rng.uniform(0.5, 1.5, N) * math.sqrt(base)).astype(np.float32)
    sV = np.array([0.01], np.float32)
    Bc = ifa.block_cols(d, causal)
    out = ifa.debug_fwd(dev(Q), dev(K), dev(V), dev(sQ), dev(sK), dev(sV), causal=causal, fill=-1)
    torch.cuda.synchronize()
    S, P, PV, O = (out[k].cpu().numpy() for k in ("S", "P", "PV", "O"))
    ref = oracle.int_flash_attn_fwd(Q[None], K[None], V[None], sQ[None], sK[None], sV, causal, Bc, tie_rel=TIE_REL, tie_abs=TIE_ABS,
                                    want_P=True)
    S_ref = oracle.qk_i32(Q, K)
    seen = np.ones((N, N), bool) if not causal else np.tril(np.ones((N, N), bool))   # keys a query sees
    assert np.array_equal(S[seen], S_ref[seen])                                        # line 9, exact
    # P: every visible entry was written (0..127), masked entries of visited tiles are 0, and it is the oracle's P
    # except where the oracle itself says the rounding is within fp32 noise of a tie (then off by at most one)
    assert P[seen].min() >= 0
    P_ref = ref["P"]
    diff = np.abs(P[seen].astype(np.int32) - P_ref[seen].astype(np.int32))
    assert diff.max() <= 1
    rows_with_diff = np.unique(np.nonzero((np.abs(P.astype(np.int32) - P_ref.astype(np.int32)) * seen) > 0)[0])
    assert np.all(ref["n_tie"][rows_with_diff] > 0), "P differs from the oracle in a row without a flagged near-tie"
    # line 13, exact: the kernel's P_j V_j against the oracle's integer GEMM on the kernel's own P
    Pk = np.where(seen & (P >= 0), P, 0).astype(np.int8)
    PV_ref = _oracle_block_pv(Pk, V, Bc)
    for j in range(N // Bc):
        rows = np.arange(N) if not causal else np.arange(j * Bc, N)                     # query blocks that visit block j
        assert np.array_equal(PV[j][rows], PV_ref[j][rows]), f"P V of key block {j}"
    # and the output of the same launch is the production output, the fused kernel's and that of the kernel that takes one head
    for copies in (1, copies_for_the_fused_kernel(1, N, N, d, causal)):
        O_prod = run_gpu(ifa, *many(copies, Q[None], K[None], V[None], sQ[None], sK[None], sV), 1, copies, causal)
        assert np.array_equal(O, first_copy(O_prod, copies).reshape(N, d)), copies


@pytest.mark.parametrize("d", [64, 128])
def test_second_gemm_accumulator_extremes_with_injected_p(ifa, d):
    # P = 127 everywhere against V = -127 / +127 columns drives |P_j V_j| to 127 * 127 * 128, the end of the range
    # the accumulator's starting constant leaves room for; random P in between.  P is injected in place of the
    # computed one, everything else is the production path.
    N = 256
    rng = np.random.default_rng(d)
    Q = rng.integers(-127, 128, (N, d), dtype=np.int8)
    K = rng.integers(-127, 128, (N, d), dtype=np.int8)
    V = rng.integers(-127, 128, (N, d), dtype=np.int8)
    P_in = rng.integers(0, 128, (N, N), dtype=np.int8)
    P_in[5] = 127; P_in[6] = 127; V[:, 7] = -127; V[:, 9] = 127; P_in[200] = 0
    ones = np.ones(N, np.float32)
    out = ifa.debug_fwd(dev(Q), dev(K), dev(V), dev(ones * 1e-4), dev(ones), dev(np.array([1.0], np.float32)), causal=False, P_in=dev(P_in))
    torch.cuda.synchronize()
    Bc = ifa.block_cols(d, False)
    PV = out["PV"].cpu().numpy()
    assert np.array_equal(out["P"].cpu().numpy(), P_in)
    assert np.array_equal(PV, _oracle_block_pv(P_in, V, Bc))
    assert PV.min() == -127 * 127 * Bc and PV.max() == 127 * 127 * Bc
    assert np.array_equal(out["S"].cpu().numpy(), oracle.qk_i32(Q, K))


# ------------------------------------------------------------------ Algorithm 1 end to end

def run_gpu(ifa, Qq, Kq, Vq, sQ, sK, sV, B, H, causal, out_dtype=None):
    heads, N, d = Qq.shape
    assert heads == B * H
    sh = (B, H, N, d)
    O = ifa.int_flash_attn_fwd(dev(Qq.reshape(sh)), dev(Kq.reshape(sh)), dev(Vq.reshape(sh)),
                               dev(sQ.reshape(B, H, N)), dev(sK.reshape(B, H, N)), dev(sV.reshape(B, H)),
                               causal=causal, out_dtype=out_dtype or torch.float32)
    torch.cuda.synchronize()
    return O


def check_against_oracle(ifa, O_gpu_rows, Qq, Kq, Vq, sQ, sK, sV, causal, row_idx=None, label="", quiet=False):
    """Asserts |O_gpu - O_oracle| <= 1e-3 max|O_oracle| on every row, O_oracle being Algorithm 1 with a valid
    resolution of its near-tie roundings (see the module docstring)."""
    d = Qq.shape[-1]
    Bc = ifa.block_cols(d, causal)
    assert np.all(np.isfinite(O_gpu_rows))
    res = oracle.compare_up_to_ties(O_gpu_rows, Qq, Kq, Vq, sQ, sK, sV, causal, Bc, row_idx=row_idx,
                                    tie_rel=TIE_REL, tie_abs=TIE_ABS, tol=TOL)
    err, scale, clean = res["err"], res["scale"], res["n_tie"] == 0
    worst_clean = (err[clean].max() / scale) if clean.any() else 0.0
    resolved = int((res["flips"] > 0).sum())
    if not quiet:
        print(f"[parity {label}] rows={len(err)} max|dO|/max|O|={err.max() / scale:.3e} "
              f"(rows without near-ties: {worst_clean:.3e}; rows with near-ties: {int((~clean).sum())}, of which "
              f"{resolved} match the oracle with flagged entries rounded the other way, "
              f"worst before that {res['err_default'].max() / scale:.3e})", flush=True)
    assert np.all(err <= TOL * scale), (err.max() / scale, int((err > TOL * scale).sum()), int((~clean).sum()))
    return err.max() / scale, worst_clean, resolved, len(err)


@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("name", ["c1", "c2"])
def test_small_workloads_every_element(ifa, name, scaled):
    w = workloads.WORKLOADS[name]
    x = quantized_inputs(w, scaled=scaled)
    O = run_gpu(ifa, x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], w.B, w.H, w.causal).cpu().numpy()
    check_against_oracle(ifa, O.reshape(-1, w.d), x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], w.causal,
                         label=f"{name} scaled={scaled}")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,H,N,d", [(1, 1, 128, 128), (1, 3, 256, 64), (2, 4, 384, 128), (1, 5, 640, 128), (1, 8, 512, 64)])
@pytest.mark.parametrize("dist", ["normal", "uniform_outlier", "student_t3"])
@pytest.mark.parametrize("fused", [False, True])
def test_shapes_masks_distributions(ifa, B, H, N, d, causal, dist, fused):
    # several key blocks, head counts that are and are not multiples of the XCD count, both head dims; `fused`: with as many copies
    # of the heads as the fused kernel wants
    w = workloads.custom("t", B, H, N, d, causal, dist=dist, seed=B * 1000 + N + d)
    x = quantized_inputs(w, scaled=True)
    copies = copies_for_the_fused_kernel(B * H, N, N, d, causal) if fused else 1
    O = first_copy(run_gpu(ifa, *many(copies, x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"]), copies * B, H, causal), copies)
    check_against_oracle(ifa, O.reshape(-1, d), x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], causal,
                         label=f"{B}x{H}x{N}x{d} causal={causal} {dist}")


@pytest.mark.parametrize("B,H", [(5, 8), (3, 8), (9, 8), (1, 7), (3, 3), (1, 16), (13, 5), (1, 71)])   # from 65 heads on the fused kernel
def test_head_counts_and_grid_shapes(ifa, B, H):
    # head counts that fill the XCD groups exactly, leave a short last group (padding workgroups), or are not a
    # multiple of 8 at all; every head must come out, each exactly once
    N, d = 256, 64
    w = workloads.custom("t", B, H, N, d, True, dist="normal", seed=31 * B + H)
    x = quantized_inputs(w, scaled=True)
    O = run_gpu(ifa, x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], B, H, True).cpu().numpy()
    check_against_oracle(ifa, O.reshape(-1, d), x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], True,
                         label=f"heads {B}x{H}")


@pytest.mark.parametrize("B,H,N,d,causal", [(3, 40, 1500, 128, True),      # masked, 12 query blocks: 8 heads per XCD group, last group short
                                             (2, 32, 2048, 64, True),       # 8 heads per group, d = 64
                                             (1, 24, 16384, 128, False),    # unmasked, 4 MB of K + V per head: 1 head per group
                                             (1, 24, 8192, 128, False)])    # 2 heads per group, 3 heads per XCD
def test_head_group_sizes_sampled_rows(ifa, B, H, N, d, causal):
    # every size of the per-XCD head group the launcher picks; every head must come out, each exactly once:
    # first, last and seeded rows of every head against the oracle
    w = workloads.custom("t", B, H, N, d, causal, dist="normal", seed=N + H)
    x = quantized_inputs(w, scaled=True)
    heads = B * H
    rows = np.unique(np.concatenate([np.arange(0, 3), np.arange(N - 3, N), np.random.default_rng(H).integers(0, N, 10)]))
    idx = np.concatenate([h * N + rows for h in range(heads)]).astype(np.int64)
    O = run_gpu(ifa, x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], B, H, causal).cpu().numpy().reshape(-1, d)
    check_against_oracle(ifa, O[idx], x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], causal, row_idx=idx,
                         label=f"head groups {B}x{H}x{N}x{d} causal={causal}")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N,d", [(1, 128), (37, 64), (127, 128), (129, 128), (200, 64), (333, 128), (1000, 128), (515, 64)])
@pytest.mark.parametrize("fused", [False, True])
def test_ragged_sequence_lengths(ifa, N, d, causal, fused):
    # N not a multiple of the 128-key block: keys >= N are masked in the last block, rows >= N are not stored
    copies = copies_for_the_fused_kernel(3, N, N, d, causal) if fused else 1
    if copies is None:
        return                                               # at most 64 queries at d = 64: never the fused kernel's
    w = workloads.custom("t", 1, 3, N, d, causal, dist="normal", seed=N + d)
    x = quantized_inputs(w, scaled=True)
    heads = 3 * copies
    sh = (1, heads, N, d)
    guard = 64                                               # canary rows after O: must stay untouched
    Obuf = torch.full((heads * N + guard, d), 12345.0, dtype=torch.float32, device="cuda")
    O = Obuf[:heads * N].view(sh)
    Qq, Kq, Vq, sQ, sK, sV = many(copies, x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"])
    ifa.int_flash_attn_fwd(dev(Qq.reshape(sh)), dev(Kq.reshape(sh)), dev(Vq.reshape(sh)), dev(sQ.reshape(1, heads, N)),
                           dev(sK.reshape(1, heads, N)), dev(sV.reshape(1, heads)), causal=causal, out=O)
    torch.cuda.synchronize()
    assert bool((Obuf[heads * N:] == 12345.0).all())
    check_against_oracle(ifa, first_copy(O, copies).reshape(-1, d), x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], causal,
                         label=f"ragged N={N} d={d} causal={causal} fused={fused}")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Nq,Nk,d", [(1, 1000, 128), (1, 128, 64), (128, 512, 128), (100, 333, 128), (256, 1024, 64),
                                     (37, 37, 128), (130, 131, 128), (64, 4096, 128), (300, 200, 128), (513, 640, 64)])
@pytest.mark.parametrize("fused", [False, True])
def test_rectangular_problems(ifa, Nq, Nk, d, causal, fused):
    # Nq query rows against Nk keys: a chunk of queries against a longer sequence, or one query.  Under the mask
    # the queries are the last Nq positions (query i sees keys <= i + Nk - Nq), so the diagonal crosses key blocks
    # at any offset; Nk < Nq is allowed without the mask only.
    if causal and Nk < Nq:
        p = lambda t: ctypes_ptr(t)
        z8 = torch.zeros((1, 1, max(Nq, Nk), d), dtype=torch.int8, device="cuda")
        zf = torch.ones((1, 1, max(Nq, Nk)), dtype=torch.float32, device="cuda")
        O = torch.empty((1, 1, Nq, d), dtype=torch.float16, device="cuda")
        rc = ifa.lib().int_flash_attn_fwd_rect(p(z8), p(z8), p(z8), p(zf), p(zf), p(zf), 1, 1, Nq, Nk, d, 1, p(O), 1, None)
        assert rc == -4
        return
    copies = copies_for_the_fused_kernel(3, Nq, Nk, d, causal) if fused else 1
    if copies is None:
        return                                               # up to 32 queries: the fused kernel has short keys at d = 128 only
    H = 3 * copies
    rng = np.random.default_rng(Nq * 7 + Nk + d)
    Qq, Kq, Vq, sQ, sK, sV = random_int8_problem(rng, 3, max(Nq, Nk), d, score_sigma=2.0)
    Qq, sQ = np.ascontiguousarray(Qq[:, :Nq]), np.ascontiguousarray(sQ[:, :Nq])
    Kq, Vq, sK = np.ascontiguousarray(Kq[:, :Nk]), np.ascontiguousarray(Vq[:, :Nk]), np.ascontiguousarray(sK[:, :Nk])
    guard = 64
    Obuf = torch.full((H * Nq + guard, d), 12345.0, dtype=torch.float32, device="cuda")
    O = Obuf[:H * Nq].view(1, H, Nq, d)
    ifa.int_flash_attn_fwd(*[dev(t[None]) for t in many(copies, Qq, Kq, Vq, sQ, sK, sV)], causal=causal, out=O)
    torch.cuda.synchronize()
    assert bool((Obuf[H * Nq:] == 12345.0).all())
    check_against_oracle(ifa, first_copy(O, copies).reshape(-1, d), Qq, Kq, Vq, sQ, sK, sV, causal,
                         label=f"rect Nq={Nq} Nk={Nk} d={d} causal={causal} fused={fused}")


@pytest.mark.parametrize("dtype", ["float16", "bfloat16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N,d", [(1, 128), (33, 64), (127, 128), (129, 64), (200, 128), (515, 128)])
@pytest.mark.parametrize("fused", [False, True])
def test_ragged_lengths_with_two_byte_outputs(ifa, N, d, causal, dtype, fused):
    # 2-byte outputs (the fused kernel's leave through its staged row-wise store): rows past N must not be written (canaries on
    # both sides of O) and the values must be the fp32 result rounded once
    copies = copies_for_the_fused_kernel(3, N, N, d, causal) if fused else 1
    heads = 3 * copies
    w = workloads.custom("t", 1, 3, N, d, causal, dist="normal", seed=17 * N + d)
    x = dict(zip(("Qq", "Kq", "Vq", "sQ", "sK", "sV"), many(copies, *[quantized_inputs(w, scaled=True)[k] for k in ("Qq", "Kq", "Vq", "sQ", "sK", "sV")])))
    sh = (1, heads, N, d)
    tdt = getattr(torch, dtype)
    guard = 256
    Obuf = torch.full((guard + heads * N + guard, d), 77.0, dtype=tdt, device="cuda")
    O = Obuf[guard:guard + heads * N].view(sh)
    args = (dev(x["Qq"].reshape(sh)), dev(x["Kq"].reshape(sh)), dev(x["Vq"].reshape(sh)), dev(x["sQ"].reshape(1, heads, N)),
            dev(x["sK"].reshape(1, heads, N)), dev(x["sV"].reshape(1, heads)))
    ifa.int_flash_attn_fwd(*args, causal=causal, out=O)
    O32 = ifa.int_flash_attn_fwd(*args, causal=causal, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert bool((Obuf[:guard] == 77.0).all()) and bool((Obuf[guard + heads * N:] == 77.0).all())
    assert torch.equal(O, O32.to(tdt))


def _random_shapes(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        d = int(rng.choice([64, 128]))
        H = int(rng.integers(1, 10))
        Nk = int(rng.integers(1, 700))
        causal = bool(rng.integers(0, 2))
        Nq = int(rng.integers(1, Nk + 1)) if causal else int(rng.integers(1, 700))
        out.append((H, Nq, Nk, d, causal))
    return out


@pytest.mark.parametrize("H,Nq,Nk,d,causal", _random_shapes(24, 2024))
def test_seeded_random_shapes(ifa, H, Nq, Nk, d, causal):
    # a fixed, seeded sample of odd shapes: any head count, any Nq, Nk (ragged in both), both head dims, both masks; as it is, and with
    # as many copies of the heads as the fused kernel wants
    rng = np.random.default_rng(H * 1000003 + Nq * 1009 + Nk)
    Qq, Kq, Vq, sQ, sK, sV = random_int8_problem(rng, H, max(Nq, Nk), d, score_sigma=float(rng.uniform(0.5, 6.0)))
    Qq, sQ = np.ascontiguousarray(Qq[:, :Nq]), np.ascontiguousarray(sQ[:, :Nq])
    Kq, Vq, sK = np.ascontiguousarray(Kq[:, :Nk]), np.ascontiguousarray(Vq[:, :Nk]), np.ascontiguousarray(sK[:, :Nk])
    for copies in (1, copies_for_the_fused_kernel(H, Nq, Nk, d, causal)):
        if copies is None:
            continue
        O = ifa.int_flash_attn_fwd(*[dev(t[None]) for t in many(copies, Qq, Kq, Vq, sQ, sK, sV)], causal=causal, out_dtype=torch.float32)
        torch.cuda.synchronize()
        check_against_oracle(ifa, first_copy(O, copies).reshape(-1, d), Qq, Kq, Vq, sQ, sK, sV, causal,
                             label=f"random H={H} Nq={Nq} Nk={Nk} d={d} causal={causal} copies={copies}")


def ctypes_ptr(t):
    import ctypes
    return ctypes.c_void_p(t.data_ptr())


def test_rectangular_rows_equal_the_square_kernel_rows(ifa):
    # the last Nq rows of the square causal problem, computed as a rectangular call: same bits.  A few heads (the few-query kernel on
    # the rectangular side) and more (the fused kernel on both)
    for H, kernel in ((18, "few"), (80, "fused")):
        N, Nq, d = 1024, 200, 128
        assert all(route(H, N, N, d, c) == "fused" and route(H, Nq, N, d, c) == kernel for c in (False, True))
        _rectangular_rows(ifa, H, N, Nq, d)


def _rectangular_rows(ifa, H, N, Nq, d):
    rng = np.random.default_rng(77)
    Qq, Kq, Vq, sQ, sK, sV = random_int8_problem(rng, H, N, d, score_sigma=2.0)
    args = lambda q, sq: (dev(q[None]), dev(Kq[None]), dev(Vq[None]), dev(sq[None]), dev(sK[None]), dev(sV[None]))
    for causal in (False, True):
        full = ifa.int_flash_attn_fwd(*args(Qq, sQ), causal=causal, out_dtype=torch.float32)
        rect = ifa.int_flash_attn_fwd(*args(np.ascontiguousarray(Qq[:, N - Nq:]), np.ascontiguousarray(sQ[:, N - Nq:])),
                                      causal=causal, out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert torch.equal(rect, full[:, :, N - Nq:])


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq", [1, 7, 32, 33, 64])
def test_few_query_calls_equal_the_square_kernel_rows(ifa, Nq, d, out_dtype):
    # A call with a few queries per head (a decode step, a short chunk) runs a kernel of its own that splits every key
    # block over the wavefronts of a workgroup; it performs the arithmetic of the square kernel on the same operands, so
    # its rows are the last Nq rows of the square problem bit for bit, with and without the mask, on a ragged length.
    N = 1231
    for H in (15, 30):
        assert all(route(H, N, N, d, c) in ("fused", "pair") and route(H, Nq, N, d, c) == "few" for c in (False, True))
        rng = np.random.default_rng(Nq * 131 + d)
        Qq, Kq, Vq, sQ, sK, sV = random_int8_problem(rng, H, N, d, score_sigma=2.0)
        args = lambda q, sq: (dev(q[None]), dev(Kq[None]), dev(Vq[None]), dev(sq[None]), dev(sK[None]), dev(sV[None]))
        for causal in (False, True):
            full = ifa.int_flash_attn_fwd(*args(Qq, sQ), causal=causal, out_dtype=out_dtype)
            few = ifa.int_flash_attn_fwd(*args(np.ascontiguousarray(Qq[:, N - Nq:]), np.ascontiguousarray(sQ[:, N - Nq:])),
                                         causal=causal, out_dtype=out_dtype)
            torch.cuda.synchronize()
            assert torch.equal(few, full[:, :, N - Nq:]), (H, Nq, d, causal)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq", [1, 7, 33, 64])
def test_few_query_calls_with_blockwise_v_scales_equal_the_square_kernel_rows(ifa, Nq, d):
    # the same with one V scale per key block (the running output is carried in units of the current block's scale)
    N = 1231
    for H in (15, 30):
        assert all(route(H, N, N, d, c) in ("fused", "pair") and route(H, Nq, N, d, c) == "few" for c in (False, True))
        rng = np.random.default_rng(Nq * 17 + d)
        Qq, Kq, Vq, sQ, sK, _ = random_int8_problem(rng, H, N, d, score_sigma=2.0)
        sVb = rng.uniform(0.005, 0.05, (H, -(-N // ifa.block_cols(d, True)))).astype(np.float32)
        args = lambda q, sq: (dev(q[None]), dev(Kq[None]), dev(Vq[None]), dev(sq[None]), dev(sK[None]), dev(sVb[None]))
        for causal in (False, True):
            full = ifa.int_flash_attn_fwd(*args(Qq, sQ), causal=causal, out_dtype=torch.float32)
            few = ifa.int_flash_attn_fwd(*args(np.ascontiguousarray(Qq[:, N - Nq:]), np.ascontiguousarray(sQ[:, N - Nq:])),
                                         causal=causal, out_dtype=torch.float32)
            torch.cuda.synchronize()
            assert torch.equal(few, full[:, :, N - Nq:]), (H, Nq, d, causal)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Nq,Nk,d", [(1, 16384, 128), (1, 1, 128), (7, 300, 64), (32, 4097, 128), (64, 127, 64), (50, 2048, 128)])
def test_few_query_calls_against_the_oracle(ifa, Nq, Nk, d, causal):
    # the same calls against Algorithm 1 itself, on several heads (8 heads: the XCD-aware mapping; 3: the plain one),
    # with canary rows behind the output
    if causal and Nk < Nq:
        return
    for H in (8, 3):
        rng = np.random.default_rng(Nq + Nk + d + H)
        Qq, Kq, Vq, sQ, sK, sV = random_int8_problem(rng, H, max(Nq, Nk), d, score_sigma=2.0)
        Qq, sQ = np.ascontiguousarray(Qq[:, :Nq]), np.ascontiguousarray(sQ[:, :Nq])
        Kq, Vq, sK = np.ascontiguousarray(Kq[:, :Nk]), np.ascontiguousarray(Vq[:, :Nk]), np.ascontiguousarray(sK[:, :Nk])
        guard = 64
        Obuf = torch.full((H * Nq + guard, d), 12345.0, dtype=torch.float32, device="cuda")
        O = Obuf[:H * Nq].view(1, H, Nq, d)
        ifa.int_flash_attn_fwd(dev(Qq[None]), dev(Kq[None]), dev(Vq[None]), dev(sQ[None]), dev(sK[None]), dev(sV[None]),
                               causal=causal, out=O)
        torch.cuda.synchronize()
        assert bool((Obuf[H * Nq:] == 12345.0).all())
        check_against_oracle(ifa, O.cpu().numpy().reshape(-1, d), Qq, Kq, Vq, sQ, sK, sV, causal,
                             label=f"few queries Nq={Nq} Nk={Nk} d={d} H={H} causal={causal}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq,Nk,H", [(1, 16384, 8), (1, 1, 3), (1, 129, 1), (3, 1000, 5), (8, 4097, 8), (5, 300, 16), (2, 20000, 2), (8, 8, 4),
                                      (9, 4097, 8), (32, 16384, 2), (20, 1000, 5), (32, 32, 3), (17, 300, 16), (12, 500, 100),
                                      (8, 258, 16), (32, 1026, 4),
                                      # the last run of key blocks is masked entirely for the early queries, where the call splits
                                      (8, 2306, 16), (32, 3074, 4), (3, 5000, 5), (5, 2049, 16), (20, 3001, 5), (17, 2300, 16), (12, 2500, 30), (5, 2305, 8), (17, 2561, 4), (12, 3585, 12), (8, 4610, 16), (5, 4097, 16), (2, 5000, 8)])
def test_key_split_calls_equal_the_sequential_walk(ifa, Nq, Nk, H, d):
    # The key-split path forms P on the grid of the running maximum of the sequential walk (it knows every block's
    # maximum before it forms any P), so it differs from the one-workgroup-per-head kernel only by the order of the
    # fp32 additions of lines 12-13: a few ulp of O, far inside the parity bar (up to 8 queries per head the scores go
    # through the workspace, from 9 to 32 the second pass recomputes them; up to 2048 keys, or with many heads, the call
    # does not split and the workspace stays as it was).  Checked against that kernel (tight)
    # and against the oracle (the strict bar), with canary rows behind the output and a workspace of exactly the size
    # the library asks for, poisoned with NaN (nothing may be read before it is written).
    for causal in (False, True):
        rng = np.random.default_rng(Nq * 7 + Nk + d + H + int(causal))
        Qq, Kq, Vq, sQ, sK, sV = random_int8_problem(rng, H, max(Nq, Nk), d, score_sigma=2.0)
        Qq, sQ = np.ascontiguousarray(Qq[:, :Nq]), np.ascontiguousarray(sQ[:, :Nq])
        Kq, Vq, sK = np.ascontiguousarray(Kq[:, :Nk]), np.ascontiguousarray(Vq[:, :Nk]), np.ascontiguousarray(sK[:, :Nk])
        args = (dev(Qq[None]), dev(Kq[None]), dev(Vq[None]), dev(sQ[None]), dev(sK[None]), dev(sV[None]))
        seq = ifa.int_flash_attn_fwd(*args, causal=causal, out_dtype=torch.float32)
        guard = 64
        Obuf = torch.full((H * Nq + guard, d), 12345.0, dtype=torch.float32, device="cuda")
        O = Obuf[:H * Nq].view(1, H, Nq, d)
        need = ifa.splitk_workspace_bytes(1, H, Nq, Nk, d)
        ws = torch.full((need // 4 + guard,), float("nan"), dtype=torch.float32, device="cuda")
        ifa.int_flash_attn_fwd_splitk(*args, causal=causal, out=O, workspace=ws[:need // 4].view(torch.uint8))
        torch.cuda.synchronize()
        assert bool((Obuf[H * Nq:] == 12345.0).all()) and bool(torch.isnan(ws[need // 4:]).all())
        assert bool(torch.isnan(ws).all()) == unsplit(H, Nq, Nk, d), "split or not"
        scale = float(seq.abs().max())
        diff = float((O - seq).abs().max())
        assert diff <= 4e-6 * scale, (Nq, Nk, H, d, causal, diff, scale)
        check_against_oracle(ifa, O.cpu().numpy().reshape(-1, d), Qq, Kq, Vq, sQ, sK, sV, causal,
                             label=f"key split Nq={Nq} Nk={Nk} d={d} H={H} causal={causal}")


@pytest.mark.parametrize("out_dtype", [torch.float16, torch.bfloat16])
def test_key_split_two_byte_outputs(ifa, out_dtype):
    # the two-byte outputs are the fp32 result rounded to nearest even, as everywhere else in the library
    H, Nq, Nk, d = 8, 4, 3000, 128
    rng = np.random.default_rng(99)
    Qq, Kq, Vq, sQ, sK, sV = random_int8_problem(rng, H, Nk, d, score_sigma=2.0)
    Qq, sQ = np.ascontiguousarray(Qq[:, :Nq]), np.ascontiguousarray(sQ[:, :Nq])
    args = (dev(Qq[None]), dev(Kq[None]), dev(Vq[None]), dev(sQ[None]), dev(sK[None]), dev(sV[None]))
    o32 = ifa.int_flash_attn_fwd_splitk(*args, causal=True, out_dtype=torch.float32)
    o16 = ifa.int_flash_attn_fwd_splitk(*args, causal=True, out_dtype=out_dtype)
    torch.cuda.synchronize()
    assert torch.equal(o16, o32.to(out_dtype))


@pytest.mark.parametrize("causal", [False, True])
def test_random_int8_grid_inputs_wide_scores(ifa, causal):
    # int8 values over the whole range with score spreads from flat to nearly one-hot rows
    rng = np.random.default_rng(5)
    for sigma in (0.3, 2.0, 12.0):
        Qq, Kq, Vq, sQ, sK, sV = random_int8_problem(rng, 8, 256, 128, score_sigma=sigma)
        for copies in (1, copies_for_the_fused_kernel(8, 256, 256, 128, causal)):
            O = first_copy(run_gpu(ifa, *many(copies, Qq, Kq, Vq, sQ, sK, sV), 2 * copies, 4, causal), copies)
            check_against_oracle(ifa, O.reshape(-1, 128), Qq, Kq, Vq, sQ, sK, sV, causal, label=f"int8 sigma={sigma} copies={copies}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("fused", [True, False])
def test_accumulator_extremes_through_the_fused_kernel(ifa, d, causal, fused):
    # Every entry is -128 or 127 and some keys repeat (or negate) a query's sign pattern, so Q K^T reaches
    # +-d * 128 * 128 (2^21 at d = 128) and, with V = -128 columns under flat rows, P V reaches -127 * 128 * B_c:
    # the int32 sums at the ends of their range must still come out exact (and through the few-query kernel, which takes two heads).
    rng = np.random.default_rng(77 + d)
    heads, N = 2, 384
    pick = lambda shape: np.where(rng.random(shape) < 0.5, -128, 127).astype(np.int8)
    Qq, Kq, Vq = pick((heads, N, d)), pick((heads, N, d)), pick((heads, N, d))
    Qq[:, 5] = -128; Kq[:, 9] = -128                           # score of (5, 9): d * 128 * 128, the largest possible
    Kq[:, 10] = 127                                            # score of (5, 10): -d * 128 * 127
    Kq[:, 20:40] = Qq[:, 200:220]                              # same sign pattern: large positive
    Kq[:, 300:310] = np.where(Qq[:, 100:110] < 0, 127, -128)   # opposite pattern: large negative
    Qq[:, 130:140] = 0                                         # flat rows: every P is 127
    Vq[:, :, 3] = -128; Vq[:, :, 4] = 127
    span = 6.0 / (d * 128.0 * 128.0)                           # scores within +-6
    sQ = np.full((heads, N), np.sqrt(span), np.float32) * rng.uniform(0.9, 1.1, (heads, N)).astype(np.float32)
    sK = np.full((heads, N), np.sqrt(span), np.float32) * rng.uniform(0.9, 1.1, (heads, N)).astype(np.float32)
    sV = np.array([0.01, 0.02], np.float32)
    copies = copies_for_the_fused_kernel(heads, N, N, d, causal) if fused else 1
    O = first_copy(run_gpu(ifa, *many(copies, Qq, Kq, Vq, sQ, sK, sV), copies, heads, causal), copies).reshape(-1, d)
    check_against_oracle(ifa, O, Qq, Kq, Vq, sQ, sK, sV, causal, label=f"extremes d={d} causal={causal} fused={fused}")
    flat = O.reshape(heads, N, d)[:, 130:140]
    if not causal:                                             # flat rows: O = s_V * column mean of V, exactly -128 / 127 s_V
        assert np.allclose(flat[:, :, 3], -128.0 * sV[:, None], rtol=1e-6) and np.allclose(flat[:, :, 4], 127.0 * sV[:, None], rtol=1e-6)


@pytest.mark.parametrize("H,N,d,causal", [(2, 100003, 128, True), (4, 70001, 64, False)])
def test_very_long_ragged_sequences_sampled_rows(ifa, H, N, d, causal):
    # hundreds of key blocks per workgroup, N odd: first, last and seeded rows of every head against the oracle
    w = workloads.custom("t", 1, H, N, d, causal, dist="normal", seed=N % 1000)
    x = quantized_inputs(w, scaled=True)
    rows = np.unique(np.concatenate([np.arange(0, 130), np.arange(N - 130, N), np.random.default_rng(1).integers(0, N, 150)]))
    idx = np.concatenate([h * N + rows for h in range(H)]).astype(np.int64)
    O = run_gpu(ifa, x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], 1, H, causal).cpu().numpy().reshape(-1, d)
    check_against_oracle(ifa, O[idx], x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], causal, row_idx=idx,
                         label=f"long N={N} d={d} causal={causal}")


@pytest.mark.parametrize("fused", [False, True])
def test_degenerate_inputs(ifa, fused):
    rng = np.random.default_rng(6)
    N, d = 256, 128
    copies = copies_for_the_fused_kernel(1, N, N, d, causal=True) if fused else 1      # (so few keys: the mask decides nothing)

    def one_head(Qq, Kq, Vq, sQ, sK, sV, causal):
        return first_copy(run_gpu(ifa, *many(copies, Qq, Kq, Vq, sQ, sK, sV), 1, copies, causal), copies).reshape(N, d)

    Qq, Kq, Vq, sQ, sK, sV = random_int8_problem(rng, 1, N, d)
    # all-zero Q: every score is 0, every P is 127, O is the (prefix) mean of V
    Z = np.zeros_like(Qq)
    for causal in (False, True):
        O = one_head(Z, Kq, Vq, sQ, sK, sV, causal)
        Vh = Vq[0].astype(np.float64) * float(sV[0])
        ref = np.cumsum(Vh, 0) / np.arange(1, N + 1)[:, None] if causal else np.broadcast_to(Vh.mean(0), (N, d))
        assert np.allclose(O, ref, rtol=1e-5, atol=1e-7)
    # all-zero V gives exactly zero
    O = one_head(Qq, Kq, np.zeros_like(Vq), sQ, sK, sV, False)
    assert not O.any()
    # one dominant key (a one-hot softmax row): O is that value row exactly
    Q1 = np.zeros_like(Qq); Q1[0, :, 0] = 100
    K1 = np.zeros_like(Kq); K1[0, 3, 0] = 100
    s = np.full((1, N), 0.03, np.float32)
    O = one_head(Q1, K1, Vq, s, s, sV, False)
    assert np.allclose(O, np.broadcast_to(Vq[0, 3].astype(np.float32) * sV[0], (N, d)), rtol=3e-7, atol=0)
    # causal row 0 sees key 0 only
    O = one_head(Qq, Kq, Vq, sQ, sK, sV, True)
    assert np.allclose(O[0], Vq[0, 0].astype(np.float32) * sV[0], rtol=3e-7, atol=0)
    # tiny and huge scales stay finite
    O = one_head(Qq, Kq, Vq, sQ * np.float32(1e-6), sK, sV * np.float32(1e4), False)
    assert np.all(np.isfinite(O))
    check_against_oracle(ifa, one_head(Qq, Kq, Vq, sQ * 40, sK, sV, True),  # x40: sharp rows
                         Qq, Kq, Vq, sQ * 40, sK, sV, True, label="sharp")


@pytest.mark.parametrize("H", [8, 40])
def test_output_dtypes_and_determinism(ifa, H):
    assert route(H, 512, 512, 128, True) == ("few" if H == 8 else "fused")
    w = workloads.custom("t", 1, H, 512, 128, True, seed=77)
    x = quantized_inputs(w, scaled=True)
    args = (x["Qq"], x["Kq"], x["Vq"], x["sQ"], x["sK"], x["sV"], 1, H, True)
    O32 = run_gpu(ifa, *args, out_dtype=torch.float32).cpu().numpy()
    O32b = run_gpu(ifa, *args, out_dtype=torch.float32).cpu().numpy()
    assert np.array_equal(O32, O32b)                                      # same input twice: identical bits
    O16 = run_gpu(ifa, *args, out_dtype=torch.float16).cpu().numpy()
    assert np.array_equal(O16, O32.astype(np.float16))                    # epilogue = RNE cast of the fp32 result
    Ob = run_gpu(ifa, *args, out_dtype=torch.bfloat16).float().cpu().numpy()
    assert np.array_equal(Ob, bf16_round(O32))
    # the 12-argument spec entry point writes fp16 on the stream given to ifa_set_stream
    sh = (1, H, 512, 128)
    out = torch.empty(sh, dtype=torch.float16, device="cuda")
    import ctypes
    t = [dev(x["Qq"].reshape(sh)), dev(x["Kq"].reshape(sh)), dev(x["Vq"].reshape(sh)),
         dev(x["sQ"].reshape(1, H, 512)), dev(x["sK"].reshape(1, H, 512)), dev(x["sV"].reshape(1, H))]
    L = ifa.lib()
    L.ifa_set_stream(ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert L.int_flash_attn_fwd(*[ctypes.c_void_p(a.data_ptr()) for a in t], 1, H, 512, 128, 1,
                                ctypes.c_void_p(out.data_ptr())) == 0
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), O16)


# ------------------------------------------------------------------ per-block V scales (the paper's stated next step)

@pytest.mark.parametrize("dtype", ["float32", "float16", "bfloat16"])
@pytest.mark.parametrize("N,d", [(128, 128), (384, 64), (200, 128), (77, 64), (1000, 128)])
def test_quantize_blockwise_bit_exact(ifa, dtype, N, d):
    rng = np.random.default_rng(N + d)
    x = rng.standard_normal((5, N, d)).astype(np.float32) * rng.uniform(0.1, 9, (5, N, 1)).astype(np.float32)
    x[2, :min(N, 128)] = 0.0                                  # an all-zero block
    xt = torch.from_numpy(x).to(getattr(torch, dtype)).cuda()
    q, s = ifa.quantize_blockwise(xt, 128)
    rq, rs = oracle.quantize_blockwise(xt.float().cpu().numpy(), 128)
    assert np.array_equal(q.cpu().numpy(), rq)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), rs.view(np.uint32))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,H,N,d,dist", [(1, 2, 128, 128, "normal"), (2, 4, 512, 128, "student_t3"), (1, 8, 640, 64, "uniform_outlier"),
                                          (1, 3, 333, 128, "student_t3"), (1, 8, 2048, 128, "student_t3")])
@pytest.mark.parametrize("fused", [False, True])
def test_attention_with_blockwise_v_scales(ifa, B, H, N, d, dist, causal, fused):
    w = workloads.custom("t", B, H, N, d, causal, dist=dist, seed=N + d + B)
    x = quantized_inputs(w, scaled=True)
    Bc = ifa.block_cols(d, causal)
    Vq, sVb = oracle.quantize_blockwise(x["V"], Bc)           # oracle-side inputs, as everywhere
    sh = (B, H, N, d)
    copies = copies_for_the_fused_kernel(B * H, N, N, d, causal) if fused else 1
    O = ifa.int_flash_attn_fwd(*[dev(t[None]) for t in many(copies, x["Qq"], x["Kq"], Vq, x["sQ"], x["sK"], sVb)], causal=causal,
                               out_dtype=torch.float32)
    torch.cuda.synchronize()
    check_against_oracle(ifa, first_copy(O, copies).reshape(-1, d), x["Qq"], x["Kq"], Vq, x["sQ"], x["sK"], sVb, causal,
                         label=f"block-V {B}x{H}x{N}x{d} {dist} causal={causal} fused={fused}")
    # and the GPU quantizer feeds it the same thing
    gq, gs = ifa.quantize_blockwise(dev(x["V"].reshape(sh)), Bc)
    assert np.array_equal(gq.cpu().numpy().reshape(Vq.shape), Vq) and np.array_equal(gs.cpu().numpy().reshape(sVb.shape), sVb)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Nq,Nk,d", [(1, 1000, 128), (128, 512, 128), (100, 333, 128), (256, 1024, 64), (130, 131, 128), (37, 700, 64)])
@pytest.mark.parametrize("fused", [False, True])
def test_rectangular_problems_with_blockwise_v_scales(ifa, Nq, Nk, d, causal, fused):
    # N_q != N_k together with one V scale per key block: chunked prefill / decode against per-block-quantized V
    B, H = 1, 3
    copies = copies_for_the_fused_kernel(H, Nq, Nk, d, causal) if fused else 1
    if copies is None:
        return
    w = workloads.custom("t", B, H, Nk, d, causal, dist="student_t3", seed=Nq + Nk + d)
    x = quantized_inputs(w, scaled=True)
    Bc = ifa.block_cols(d, causal)
    Vq, sVb = oracle.quantize_blockwise(x["V"], Bc)
    Qq, sQ = x["Qq"][:, Nk - Nq:], x["sQ"][:, Nk - Nq:]       # the last Nq positions as queries
    O = ifa.int_flash_attn_fwd(*[dev(t[None]) for t in many(copies, Qq, x["Kq"], Vq, sQ, x["sK"], sVb)], causal=causal, out_dtype=torch.float32)
    torch.cuda.synchronize()
    check_against_oracle(ifa, first_copy(O, copies).reshape(-1, d), Qq, x["Kq"], Vq, sQ, x["sK"], sVb, causal,
                         label=f"block-V rect {Nq}x{Nk}x{d} causal={causal} fused={fused}")


def test_blockwise_v_scales_improve_heavy_tailed_accuracy(ifa):
    # the reason for per-block scales: a few loud tokens no longer set the resolution of the whole head
    w = workloads.custom("t", 1, 4, 2048, 128, True, dist="student_t3", seed=99)
    x = quantized_inputs(w, scaled=True)
    sh = (1, 4, 2048, 128)
    ref = oracle.attention_fp64(x["Q"], x["K"], x["V"], causal=True, scale=128 ** -0.5)
    base = dict(causal=True, out_dtype=torch.float32)
    args = [dev(x["Qq"].reshape(sh)), dev(x["Kq"].reshape(sh))]
    sc = [dev(x["sQ"].reshape(1, 4, 2048)), dev(x["sK"].reshape(1, 4, 2048))]
    O_t = ifa.int_flash_attn_fwd(*args, dev(x["Vq"].reshape(sh)), *sc, dev(x["sV"].reshape(1, 4)), **base).cpu().numpy().reshape(-1, 128)
    Vb, sVb = ifa.quantize_blockwise(dev(x["V"].reshape(sh)), 128)
    O_b = ifa.int_flash_attn_fwd(*args, Vb, *sc, sVb, **base).cpu().numpy().reshape(-1, 128)
    mre_t = np.abs(O_t - ref).sum() / np.abs(ref).sum()
    mre_b = np.abs(O_b - ref).sum() / np.abs(ref).sum()
    print(f"[MRE student-t N=2048] tensor-level V scale {mre_t:.4%}   per-block V scale {mre_b:.4%}", flush=True)
    assert mre_b < mre_t


# ------------------------------------------------------------------ full-size workloads, sampled rows

def _full_size(ifa, name, scaled, full_heads, rows_per_head, vblock=False):
    """The whole workload through the launch configuration bench.py times; the oracle on every row of the first
    `full_heads` heads and `rows_per_head` seeded rows of every other head.  vblock: one V scale per key block."""
    w = workloads.WORKLOADS[name]
    Bc = ifa.block_cols(w.d, w.causal)
    sh = (w.B, w.H, w.N, w.d)
    Qd = torch.empty(sh, dtype=torch.int8, device="cuda")
    Kd = torch.empty_like(Qd)
    Vd = torch.empty_like(Qd)
    sQd = torch.empty((w.B, w.H, w.N), dtype=torch.float32, device="cuda")
    sKd = torch.empty_like(sQd)
    sVd = torch.empty((w.B, w.H, (w.N + Bc - 1) // Bc) if vblock else (w.B, w.H), dtype=torch.float32, device="cuda")
    sample = workloads.sample_rows(w, full_heads, rows_per_head)
    kept = {}
    fold = np.float32(1.0 / math.sqrt(w.d)) if scaled else np.float32(1.0)
    for h in range(w.heads):                                   # oracle-quantized inputs, one head at a time
        x = quantized_inputs(w, heads=[h])
        sq = (x["sQ"] * fold).astype(np.float32)
        b, hh = divmod(h, w.H)
        Vq, sv = oracle.quantize_blockwise(x["V"], Bc) if vblock else (x["Vq"], x["sV"])
        Qd[b, hh].copy_(torch.from_numpy(x["Qq"][0])); Kd[b, hh].copy_(torch.from_numpy(x["Kq"][0]))
        Vd[b, hh].copy_(torch.from_numpy(Vq[0]))
        sQd[b, hh].copy_(torch.from_numpy(sq[0])); sKd[b, hh].copy_(torch.from_numpy(x["sK"][0]))
        sVd[b, hh] = torch.from_numpy(np.asarray(sv[0], np.float32))
        kept[h] = (x["Qq"][0], x["Kq"][0], Vq[0], sq[0], x["sK"][0], np.asarray(sv[0], np.float32))
    out_dtype = torch.float32                                  # parity on the fp32 result; casts are tested above, on both kernels
    O = ifa.int_flash_attn_fwd(Qd, Kd, Vd, sQd, sKd, sVd, causal=w.causal, out_dtype=out_dtype)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(O).all())
    # oracle on the sampled rows, head by head (rows are independent)
    worst, worst_clean, ties, n = 0.0, 0.0, 0, 0
    for h, rows in sample:
        Qq, Kq, Vq, sq, sk, sv = kept[h]
        b, hh = divmod(h, w.H)
        got = O[b, hh].cpu().numpy()[rows]
        r = check_against_oracle(ifa, got, Qq[None], Kq[None], Vq[None], sq[None], sk[None],
                                 sv.reshape(1, -1) if vblock else sv.reshape(1), w.causal, row_idx=rows, quiet=True)
        worst, worst_clean, ties, n = max(worst, r[0]), max(worst_clean, r[1]), ties + r[2], n + r[3]
    print(f"[parity {name} scaled={scaled} vblock={vblock}] sampled rows={n} max|dO|/max|O| per head={worst:.3e} "
          f"(rows without near-ties: {worst_clean:.3e}, rows matched with flagged entries rounded the other way: {ties})", flush=True)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("scaled", [True, False])
def test_c3_full_size_sampled_rows(ifa, scaled):
    _full_size(ifa, "c3", scaled, full_heads=2, rows_per_head=64)


@pytest.mark.timeout(600)
def test_c5_full_size_sampled_rows(ifa):
    _full_size(ifa, "c5", True, full_heads=2, rows_per_head=64)


@pytest.mark.timeout(900)
def test_c4_full_size_sampled_rows(ifa):
    _full_size(ifa, "c4", True, full_heads=2, rows_per_head=64)


@pytest.mark.timeout(900)
def test_c4_full_size_sampled_rows_blockwise_v_scales(ifa):
    _full_size(ifa, "c4", True, full_heads=2, rows_per_head=64, vblock=True)

// INT-FlashAttention forward (Algorithm 1) for gfx950: calls with few queries per head (a decode step, a few draft
// tokens, a short chunk of a prefill).  Five families, all built from the tile code of the fused kernel
// (intfa_attention_tiles.h: same LDS layout, same MFMA operand order, same staging copies) and the same arithmetic:
//   int_flash_attn_fwd_packed_kernel   one workgroup of four wavefronts per head and group of 32 queries, one key block at a time;
//                                      the calls of ifa_packed_queries();
//   int_flash_attn_fwd_pair_kernel     one workgroup of twelve wavefronts for two groups of 32 queries of a head; the calls of ifa_pair_queries();
//   int_flash_attn_fwd_narrow_kernel   one or two workgroups per head and group of 32 queries, the key blocks split over
//                                      their wavefronts; bit-identical to the fused kernel's rows, needs no memory
//                                      beyond inputs and outputs; the calls of ifa_few_queries();
//   int_flash_attn_fwd_decode_kernel   two or four workgroups per head with one query (.._draft_kernel: two to eight), 16 key blocks at a time; the calls
//                                      of the few-query kernel that ifa_decode_query() names;
//   splitk_*                           the key axis of a head split over many workgroups, exactly: lines 9-10 for every
//                                      block first, then lines 11-13 on the known running maximum, then a merge;
//                                      int_flash_attn_fwd_splitk (caller's workspace) and _splitk_static (built in).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <hip/hip_bf16.h>
#include <stdint.h>
#include <mutex>
#include <type_traits>
#include <utility>

#include "intfa.h"
#include "intfa_internal.h"
#include "intfa_attention_tiles.h"

namespace {

using namespace ifa_tiles;

// ---- few queries, many keys (a decode step, a short chunk of a prefill) ---------------------------------------
// With at most a few dozen queries per head the fused kernel would keep three of its four wavefronts idle and one
// workgroup per head cannot fill the chip; what limits such a call is the latency of one key block after the other.
// Here the twelve wavefronts of a workgroup share ONE group of 32 queries and take NARROW_NB = 2 key blocks at a time,
// in two roles that run one group of blocks apart:
//   eight S wavefronts (block b of the group, key tile t): lines 9-11 for that tile.  A wavefront copies the K rows it reads
//       itself, two groups ahead, and holds the operands of the next group in registers, so its own counted waits order the
//       copies.  The extrema of the tiles meet in LDS (first barrier), every wavefront then knows m of line 10 after each
//       block of the group in order, and the P bytes go to LDS (second barrier);
//   four PV wavefronts (d tile): lines 12-13 for the group before, block by block in order.  They take its P bytes and V^T
//       operands to registers by the first barrier, which frees both places in LDS, and also copy V, a group ahead.
// What bounds it: one CU takes in about 60 GB/s however many copies are in flight (a plain streaming kernel measures 59-61
// with 32 workgroups), which is 1.07 us per group of 64 KB at d = 128; the chain MFMA - scale - exchange - exp - exchange of a
// group takes 1.0 us.  One block at a time by four wavefronts took 1.29 us per 32 KB.  DS = 2 (d = 128): two workgroups per
// (head, query group), each with half of the d columns of V and O.  Both compute the scores; K and the lines of V are then
// read twice, by CUs of one XCD at about the same time, and each CU takes in 48 KB per group.
// 32 heads of 4099 keys, one query: 21 us (without DS = 2 23.7, the packed kernel 42.5); K and V not in the caches: 128 heads of
// 16384 (DS = 1) 95 us = 5.7 TB/s (the packed kernel 148), 512 of 4096 91 us = 5.9 TB/s (131).
// LATE (d = 64, where the copies of a group take half as long and the PV wavefronts' way to the first barrier decides): they only
// bring P and V to registers and fold the group before while those come in; their MFMAs follow the barrier, and the S wavefronts, which hold
// P anyway, sum it up.  8 heads x 300 queries x 3000 keys 13.8 -> 12.8 us, 32 x 1 x 4099 17.8 -> 16.5, 64 x 4 x 8000 32.3 -> 30.0; at d = 128 the
// same measures 2 % faster to 2 % slower (32 x 1 x 4099 20.9 -> 21.2).
// Every number is computed by the same instruction sequence on the same operands as in the fused kernel (the
// integer sums are exact, the extremum is order-independent, the row sum l is taken over the same P dwords), so
// the rows are bit-identical to those of the same call on the fused kernel, and with one V scale per head to the
// corresponding rows of any other call: still Algorithm 1 at B_c = 128.  (With per-block V scales and the mask a row goes
// through the scale of a block that only other rows of its group of 32 see; which rows those are depends on N_q.)
constexpr int NARROW_BR = 32;      // queries per workgroup
constexpr int NARROW_NB = 2;       // key blocks per group
constexpr int NARROW_S_WAVES = 4 * NARROW_NB;
constexpr int NARROW_THREADS = (NARROW_S_WAVES + 4) * 64;

template <int D, int DS> struct SmemNarrow {
    alignas(4096) int8_t k[2][NARROW_NB][BC * D];
    alignas(4096) int8_t v[2][NARROW_NB][BC * (D / DS)];
    alignas(256) float sk[2][NARROW_NB * 4][64];          // per S wavefront: the 32 s_K of its key tile (+ 32 unused)
    alignas(16) v4i p[NARROW_NB][4][64];                  // per block, key tile and lane: the 16 P bytes of that lane (line 11)
    alignas(16) int ps[D == 64 ? NARROW_NB : 1][64][4];   // (LATE) per block, lane and key tile: their sum (line 12)
    alignas(16) float ext[2][NARROW_NB][32][4];           // per block, query and key tile: the extremum of a (line 10)
};
static_assert(sizeof(SmemNarrow<128, 1>) <= 160 * 1024, "LDS budget");

template <int D, bool CAUSAL, bool VB, typename OutT, int DS>
__global__ __launch_bounds__(NARROW_THREADS, 3) void int_flash_attn_fwd_narrow_kernel(
    const int8_t *__restrict__ Q, const int8_t *__restrict__ K, const int8_t *__restrict__ V,
    const float *__restrict__ sQ, const float *__restrict__ sK, const float *__restrict__ sV,
    int heads, int Nq, int Nk, int once, OutT *__restrict__ O) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ SmemNarrow<D, DS> sm;
    constexpr int KS = D / 32, NB = NARROW_NB, DV = D / DS;
    constexpr bool LATE = D == 64;                               // (see above)

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T_c = (Nk + BC - 1) / BC;
    const int qgroups = (Nq + NARROW_BR - 1) / NARROW_BR;
    const int shift = CAUSAL ? Nk - Nq : 0;
    int head, qg, half;
    if (!map_query_group<DS>(blockIdx.x, heads, qgroups, head, qg, half)) return;
    const int col0 = half * DV;                                  // first column of V and O
    const int first_q = qg * NARROW_BR;
    const int q_head = first_q + r;
    const long qrow = static_cast<long>(head) * Nq + min(q_head, Nq - 1);   // rows past Nq: a clamped copy, never stored
    const float nq2 = sQ[qrow] * (-LOG2E * ACC_UNIT);
    const int nblocks = CAUSAL ? min(Nk - 1, min(first_q + NARROW_BR, Nq) - 1 + shift) / BC + 1 : T_c;
    const int ngroups = (nblocks + NB - 1) / NB;
    float m2 = -INFINITY;                                        // line 6; kept in step by both roles
    v16i acc0;                                                   // what both accumulations start from
#pragma unroll
    for (int v = 0; v < 16; ++v) acc0[v] = ACC_START_I;
    // line 10 for the blocks of a group: the running maximum after each; leaves m2 at the last
    struct Maxima { float v[NB]; };
    auto maxima = [&](int parity) {
        Maxima m;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const v4f e = *reinterpret_cast<const v4f *>(&sm.ext[parity][b][r][0]);
            m2 = fmaxf(m2, min4(e) * nq2);
            m.v[b] = m2;
        }
        return m;
    };

    if (wave < NARROW_S_WAVES) {
        // ---- S wavefront: key tile t of block `blk` of every group
        constexpr int PER_GROUP = KS + 1;                        // copy instructions per group
        const int t = wave & 3, blk = wave >> 2;
        const BufRsrc rK = make_rsrc(K + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
        const BufRsrc rSK = make_rsrc(sK + static_cast<long>(head) * Nk, static_cast<unsigned>(Nk) * 4);
        const lds_ptr kbuf = (lds_ptr)(&sm.k[0][blk][0]);
        const lds_ptr skbuf = (lds_ptr)(&sm.sk[0][wave][0]);
        const LaneOffsets<D> lo(lane, t);
        // line 8: this wavefront's 32 rows of K and their s_K (lanes 32-63 repeat lanes 0-31): it alone reads what it
        // copies, so its own counted wait orders the two.  Rows past the end come as zeros and are masked below; a group past
        // the last one is requested nowhere, so that every group costs PER_GROUP copies.
        auto stage_group = [&](int gi) {
            const int jb = gi * NB + blk;
            const bool real = jb < nblocks;
            const Prefetch pf = {rK, rK, rSK, real ? jb * BC * D : NOWHERE, real ? jb * BC * 4 : NOWHERE, kbuf + (gi & 1) * (NB * BC * D), kbuf,
                                 skbuf + (gi & 1) * (NB * 4 * 256)};
            if (once) prefetch_k<D, true>(pf, lo, t);
            else prefetch_k<D>(pf, lo, t);
            lds_copy4(pf.sk, pf.lsk, 4 * r + 128 * t, pf.skoff);
        };
        stage_group(0);
        stage_group(1);
        const int8_t *qptr = Q + qrow * D + 16 * g;              // line 5
        v4i qf[KS];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) qf[kk] = *reinterpret_cast<const v4i *>(qptr + 32 * kk);
        // landed BEFORE the loop as far as the compiler is concerned: a wait of its own inside the loop would be a wait for
        // the staged copies as well
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(qf[kk]));
        v4i kop[KS];
        v4f skv[4];
        auto read_group = [&](int gi) {
            const lds_ptr ks = kbuf + (gi & 1) * (NB * BC * D), sk = skbuf + (gi & 1) * (NB * 4 * 256);
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) kop[kk] = *reinterpret_cast<LDS_AS const v4i *>(k_operand<D>(ks, lo, kk) + 32 * t * D);
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) skv[vq] = *reinterpret_cast<LDS_AS const v4f *>(sk + lo.sk + 32 * vq);
        };
        wait_vmcnt<PER_GROUP>();
        __builtin_amdgcn_sched_barrier(0);
        read_group(0);
        wait_lds();
        for (int gi = 0; gi < ngroups; ++gi) {                   // line 7
            // line 9, integer part
            v16i sacc = acc0;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) sacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kop[kk], qf[kk], sacc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            stage_group(gi + 2);                                 // under the MFMAs, into the place group gi has left
            __builtin_amdgcn_sched_barrier(0);
            // line 9, fp32 part, and the extrema; kept keys: index inside the block <= klimit (the causal diagonal, the
            // ragged end of the sequence, a block past the last one)
            const int j0 = (gi * NB + blk) * BC;
            const int tail = Nk - 1 - j0;
            const int klimit = CAUSAL ? min(q_head + shift - j0, tail) : tail;
            const bool masked = CAUSAL ? (j0 + BC - 1 > min(first_q + shift, Nk - 1)) : (tail < BC - 1);   // wave-uniform
            float a[16], bmin = INFINITY;
            auto scale = [&](auto with_mask) {
#pragma unroll
                for (int vq = 0; vq < 4; ++vq)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float x = (ACC_START_F - __int_as_float(sacc[4 * vq + e])) * skv[vq][e];
                        if (decltype(with_mask)::value && (32 * t + 8 * vq + 4 * g + e > klimit)) x = INFINITY;
                        a[4 * vq + e] = x;
                        bmin = fminf(bmin, x);
                    }
            };
            if (masked) scale(std::true_type{});
            else scale(std::false_type{});
            bmin = pair_min(bmin);
            if (g == 0) sm.ext[gi & 1][blk][r][t] = bmin;
            __syncthreads();
            // lines 10, 11, while the operands of the next group come in from LDS
            const auto m = maxima(gi & 1);
            wait_vmcnt<PER_GROUP>();                             // group gi + 1 has landed (group gi + 2 may be in flight)
            __builtin_amdgcn_sched_barrier(0);
            read_group(gi + 1);
            const float mm = (blk ? m.v[1] : m.v[0]) - LOG2_R_NORM;
            v4i pw;
            uint32_t psum = 0;
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(a[4 * vq + e], nq2, -mm));
                const uint32_t w = pack_p4(x);
                if (LATE) psum = __builtin_amdgcn_sad_u8(w, 0u, psum);
                pw[vq] = static_cast<int>(w);
            }
            sm.p[blk][t][lane] = pw;
            if constexpr (LATE) sm.ps[blk][lane][t] = static_cast<int>(psum);
            wait_lds();                                          // (the operands of group gi + 1 are in registers too)
            __syncthreads();
        }
        wait_all_memory();                                       // requests past the last group: nothing of mine stays in flight
        __syncthreads();                                         // the PV wavefronts' last group
        return;
    }

    // ---- PV wavefront: d tile dt of O^T = V^T P^T, one group of blocks behind
    const int dt = wave - NARROW_S_WAVES;
    const BufRsrc rV = make_rsrc(V + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const lds_ptr vbuf = (lds_ptr)(&sm.v[0][0][0]);
    const LaneOffsets<DV> lo(lane, dt);
    // With DS = 2 a row of the tile is a half row of V: the copies of LaneOffsets<DV> with the row stride of V (a piece is
    // 1024 / DV = 16 rows, which its swizzle does not see).
    constexpr int PIECES = DV / 32;
    const int srow = dt * 32 + lane / (DV / 16);
    const unsigned gvs = srow * D + col0 + 16 * ((lane % (DV / 16)) ^ v_swz<DV>(srow));
    // V of group gi (this wavefront's quarter of every block); a block past the last one is requested nowhere and comes as
    // zeros, so that every group costs NB * PIECES copies
    auto stage_blocks = [&](int gi, auto nt) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int jb = gi * NB + b;
            const int voff = jb < nblocks ? jb * BC * D : NOWHERE;
            const lds_ptr dst = vbuf + ((gi & 1) * NB + b) * (BC * DV);
            const Prefetch pf = {rV, rV, rV, voff, NOWHERE, vbuf, dst, vbuf};
            if constexpr (DS == 1) prefetch_v<D, decltype(nt)::value>(pf, lo, dt);
            else {
#pragma unroll
                for (int i = 0; i < PIECES; ++i) lds_copy16<decltype(nt)::value>(rV, dst + (dt * PIECES + i) * 1024, gvs, voff + i * (1024 / DV) * D);
            }
        }
    };
    auto stage_group = [&](int gi) {
        if (once) stage_blocks(gi, std::true_type{});
        else stage_blocks(gi, std::false_type{});
    };
    float l = 0.0f, o[16];                                       // this d tile of the running output (units of 2^26), l of the whole row
#pragma unroll
    for (int v = 0; v < 16; ++v) o[v] = 0.0f;
    // s_V: one scalar per head, or (VB) one per key block of this head, read through the scalar cache
    const float *sVh = VB ? sV + static_cast<long>(head) * T_c : sV + head;
    float sv_prev = 1.0f;
    const bool works = dt < PIECES;                              // two d tiles in a half (or D = 64): the other wavefronts only copy
    stage_group(0);
    v16i pacc[NB];
    float alpha[NB], psum[NB];
    // lines 12, 13 of group gi, block by block in order.  (A block past the last one: the maximum stays, P is 0, nothing changes.)
    auto fold = [&](int gi) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int jb = gi * NB + b;
            float alpha_o = alpha[b];
            if (VB && jb < nblocks) {                            // one V scale per key block: the running output is kept in units of the current block's
                const float sv_j = uniform(sVh[jb]);
                alpha_o = alpha[b] * uniform(sv_prev * __builtin_amdgcn_rcpf(sv_j));
                sv_prev = sv_j;
            }
            l = __builtin_fmaf(l, alpha[b], psum[b]);
#pragma unroll
            for (int v = 0; v < 16; ++v) o[v] = __builtin_fmaf(o[v], alpha_o, -(ACC_START_F - __int_as_float(pacc[b][v])));
        }
    };
    for (int gi = 0; gi <= ngroups; ++gi) {
        // Everything group gi - 1 needs goes to registers first, so that its place in LDS is free after the first barrier.
        const float m_before = m2;
        Maxima m = {};
        v4i pf[NB][4], vop[NB][4], ps[NB];
        auto products = [&]() {
            m = maxima((gi - 1) & 1);
            if (!LATE) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int b = 0; b < NB; ++b) pacc[b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vop[b][mt], pf[b][mt], mt == 0 ? acc0 : pacc[b], 0, 0, 0);
        };
        auto alphas = [&]() {
#pragma unroll
            for (int b = 0; b < NB; ++b) alpha[b] = __builtin_amdgcn_exp2f((b == 0 ? m_before : m.v[b == 0 ? 0 : b - 1]) - m.v[b]);
        };
        if (gi > 0 && works) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const lds_ptr vs = vbuf + (((gi - 1) & 1) * NB + b) * (BC * DV);
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const v2i t0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<DV>(vs, lo, dt) + 32 * mt * DV));
                    const v2i t1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<DV>(vs, lo, dt) + 16 * DV + 32 * mt * DV));
                    vop[b][mt] = v4i{t0[0], t0[1], t1[0], t1[1]};
                    pf[b][mt] = sm.p[b][mt][lane];
                }
                if constexpr (LATE) ps[b] = *reinterpret_cast<const v4i *>(&sm.ps[b][lane][0]);
            }
            if constexpr (LATE) {
                __builtin_amdgcn_sched_barrier(0);
                if (gi > 1) fold(gi - 2);
                __builtin_amdgcn_sched_barrier(0);
                wait_lds();
            } else {
                products();
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    uint32_t sum = 0;
#pragma unroll
                    for (int i = 0; i < 16; ++i) sum = __builtin_amdgcn_sad_u8(static_cast<uint32_t>(pf[b][i >> 2][i & 3]), 0u, sum);
                    psum[b] = static_cast<float>(sum);
                }
            }
        }
        __syncthreads();
        if (gi < ngroups) stage_group(gi + 1);
        if (gi > 0 && works) {
            if constexpr (LATE) {
                products();
                alphas();
#pragma unroll
                for (int b = 0; b < NB; ++b) psum[b] = static_cast<float>(ps[b][0] + ps[b][1] + ps[b][2] + ps[b][3]);
            } else {
                alphas();
                fold(gi - 1);
            }
        }
        if (gi < ngroups) {
            wait_vmcnt<NB * PIECES>();                           // my part of V of group gi has landed (group gi + 1 may be in flight)
            __syncthreads();                                     // everyone's has, and P of group gi is in LDS
        }
    }
    if (LATE && works) fold(ngroups - 1);
    wait_all_memory();

    // lines 15-17 for d tile dt (d = 32 * dt + 8 * (v / 4) + 4 * g + v % 4 of query r)
    const float lt = l + swap32(l);
    const float f = (VB ? sv_prev : sVh[0]) * ACC_UNIT / lt;
    if (q_head < Nq && works) {
        OutT *orow = O + (static_cast<long>(head) * Nq + q_head) * D + col0 + 32 * dt + 4 * g;
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            if constexpr (sizeof(OutT) == 2) {
                *reinterpret_cast<uint2 *>(orow + 8 * vq) = Pack4<OutT>::pack(o[4 * vq] * f, o[4 * vq + 1] * f, o[4 * vq + 2] * f, o[4 * vq + 3] * f);
            } else {
                *reinterpret_cast<v4f *>(orow + 8 * vq) = v4f{o[4 * vq] * f, o[4 * vq + 1] * f, o[4 * vq + 2] * f, o[4 * vq + 3] * f};
            }
        }
    }
#endif
}

// ---- more query groups than CUs: two groups of 32 queries per workgroup ------------------------------------------
// The kernel above leaves each of its roles idle for half of a step: the S wavefronts wait for the PV wavefronts to take V and P, the PV
// wavefronts for the next P.  With more groups of queries than CUs a workgroup therefore takes TWO groups, A and B, half a
// step apart, on the same K and V, each copied and read from LDS once for both.  A step (PAIR_NB = 2 key blocks) has two half steps:
//     S wavefronts    even: line 9 of A, lines 10-11 of B for the blocks before      odd: lines 10-11 of A, line 9 of B
//     PV wavefronts   even: lines 12-13 of A for the blocks before                   odd: lines 12-13 of B
// Neither part of a half step waits for the other: P of one group forms under the MFMAs of the other's scores, and a PV wavefront folds
// the half step before while its operands come in from LDS.  One barrier ends a half step: what it leaves in LDS -- extrema, P
// bytes, their sums, the factors alpha -- is read in the next.
// What bounds it: a half step takes 1985 cycles, of which the wavefronts of a SIMD issue vector instructions in 1440 (326 of them, 16
// MFMAs) and LDS is busy for 660 beside the copies; the rest is waits for LDS and the barrier.  The copies spread between the
// vector instructions, a higher priority for either role, and 10 % fewer vector instructions all measured the same within 2 %.
// 32 heads x 512 queries x 8192 keys 60 us = 1110 TOP/s (79 on the kernel above, 106 on the fused one); 65 x 128 x 1500 25 -> 17, 4 x 8192 x 8192 causal 107 -> 69.
// Rows are bit-identical to the other kernels'.  Where the lines lie: ifa_pair_queries().
constexpr int PAIR_NB = 2;         // key blocks per step
constexpr int PAIR_BR = 64;        // queries per workgroup

template <int D> struct SmemPair {
    alignas(4096) int8_t k[2][PAIR_NB][BC * D];
    alignas(4096) int8_t v[2][PAIR_NB][BC * D];
    alignas(256) float sk[2][PAIR_NB * 4][64];            // per S wavefront: the 32 s_K of its key tile (+ 32 unused)
    alignas(16) v4i p[2][PAIR_NB][4][64];                 // per query group, block, key tile and lane: the 16 P bytes of that lane
    alignas(16) int ps[2][PAIR_NB][64][4];                // per query group, block, lane and key tile: their sum
    alignas(16) float ext[2][PAIR_NB][32][4];             // per query group, block, query and key tile: the extremum (line 10)
    alignas(16) float alpha[2][PAIR_NB][32];              // per query group, block and query: e^(m_old - m)
};
static_assert(sizeof(SmemPair<128>) <= 160 * 1024 && offsetof(SmemPair<64>, v) % 4096 == 0, "LDS budget and tile bases");

template <int D, bool CAUSAL, bool VB, typename OutT>
__global__ __launch_bounds__(NARROW_THREADS, 3) void int_flash_attn_fwd_pair_kernel(
    const int8_t *__restrict__ Q, const int8_t *__restrict__ K, const int8_t *__restrict__ V,
    const float *__restrict__ sQ, const float *__restrict__ sK, const float *__restrict__ sV,
    int heads, int Nq, int Nk, int head_group, OutT *__restrict__ O) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ SmemPair<D> sm;
    constexpr int KS = D / 32, NB = PAIR_NB;

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T_c = (Nk + BC - 1) / BC, T_r = (Nq + PAIR_BR - 1) / PAIR_BR;
    const int shift = CAUSAL ? Nk - Nq : 0;
    int head, qord;
    map_workgroup(blockIdx.x, heads, T_r, head_group, CAUSAL, head, qord, false);
    const int first_q = (CAUSAL ? T_r - 1 - qord : qord) * PAIR_BR;
    // query group x (0: A, 1: B): queries first_q + 32 x + r.  Rows past Nq: a clamped copy, never stored
    int blocks[2];                                               // key blocks of either group, up to the last key it sees
    float nq2[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        blocks[x] = CAUSAL ? min(Nk - 1, min(first_q + 32 * x + 32, Nq) - 1 + shift) / BC + 1 : T_c;
        nq2[x] = sQ[static_cast<long>(head) * Nq + min(first_q + 32 * x + r, Nq - 1)] * (-LOG2E * ACC_UNIT);
    }
    const int nblocks = blocks[1];                               // (of the later queries: no fewer than blocks[0])
    const int nsteps = (nblocks + NB - 1) / NB;

    v16i acc0;                                                   // what both accumulations start from
#pragma unroll
    for (int v = 0; v < 16; ++v) acc0[v] = ACC_START_I;

    if (wave < NARROW_S_WAVES) {
        // ---- S wavefront: key tile t of block `blk` of every step, for both query groups
        constexpr int PER_STEP = KS + 1;                         // copy instructions per step
        const int t = wave & 3, blk = wave >> 2;
        const BufRsrc rK = make_rsrc(K + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
        const BufRsrc rSK = make_rsrc(sK + static_cast<long>(head) * Nk, static_cast<unsigned>(Nk) * 4);
        const lds_ptr kbuf = (lds_ptr)(&sm.k[0][blk][0]);
        const lds_ptr skbuf = (lds_ptr)(&sm.sk[0][wave][0]);
        const LaneOffsets<D> lo(lane, t);
        // line 8: this wavefront's 32 rows of K and their s_K, which it alone reads, so that its own counted wait orders the two.
        // A block past the last one is requested nowhere, so that every step costs PER_STEP copies.
        auto stage_step = [&](int n) {
            const int jb = n * NB + blk;
            const bool real = jb < nblocks;
            const Prefetch pf = {rK, rK, rSK, real ? jb * BC * D : NOWHERE, real ? jb * BC * 4 : NOWHERE, kbuf + (n & 1) * (NB * BC * D), kbuf,
                                 skbuf + (n & 1) * (NB * 4 * 256)};
            prefetch_k<D>(pf, lo, t);
            lds_copy4(pf.sk, pf.lsk, 4 * r + 128 * t, pf.skoff);
        };
        stage_step(0);
        stage_step(1);
        v4i qf[2][KS];                                           // line 5
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int8_t *qptr = Q + (static_cast<long>(head) * Nq + min(first_q + 32 * x + r, Nq - 1)) * D + 16 * g;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) qf[x][kk] = *reinterpret_cast<const v4i *>(qptr + 32 * kk);
        }
        // landed BEFORE the loop as far as the compiler is concerned: a wait of its own inside the loop would be a wait for
        // the staged copies as well
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(qf[x][kk]));
        asm volatile("" : "+v"(nq2[0]), "+v"(nq2[1]));
        v4i kop[KS];
        v4f skv[4];
        auto read_k = [&](int n) {
            const lds_ptr ks = kbuf + (n & 1) * (NB * BC * D);
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) kop[kk] = *reinterpret_cast<LDS_AS const v4i *>(k_operand<D>(ks, lo, kk) + 32 * t * D);
        };
        auto read_sk = [&](int n) {
            const lds_ptr sk = skbuf + (n & 1) * (NB * 4 * 256);
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) skv[vq] = *reinterpret_cast<LDS_AS const v4f *>(sk + lo.sk + 32 * vq);
        };
        v16i sacc;
        float a[2][16];
        // line 9 of group x, integer part
        auto gemm = [&](int x) {
            sacc = acc0;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) sacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kop[kk], qf[x][kk], sacc, 0, 0, 0);
        };
        // line 9, fp32 part, and the extrema; kept keys: index inside the block <= klimit (the causal diagonal, the
        // ragged end of the sequence, a block past the last one)
        auto scores = [&](int x, int n) {
            const int j0 = (n * NB + blk) * BC, fq = first_q + 32 * x;
            const int tail = Nk - 1 - j0;
            const int klimit = CAUSAL ? min(fq + r + shift - j0, tail) : tail;
            const bool masked = CAUSAL ? (j0 + BC - 1 > min(fq + shift, Nk - 1)) : (tail < BC - 1);   // wave-uniform
            float bmin = INFINITY;
            auto scale = [&](auto with_mask) {
#pragma unroll
                for (int vq = 0; vq < 4; ++vq)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float y = (ACC_START_F - __int_as_float(sacc[4 * vq + e])) * skv[vq][e];
                        if (decltype(with_mask)::value && (32 * t + 8 * vq + 4 * g + e > klimit)) y = INFINITY;
                        a[x][4 * vq + e] = y;
                        bmin = fminf(bmin, y);
                    }
            };
            if (masked) scale(std::true_type{});
            else scale(std::false_type{});
            bmin = pair_min(bmin);
            if (g == 0) sm.ext[x][blk][r][t] = bmin;
        };
        // lines 10, 11 of group x; every wavefront follows the running maximum through both blocks of the step
        float m2[2] = {-INFINITY, -INFINITY};                    // line 6
        auto weights = [&](int x) {
            float before = m2[x], m = m2[x];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const v4f e = *reinterpret_cast<const v4f *>(&sm.ext[x][b][r][0]);
                m2[x] = fmaxf(m2[x], min4(e) * nq2[x]);
                if (b == blk) m = m2[x];
                if (b < blk) before = m2[x];
            }
            if (t == 0 && g == 0) sm.alpha[x][blk][r] = __builtin_amdgcn_exp2f(before - m);
            const float mm = m - LOG2_R_NORM;
            v4i pw;
            uint32_t psum = 0;
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                float e[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) e[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(a[x][4 * vq + i], nq2[x], -mm));
                const uint32_t w = pack_p4(e);
                psum = __builtin_amdgcn_sad_u8(w, 0u, psum);
                pw[vq] = static_cast<int>(w);
            }
            sm.p[x][blk][t][lane] = pw;
            sm.ps[x][blk][lane][t] = static_cast<int>(psum);
        };
        wait_vmcnt<PER_STEP>();                                  // step 0 has landed
        __builtin_amdgcn_sched_barrier(0);
        read_k(0);
        read_sk(0);
        wait_lds();
        for (int n = 0; n < nsteps; ++n) {                       // line 7
            gemm(0);
            __builtin_amdgcn_sched_barrier(0);
            stage_step(n + 2);                                   // into the place step n has left
            __builtin_amdgcn_sched_barrier(0);
            if (n > 0) weights(1);
            scores(0, n);
            wait_lds();
            __syncthreads();
            gemm(1);
            __builtin_amdgcn_sched_barrier(0);
            wait_vmcnt<PER_STEP>();                              // step n + 1 has landed (step n + 2 may be in flight)
            __builtin_amdgcn_sched_barrier(0);
            read_k(n + 1);
            weights(0);
            scores(1, n);
            read_sk(n + 1);
            wait_lds();
            __syncthreads();
        }
        weights(1);
        wait_all_memory();                                       // requests past the last step: nothing of mine stays in flight
        __syncthreads();
        return;
    }

    // ---- PV wavefront: d tile dt of O^T = V^T P^T
    const int dt = wave - NARROW_S_WAVES;
    const BufRsrc rV = make_rsrc(V + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const lds_ptr vbuf = (lds_ptr)(&sm.v[0][0][0]);
    const LaneOffsets<D> lo(lane, dt);
    // V of step n (this wavefront's quarter of every block); a block past the last one is requested nowhere and comes as zeros
    auto stage_step = [&](int n) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int jb = n * NB + b;
            const Prefetch pf = {rV, rV, rV, jb < nblocks ? jb * BC * D : NOWHERE, NOWHERE, vbuf, vbuf + ((n & 1) * NB + b) * (BC * D), vbuf};
            prefetch_v<D>(pf, lo, dt);
        }
    };
    float l[2] = {0.0f, 0.0f}, o[2][16];                         // this d tile of the running output (units of 2^26), l of the whole row
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[x][v] = 0.0f;
    // s_V: one scalar per head, or (VB) one per key block of this head, read through the scalar cache
    const float *sVh = VB ? sV + static_cast<long>(head) * T_c : sV + head;
    float sv_prev[2] = {1.0f, 1.0f};
    const bool works = dt < KS;                                  // two d tiles at D = 64: the other wavefronts only copy
    v4i vop[NB][4];
    v16i pacc[NB];
    float alpha[NB];
    int psum[NB];
    // lines 12, 13 of group x for step n, block by block in order, from what gemm() left.  (A block past the last one: the maximum
    // stays, P is 0, nothing changes.)
    auto fold = [&](int x, int n) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int jb = n * NB + b;
            float alpha_o = alpha[b];
            if (VB && jb < blocks[x]) {                          // one V scale per key block: the running output is kept in units of the current block's
                const float sv_j = uniform(sVh[jb]);
                alpha_o = alpha[b] * uniform(sv_prev[x] * __builtin_amdgcn_rcpf(sv_j));
                sv_prev[x] = sv_j;
            }
            l[x] = __builtin_fmaf(l[x], alpha[b], static_cast<float>(psum[b]));
#pragma unroll
            for (int v = 0; v < 16; ++v) o[x][v] = __builtin_fmaf(o[x][v], alpha_o, -(ACC_START_F - __int_as_float(pacc[b][v])));
        }
    };
    // line 13, integer part, of group x for step n, and what its fold will take; `before` runs while the operands come in from LDS
    auto gemm = [&](int x, int n, auto before) {
        v4i pf[NB][4], ps[NB];
        float al[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) pf[b][mt] = sm.p[x][b][mt][lane];
            ps[b] = *reinterpret_cast<const v4i *>(&sm.ps[x][b][lane][0]);
            al[b] = sm.alpha[x][b][r];
        }
        __builtin_amdgcn_sched_barrier(0);
        before();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int b = 0; b < NB; ++b) pacc[b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vop[b][mt], pf[b][mt], mt == 0 ? acc0 : pacc[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            alpha[b] = al[b];
            psum[b] = ps[b][0] + ps[b][1] + ps[b][2] + ps[b][3];
        }
    };
    stage_step(0);
    stage_step(1);
    __syncthreads();                                             // half step 0: nothing to do yet
    wait_vmcnt<NB * KS>();                                       // my part of V of step 0 has landed (step 1 may be in flight)
    __syncthreads();
    for (int n = 0; n < nsteps; ++n) {
        if (works) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const lds_ptr vs = vbuf + ((n & 1) * NB + b) * (BC * D);
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const v2i t0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<D>(vs, lo, dt) + 32 * mt * D));
                    const v2i t1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<D>(vs, lo, dt) + 16 * D + 32 * mt * D));
                    vop[b][mt] = v4i{t0[0], t0[1], t1[0], t1[1]};
                }
            }
            gemm(0, n, [&]() { if (n > 0) fold(1, n - 1); });
        }
        wait_lds();
        __syncthreads();                                         // V of step n is in registers, P of group B in LDS
        stage_step(n + 2);
        if (works) gemm(1, n, [&]() { fold(0, n); });
        if (n + 1 < nsteps) {
            wait_vmcnt<NB * KS>();                               // my part of V of step n + 1 has landed (step n + 2 may be in flight)
            __syncthreads();                                     // everyone's has, and P of group A is in LDS
        }
    }
    if (works) fold(1, nsteps - 1);
    wait_all_memory();

    // lines 15-17 for d tile dt (d = 32 * dt + 8 * (v / 4) + 4 * g + v % 4 of query r)
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const float lt = l[x] + swap32(l[x]);
        const float f = (VB ? sv_prev[x] : sVh[0]) * ACC_UNIT / lt;
        const int q_head = first_q + 32 * x + r;
        if (q_head < Nq && works) {
            OutT *orow = O + (static_cast<long>(head) * Nq + q_head) * D + 32 * dt + 4 * g;
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                if constexpr (sizeof(OutT) == 2) {
                    *reinterpret_cast<uint2 *>(orow + 8 * vq) = Pack4<OutT>::pack(o[x][4 * vq] * f, o[x][4 * vq + 1] * f, o[x][4 * vq + 2] * f, o[x][4 * vq + 3] * f);
                } else {
                    *reinterpret_cast<v4f *>(orow + 8 * vq) = v4f{o[x][4 * vq] * f, o[x][4 * vq + 1] * f, o[x][4 * vq + 2] * f, o[x][4 * vq + 3] * f};
                }
            }
        }
    }
#endif
}

// ---- few queries, few keys (or d = 64 and more workgroups than CUs) ----------------------------------------------
// The kernel above needs twelve wavefronts and a CU for one group of queries, takes two key blocks at a time and ends one step after
// its scores do.  On few keys that is mostly start and end.  Here four wavefronts take one key block at a time in one role:
//     wavefront w computes S^T for key tile w (32 keys), scales it, takes its extremum;
//     the four per-query extrema meet in LDS (first barrier of the block): everyone knows m of line 10 for the whole block;
//     wavefront w computes the 16 P bytes per lane of its key tile and leaves them in LDS (second barrier);
//     wavefront w then computes the d tile w (32 of the d columns) of O^T = V^T P^T over all 128 keys, with the P operands of
//     the four key tiles from LDS, and folds it into its 16 registers of the running output.
// What bounds it is that chain, 1.3 us per block, which is why it loses on longer key sequences; at d = 64 two workgroups share a CU
// and fill in for each other.  K and V come in through a ring of PACKED_NSTAGE blocks, filled three ahead; the wait for a block is
// a counted s_waitcnt (every wavefront issues the same number of copies per block) in front of the second barrier of the block
// before, which thereby also publishes the staged block; the first barrier releases the stage of the block before.
// The arithmetic is that of the other two kernels, operation by operation.  Where the lines lie: ifa_packed_queries().
constexpr int PACKED_BR = 32;      // queries per workgroup
constexpr int PACKED_NSTAGE = 4;

template <int D> struct SmemPacked {
    alignas(4096) int8_t k[PACKED_NSTAGE][BC * D];
    alignas(4096) int8_t v[PACKED_NSTAGE][BC * D];
    alignas(512) float sk[PACKED_NSTAGE][BC];
    alignas(16) float ext[4][32];          // per key tile and query: the tile's extremum of a (line 10)
    alignas(16) v4i p[4][64];              // per key tile and lane: the 16 P bytes of that lane (line 11)
};
static_assert(sizeof(SmemPacked<128>) <= 160 * 1024 && 2 * sizeof(SmemPacked<64>) <= 160 * 1024 && offsetof(SmemPacked<64>, v) % 4096 == 0, "LDS budget (d = 64: two workgroups per CU) and tile bases");

template <int D, bool CAUSAL, bool VB, typename OutT>
__global__ __launch_bounds__(THREADS) void int_flash_attn_fwd_packed_kernel(
    const int8_t *__restrict__ Q, const int8_t *__restrict__ K, const int8_t *__restrict__ V,
    const float *__restrict__ sQ, const float *__restrict__ sK, const float *__restrict__ sV,
    int heads, int Nq, int Nk, OutT *__restrict__ O) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ SmemPacked<D> sm;
    constexpr int KS = D / 32;
    constexpr int PER_BLOCK = 2 * KS + 1;                        // copy instructions per wavefront and block

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T_c = (Nk + BC - 1) / BC;
    const int qgroups = (Nq + PACKED_BR - 1) / PACKED_BR;
    const int shift = CAUSAL ? Nk - Nq : 0;
    // all query groups of a head on one XCD (workgroups go round-robin over the 8 XCDs by linear id)
    int head, qg;
    if ((heads & 7) == 0) { const int s_ = blockIdx.x >> 3; head = (s_ / qgroups) * 8 + (blockIdx.x & 7); qg = s_ % qgroups; }
    else { head = blockIdx.x / qgroups; qg = blockIdx.x % qgroups; }
    const int first_q = qg * PACKED_BR;
    const int q_head = first_q + r;
    const long qrow = static_cast<long>(head) * Nq + min(q_head, Nq - 1);   // rows past Nq: a clamped copy, never stored

    const int8_t *Kh = K + static_cast<long>(head) * Nk * D;
    const int8_t *Vh = V + static_cast<long>(head) * Nk * D;
    const float *sKh = sK + static_cast<long>(head) * Nk;
    const lds_ptr kbuf = (lds_ptr)(&sm.k[0][0]);
    const lds_ptr vbuf = (lds_ptr)(&sm.v[0][0]);
    const lds_ptr skbuf = (lds_ptr)(&sm.sk[0][0]);
    const int nblocks = CAUSAL ? min(Nk - 1, min(first_q + PACKED_BR, Nq) - 1 + shift) / BC + 1 : T_c;

    const BufRsrc rK = make_rsrc(Kh, static_cast<unsigned>(Nk) * D);
    const BufRsrc rV = make_rsrc(Vh, static_cast<unsigned>(Nk) * D);
    const BufRsrc rSK = make_rsrc(sKh, static_cast<unsigned>(Nk) * 4);
    const LaneOffsets<D> lo(lane, wave);

    // line 8 for block jb into stage jb % PACKED_NSTAGE; a block past the last one is requested nowhere (no data moves), so
    // that every block costs every wavefront PER_BLOCK copy instructions and the counted wait below stays valid
    auto stage_block = [&](int jb) {
        const int st = jb % PACKED_NSTAGE;
        const bool real = jb < nblocks;
        const Prefetch pf = {rK, rV, rSK, real ? jb * BC * D : NOWHERE, real ? jb * BC * 4 : NOWHERE,
                             kbuf + st * BC * D, vbuf + st * BC * D, skbuf + st * BC * 4};
        prefetch_k<D>(pf, lo, wave);
        prefetch_v<D>(pf, lo, wave);
        lds_copy4(pf.sk, pf.lsk + 256 * (wave & 1), 4 * lane + 256 * (wave & 1), pf.skoff);   // wavefronts 2, 3 repeat 0, 1
    };
    stage_block(0);
    stage_block(1);
    stage_block(2);

    // line 5
    const int8_t *qptr = Q + qrow * D + 16 * g;
    v4i qf[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = *reinterpret_cast<const v4i *>(qptr + 32 * kk);
    float nq2 = sQ[qrow] * (-LOG2E * ACC_UNIT);
    // The loads above must have landed BEFORE the loop as far as the compiler is concerned: a wait for them inside the
    // loop would be a wait for every outstanding vector-memory operation, the staged copies included.
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(qf[kk]));
    asm volatile("" : "+v"(nq2));

    // line 6: this wavefront's d tile of the running output (units of 2^26), m and l of the whole row
    float m2 = -INFINITY, l = 0.0f, o[16];
    v16i acc0;                                                   // what both accumulations start from
#pragma unroll
    for (int v = 0; v < 16; ++v) { o[v] = 0.0f; acc0[v] = ACC_START_I; }

    // s_V: one scalar per head, or (VB) one per key block of this head, read through the scalar cache
    const float *sVh = VB ? sV + static_cast<long>(head) * T_c : sV + head;
    float sv_prev = 1.0f;
    wait_vmcnt<2 * PER_BLOCK>();                                 // my pieces of block 0 have landed (blocks 1 and 2 may be in flight)
    __syncthreads();                                             // everyone's have
    for (int jb = 0; jb < nblocks; ++jb) {                       // line 7
        const int st = jb % PACKED_NSTAGE, j0 = jb * BC;
        // with one V scale per key block the running output is kept in units of the current block's scale (as in the fused kernel)
        const float sv_j = VB ? uniform(sVh[jb]) : 1.0f;
        const float oscale = VB ? uniform(sv_prev * __builtin_amdgcn_rcpf(sv_j)) : 1.0f;
        sv_prev = sv_j;
        const lds_ptr ks = kbuf + st * BC * D, vs = vbuf + st * BC * D, sk = skbuf + st * BC * 4;

        // line 9 for key tile `wave`
        v4i kop[KS];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) kop[kk] = *reinterpret_cast<LDS_AS const v4i *>(k_operand<D>(ks, lo, kk) + 32 * wave * D);
        v4f skv[4];
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) skv[vq] = *reinterpret_cast<LDS_AS const v4f *>(sk + lo.sk + 128 * wave + 32 * vq);
        // (registers are plentiful here: the accumulators start from a register block holding the constant, and every
        // MFMA is the compiler's own, with its dependency handling)
        v16i sacc = acc0;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) sacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kop[kk], qf[kk], sacc, 0, 0, 0);
        // kept keys: index inside the block <= klimit (the causal diagonal, the ragged end of the sequence)
        const int tail = Nk - 1 - j0;
        const int klimit = CAUSAL ? min(q_head + shift - j0, tail) : tail;
        const bool masked = CAUSAL ? (j0 + BC - 1 > min(first_q + shift, Nk - 1)) : (tail < BC - 1);   // wave-uniform
        float a[16], bmin = INFINITY;
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float x = (ACC_START_F - __int_as_float(sacc[4 * vq + e])) * skv[vq][e];
                if (masked && (32 * wave + 8 * vq + 4 * g + e > klimit)) x = INFINITY;
                a[4 * vq + e] = x;
                bmin = fminf(bmin, x);
            }
        bmin = pair_min(bmin);
        if (g == 0) sm.ext[wave][r] = bmin;
        __syncthreads();
        // every wavefront is past the second GEMM of block jb - 1: the stage that block used takes block jb + 3
        stage_block(jb + 3);
        // line 10 over the whole block
        bmin = fminf(fminf(sm.ext[0][r], sm.ext[1][r]), fminf(sm.ext[2][r], sm.ext[3][r]));
        const float m_new = fmaxf(m2, bmin * nq2);
        const float alpha = __builtin_amdgcn_exp2f(m2 - m_new);
        const float mm = m_new - LOG2_R_NORM;
        m2 = m_new;
        // line 11 for key tile `wave`
        v4i pw;
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(a[4 * vq + e], nq2, -mm));
            const uint32_t w = pack_p4(x);
            pw[vq] = static_cast<int>(w);
        }
        sm.p[wave][lane] = pw;
        wait_vmcnt<2 * PER_BLOCK>();                             // my pieces of block jb + 1 have landed (two later blocks may be in flight)
        __syncthreads();                                         // everyone's have, and every P tile of this block is in LDS
        // lines 12, 13: d tile `wave` of O^T = V^T P^T over the four key tiles, the row sum over the same P dwords
        if (wave >= KS) continue;                                // D = 64: two d tiles; the other wavefronts only take part above
        v16i pacc;
        uint32_t psum = 0;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const v4i pf = sm.p[mt][lane];
            const v2i t0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<D>(vs, lo, wave) + 32 * mt * D));
            const v2i t1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<D>(vs, lo, wave) + 16 * D + 32 * mt * D));
            const v4i vop = {t0[0], t0[1], t1[0], t1[1]};
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) psum = __builtin_amdgcn_sad_u8(static_cast<uint32_t>(pf[vq]), 0u, psum);
            pacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(vop, pf, mt == 0 ? acc0 : pacc, 0, 0, 0);
        }
        l = __builtin_fmaf(l, alpha, static_cast<float>(psum));
        const float alpha_o = VB ? alpha * oscale : alpha;
#pragma unroll
        for (int v = 0; v < 16; ++v) o[v] = __builtin_fmaf(o[v], alpha_o, -(ACC_START_F - __int_as_float(pacc[v])));
    }
    wait_all_memory();                                           // requests past the last block: nothing of mine stays in flight

    // lines 15-17 for d tile `wave` (d = 32 * wave + 8 * (v / 4) + 4 * g + v % 4 of query r)
    const float lt = l + swap32(l);
    const float f = (VB ? sv_prev : sVh[0]) * ACC_UNIT / lt;
    if (q_head < Nq && wave < KS) {
        OutT *orow = O + (static_cast<long>(head) * Nq + q_head) * D + 32 * wave + 4 * g;
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            if constexpr (sizeof(OutT) == 2) {
                *reinterpret_cast<uint2 *>(orow + 8 * vq) = Pack4<OutT>::pack(o[4 * vq] * f, o[4 * vq + 1] * f, o[4 * vq + 2] * f, o[4 * vq + 3] * f);
            } else {
                *reinterpret_cast<v4f *>(orow + 8 * vq) = v4f{o[4 * vq] * f, o[4 * vq + 1] * f, o[4 * vq + 2] * f, o[4 * vq + 3] * f};
            }
        }
    }
#endif
}

// ---- one query per head (a decode step) ---------------------------------------------------------------------------
// The few-query kernel forms P for 32 queries two key blocks at a time, with two barriers and the chain MFMA - scale - exchange - exp - exchange - MFMA in
// each such step (1.0 us), also where there is one query.  Here a workgroup takes a WINDOW of 16 key blocks at once, one to each of its 16 wavefronts, and
// a wavefront does everything for its own block:
//   line 9 key tile by key tile, the integer sums of the one query to LDS; then, four keys to a lane, their scaling and the extremum of the
//   block; (barrier) the running maximum in front of it from the extrema of all, P, alpha and row sum; P V of the block, its sums to LDS;
//   (barrier) a thread per output column folds the blocks of the window in order: lines 12 and 13.
// Two barriers per 2048 keys.  K and V come through a ring per wavefront, ordered by its counted waits, which runs on through the barriers.  Four (d = 64: two)
// workgroups per head, on one XCD, have 32 columns of V and O each; all read K, each beginning with another of a wavefront's tiles: what one
// brings in, the others find in L2 (a CU takes in 59 GB/s from beyond it and 120 - 140 out of it).
// What bounds it is the chain of a wavefront through a window, 5 us at d = 128 (4.9 with the next entry of the ring requested before the operands of this one are read,
// as it is; 5.9 with the place of this one refilled once they are read, twice as much in flight; with products of 32 x 32 x 32, whose chains are
// twice as long, 5.9 and 6.2; eight wavefronts with two blocks each and 32 x 32 x 32 6.4), beside 2.3 us that 320 KB take at best (23 % of the cycles issue vector
// instructions, 27 % are LDS's); as long with per-block V scales, which cost .6 us a call.  Few-query kernel / this one, us, in a graph:
// 32 heads x 4099 keys 20.7 / 14.6, 8 x 2603 13.1 / 8.9, 64 x 579 6.3 / 4.9, 16 x 16384 64.8 / 42.1, 64 x 18595 97.6 / 79; d = 64, 32 x 4099 16.2 / 11.0, 64 x 32768 109 / 74.
// The numbers are those of the other kernels: integer sums, the maximum is order-independent, the row sum is kept per half of the keys (bit 2 of the key's index)
// as their lanes do, and the fp32 folds are the same, block by block.
constexpr int DEC_WAVES = 16, DEC_THREADS = DEC_WAVES * 64;      // wavefronts = key blocks per window
template <int D, int DS, int RING> struct DecodePlan {
    static constexpr int DV = D / DS;
    static constexpr int VE = 4 / DS;                            // ring entries (32 D bytes) of V, 32 DS keys each, behind four key tiles of K
    static constexpr int EPW = 4 + VE;                           // ... per window
    static constexpr int R = RING;                               // entries of the ring, one of them being read
    static constexpr int copies(int k) { return D / 32 + (k % EPW == 0 ? 2 : 0); }   // of entry k (the first of a window brings the s_K)
    static constexpr int behind(int k) { int n = 0; for (int j = 1; j < R - 1; ++j) n += copies(k + j); return n; }   // in flight behind entry k
};
template <int D, int DS> struct SmemDecode {
    using P = DecodePlan<D, DS, D == 128 ? 2 : 4>;
    alignas(4096) int8_t ring[DEC_WAVES][P::R][32 * D];
    alignas(16) int s[DEC_WAVES][BC];                            // Q K^T of the wavefront's block; then its P bytes (8 dwords per key tile)
    alignas(256) float sk[2][DEC_WAVES][BC];                     // of this window and the next
    alignas(16) float pv[DEC_WAVES][P::DV];                      // minus P V, units of 2^26
    alignas(16) float ext[DEC_WAVES];                            // extremum of a per block (line 10)
    alignas(16) float alpha[DEC_WAVES];                          // e^(m_old - m)
    alignas(16) float psum[DEC_WAVES][2];                        // the row sums over either half of the keys
};
static_assert(sizeof(SmemDecode<128, 4>) <= 160 * 1024 && sizeof(SmemDecode<64, 2>) <= 160 * 1024, "LDS budget");

template <typename F, int... I> __device__ __forceinline__ void for_each_int(F f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
#if defined(__HIP_DEVICE_COMPILE__)
template <int CTRL> __device__ __forceinline__ unsigned dpp(unsigned old, unsigned x) {
    return static_cast<unsigned>(__builtin_amdgcn_update_dpp(static_cast<int>(old), static_cast<int>(x), CTRL, 0xf, 0xf, false));
}
constexpr int ROW_SHR = 0x110, ROW_ROR = 0x120;
// minimum over the 32 lanes of a half wavefront; sum over those of them of one parity
__device__ __forceinline__ float half_min(float x) {
    for_each_int([&](auto i) {
        const unsigned u = __float_as_uint(x);
        x = fminf(x, __uint_as_float(dpp<ROW_ROR | (1 << decltype(i)::value)>(u, u)));
    }, std::make_integer_sequence<int, 4>{});
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fminf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}
__device__ __forceinline__ unsigned parity_sum(unsigned x) {
    x += dpp<ROW_ROR | 8>(x, x);
    x += dpp<ROW_ROR | 4>(x, x);
    x += dpp<ROW_ROR | 2>(x, x);
    const auto sw = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return sw[0] + sw[1];
}
__device__ __forceinline__ float lane_value(float x, int lane) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), lane)); }
#endif

template <int D, int DS>
__global__ __launch_bounds__(DEC_THREADS, 4) void int_flash_attn_fwd_decode_kernel(
    const int8_t *__restrict__ Q, const int8_t *__restrict__ K, const int8_t *__restrict__ V,
    const float *__restrict__ sQ, const float *__restrict__ sK, const float *__restrict__ sV,
    int heads, int Nk, int vblock, int o_dtype, void *__restrict__ O) {
#if defined(__HIP_DEVICE_COMPILE__)
    using P = typename SmemDecode<D, DS>::P;
    __shared__ SmemDecode<D, DS> sm;
    constexpr int KS = D / 32, KK = D / 64, DV = P::DV, VE = P::VE, EPW = P::EPW, R = P::R;
    static_assert(DV == 32, "one d tile");

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, c = lane & 15, G = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T_c = (Nk + BC - 1) / BC, windows = (T_c + DEC_WAVES - 1) / DEC_WAVES;
    int head, qg, part;
    if (!map_query_group<DS>(blockIdx.x, heads, 1, head, qg, part)) return;
    const int col0 = part * DV;                                  // first column of V and O

    const BufRsrc rK = make_rsrc(K + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const BufRsrc rV = make_rsrc(V + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const BufRsrc rSK = make_rsrc(sK + static_cast<long>(head) * Nk, static_cast<unsigned>(Nk) * 4);
    const LaneOffsets<D> lo(lane, 0);
    const lds_ptr ring = (lds_ptr)(&sm.ring[wave][0][0]), skbuf = (lds_ptr)(&sm.sk[0][wave][0]);
    const unsigned gv = (lane / (DV / 16)) * D + col0 + 16 * (lane % (DV / 16));    // V: whole rows of DV bytes, which the transposing reads take without conflicts
    const int turn = part * (4 / DS);                            // which of its key tiles a wavefront begins with
    int in = 0, slot = 0;                                                // of the ring: the oldest entry's
    // entry k of window w into the ring; what lies past the end comes as zeros, what is past the last window is requested nowhere: the counts stay valid
    auto issue = [&](auto k_, int w) {
        constexpr int k = decltype(k_)::value % EPW;
        const int key0 = (w * DEC_WAVES + wave) * BC;            // first key of this wavefront's block
        const lds_ptr dst = ring + in * (32 * D);
        in = in + 1 == R ? 0 : in + 1;
        if constexpr (k < 4) {
            const int key = key0 + 32 * ((k + turn) & 3), off = key < Nk ? key * D : NOWHERE;
            lds_copy16_run<KS>(rK, dst, lo.gk, lo.gk, off);
            if constexpr (k == 0) {
#pragma unroll
                for (int i = 0; i < 2; ++i) lds_copy4(rSK, skbuf + (w & 1) * (DEC_WAVES * BC * 4) + 256 * i, 4 * lane, key0 + 64 * i < Nk ? (key0 + 64 * i) * 4 : NOWHERE);
            }
        } else {
            const int key = key0 + 32 * DS * (k - 4), off = key < Nk ? key * D : NOWHERE;
#pragma unroll
            for (int i = 0; i < KS; ++i) lds_copy16(rV, dst + 1024 * i, gv, off + i * (1024 / DV) * D);
        }
    };
    for_each_int([&](auto k) { issue(k, 0); }, std::make_integer_sequence<int, R - 1>{});

    // line 5, in every column of the operand.  The products are 16 x 16 x 64: half of the work of 32 x 32 x 32 goes to columns that nobody asked for, and
    // their chains are half as long.  Lane (c, G) = (lane % 16, lane / 16) holds 16 bytes from 16 G on of row c, and of the result rows 4 G .. 4 G + 3 of column c.
    const int8_t *qptr = Q + static_cast<long>(head) * D + 16 * G;
    v4i qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const v4i *>(qptr + 64 * kk);
    float nq2 = sQ[head] * (-LOG2E * ACC_UNIT);
    // landed BEFORE the loop as far as the compiler is concerned: a wait of its own inside would be a wait for the copies as well
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(qf[kk]));
    asm volatile("" : "+v"(nq2));
    const v4i acc0 = {ACC_START_I, ACC_START_I, ACC_START_I, ACC_START_I};   // what both accumulations start from
    const unsigned k0 = c * D + 16 * (G ^ k_swz<D>(c));          // K operand (see LaneOffsets): the next 64 columns at k0 ^ 64, the next 16 keys, which the swizzle does not see, at + 16 D
    // transposing read of V, keys 16 G .. 16 G + 7 of 64: lane i of the group addresses row i / 2, byte half i % 2, and receives column i
    const unsigned v0 = (16 * G + (c >> 1)) * DV + 8 * (c & 1);

    const float *sVh = vblock ? sV + static_cast<long>(head) * T_c : sV + head;
    float carry = -INFINITY;                                     // m in front of the window (line 6)
    float o = 0.0f, l0 = 0.0f, l1 = 0.0f, sv_prev = 1.0f;        // of column tid
    int *const pbytes = &sm.s[wave][0];

    for (int w = 0; w < windows; ++w) {
        const bool mine = w * DEC_WAVES + wave < T_c;            // (wave-uniform) the last window may have no block for this wavefront
        // the coming entry has landed; the one R - 1 further on goes into the place of the last one; take(where it is) reads it
        auto advance = [&](auto k_, auto take) {
            constexpr int k = decltype(k_)::value;
            wait_vmcnt<P::behind(k)>();
            __builtin_amdgcn_sched_barrier(0);
            issue(std::integral_constant<int, k + R - 1>{}, w + (k + R - 1) / EPW);
            __builtin_amdgcn_sched_barrier(0);
            take(ring + slot * (32 * D));
            slot = slot + 1 == R ? 0 : slot + 1;
        };
        float a[4], bmin = INFINITY;
        if (mine) {
        // line 9, integer part, key tile by key tile; the lanes of one column hand the sums on
        for_each_int([&](auto k) {
            const int tile = (decltype(k)::value + turn) & 3;
            v4i kop[2][KK], sacc[2];
            advance(k, [&](lds_ptr ks) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) kop[h][kk] = *reinterpret_cast<LDS_AS const v4i *>(lds_xor(ks, 64 * kk, k0) + 16 * D * h);
            });
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                for (int h = 0; h < 2; ++h) sacc[h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(kop[h][kk], qf[kk], kk == 0 ? acc0 : sacc[h], 0, 0, 0);
            if (c == 0) {
#pragma unroll
                for (int h = 0; h < 2; ++h) *reinterpret_cast<v4i *>(&sm.s[wave][32 * tile + 16 * h + 4 * G]) = sacc[h];
            }
        }, std::make_integer_sequence<int, 4>{});
        // line 9, fp32 part, and the extremum of the block: keys 4 r .. 4 r + 3 of it (lanes 32 - 63 repeat lanes 0 - 31); the one query sees every key there is
        const int left = Nk - ((w * DEC_WAVES + wave) * BC + 4 * r);
        const v4f skv = *reinterpret_cast<const v4f *>(&sm.sk[w & 1][wave][4 * r]);
        const v4i acc = *reinterpret_cast<const v4i *>(&sm.s[wave][4 * r]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float x = (ACC_START_F - __int_as_float(acc[e])) * skv[e];
            if (e >= left) x = INFINITY;
            a[e] = x;
            bmin = fminf(bmin, x);
        }
        bmin = half_min(bmin);
        }
        if (lane == 0) sm.ext[wave] = bmin;
        __syncthreads();
        // lines 10, 11 and the row sums of 12
        const float x = sm.ext[lane & 15];
        float upto = x;                                          // extremum over the blocks up to this one
        for_each_int([&](auto i) {
            constexpr int n = 1 << decltype(i)::value;
            upto = fminf(upto, __uint_as_float(dpp<ROW_SHR | n>(0x7f800000u, __float_as_uint(upto))));
        }, std::make_integer_sequence<int, 4>{});
        const float m_old = wave ? fmaxf(carry, lane_value(upto, wave - 1) * nq2) : carry, m = fmaxf(m_old, lane_value(x, wave) * nq2), mm = m - LOG2_R_NORM;
        carry = fmaxf(carry, lane_value(upto, 15) * nq2);
        if (mine) {
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(a[e], nq2, -mm));
        const uint32_t p = pack_p4(y);
        pbytes[r] = static_cast<int>(p);
        const unsigned sum = parity_sum(__builtin_amdgcn_sad_u8(p, 0u, 0u));
        if (lane < 2) sm.psum[wave][lane] = static_cast<float>(sum);
        if (lane == 0) sm.alpha[wave] = __builtin_amdgcn_exp2f(m_old - m);
        // line 13, P V of the block
        v4i pacc[2];
        for_each_int([&](auto e_) {
            constexpr int e = decltype(e_)::value, N64 = DS / 2; // runs of 64 keys in an entry
            v4i vop[N64][2], pf[N64];
            advance(std::integral_constant<int, 4 + e>{}, [&](lds_ptr vs) {
#pragma unroll
                for (int t = 0; t < N64; ++t) {
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt) {
                        const lds_ptr va = vs + v0 + 64 * t * DV + 16 * dt;
                        const v2i t0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(va));
                        const v2i t1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(va + 8 * DV));
                        vop[t][dt] = v4i{t0[0], t0[1], t1[0], t1[1]};
                    }
                    pf[t] = *reinterpret_cast<const v4i *>(&pbytes[16 * (e * N64 + t) + 4 * G]);
                }
            });
#pragma unroll
            for (int t = 0; t < N64; ++t)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) pacc[dt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vop[t][dt], pf[t], e + t == 0 ? acc0 : pacc[dt], 0, 0, 0);
        }, std::make_integer_sequence<int, VE>{});
        if (c == 0) {
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) {
                v4f t;
#pragma unroll
                for (int i = 0; i < 4; ++i) t[i] = ACC_START_F - __int_as_float(pacc[dt][i]);
                *reinterpret_cast<v4f *>(&sm.pv[wave][16 * dt + 4 * G]) = t;
            }
        }
        }
        __syncthreads();
        // lines 12, 13: the blocks of the window in order
        if (tid < DV) {
            float t[DEC_WAVES], al[DEC_WAVES], ps[DEC_WAVES][2];
#pragma unroll
            for (int b = 0; b < DEC_WAVES; ++b) { t[b] = sm.pv[b][tid]; al[b] = sm.alpha[b]; ps[b][0] = sm.psum[b][0]; ps[b][1] = sm.psum[b][1]; }
#pragma unroll
            for (int b = 0; b < DEC_WAVES; ++b) {
                const int jb = w * DEC_WAVES + b;
                if (jb < T_c) {
                    float alpha_o = al[b];
                    if (vblock) {                                // one V scale per key block: the running output is kept in units of the current block's
                        const float sv_j = sVh[jb];
                        alpha_o = al[b] * (sv_prev * __builtin_amdgcn_rcpf(sv_j));
                        sv_prev = sv_j;
                    }
                    l0 = __builtin_fmaf(l0, al[b], ps[b][0]);
                    l1 = __builtin_fmaf(l1, al[b], ps[b][1]);
                    o = __builtin_fmaf(o, alpha_o, -t[b]);
                }
            }
        }
    }
    wait_all_memory();                                           // requests past the last window: nothing of mine stays in flight

    // lines 15-17
    if (tid < DV) {
        const float f = (vblock ? sv_prev : sVh[0]) * ACC_UNIT / (l0 + l1);
        float y = o * f;
        asm volatile("" : "+v"(y));                              // the fp32 product, rounded once more below
        const long at = static_cast<long>(head) * D + col0 + tid;
        if (o_dtype == IFA_F32) static_cast<float *>(O)[at] = y;
        else if (o_dtype == IFA_F16) static_cast<uint16_t *>(O)[at] = static_cast<uint16_t>(Pack4<__half>::pack(y, 0.0f, 0.0f, 0.0f).x & 0xffffu);
        else static_cast<uint16_t *>(O)[at] = static_cast<uint16_t>(Pack4<__hip_bfloat16>::pack(y, 0.0f, 0.0f, 0.0f).x & 0xffffu);
    }
#endif
}

// ---- two to eight queries per head (a few draft tokens) ------------------------------------------------------------
// The decode kernel with the queries in the columns of its products: a lane (c, G) holds the scores of query c for 32 of the block's keys, and P in the order in which
// the second product takes it, so neither goes through LDS.  A window takes 5.3 - 6 us (the decode kernel's 5), half of it vector issue; per-block V scales add .4 - 1.4 us a call.  Few-query kernel / this
// one, us: 32 heads x 5 queries x 4900 keys 23.9 / 19.1, 8 x 8 x 2048 10.8 / 8.1, 32 x 8 x 16384 75 / 51; d = 64, 64 x 8 x 4900 20.3 / 15.2, 32 x 2 x 16384 56 / 37.
constexpr int DRAFT_MAX_Q = 8;
template <int D, int DS> struct SmemDraft {
    using P = DecodePlan<D, DS, D == 128 ? 2 : 3>;
    alignas(4096) int8_t ring[DEC_WAVES][P::R][32 * D];
    alignas(256) float sk[DEC_WAVES][BC];
    alignas(16) float pv[DEC_WAVES][DRAFT_MAX_Q][P::DV];         // minus P V, units of 2^26
    alignas(16) float ext[DEC_WAVES][16];                        // extremum of a per block and query (line 10)
    alignas(16) float alpha[DRAFT_MAX_Q][DEC_WAVES];             // e^(m_old - m)
    alignas(16) float psum[DRAFT_MAX_Q][DEC_WAVES][2];           // the row sums over either half of the keys
};
// (the s_K of the next window are asked for with the first entry of V at the earliest, when those of this one have been used)
static_assert(sizeof(SmemDraft<128, 4>) <= 160 * 1024 && SmemDraft<128, 4>::P::EPW - SmemDraft<128, 4>::P::R + 1 >= 4 && SmemDraft<64, 2>::P::EPW - SmemDraft<64, 2>::P::R + 1 >= 4, "LDS, ring");

template <int D, int DS>
__global__ __launch_bounds__(DEC_THREADS, 4) void int_flash_attn_fwd_draft_kernel(
    const int8_t *__restrict__ Q, const int8_t *__restrict__ K, const int8_t *__restrict__ V,
    const float *__restrict__ sQ, const float *__restrict__ sK, const float *__restrict__ sV,
    int heads, int Nq, int Nk, int causal, int vblock, int o_dtype, void *__restrict__ O) {
#if defined(__HIP_DEVICE_COMPILE__)
    using P = typename SmemDraft<D, DS>::P;
    __shared__ SmemDraft<D, DS> sm;
    constexpr int KS = D / 32, KK = D / 64, DV = P::DV, VE = P::VE, EPW = P::EPW, R = P::R, NQ = DRAFT_MAX_Q;
    static_assert(DV == 32, "two d tiles of 16");

    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, G = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T_c = (Nk + BC - 1) / BC, windows = (T_c + DEC_WAVES - 1) / DEC_WAVES;
    int head, qg, part;
    if (!map_query_group<DS>(blockIdx.x, heads, 1, head, qg, part)) return;
    const int col0 = part * DV;                                  // first column of V and O

    const BufRsrc rK = make_rsrc(K + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const BufRsrc rV = make_rsrc(V + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const BufRsrc rSK = make_rsrc(sK + static_cast<long>(head) * Nk, static_cast<unsigned>(Nk) * 4);
    const LaneOffsets<D> lo(lane, 0);
    const lds_ptr ring = (lds_ptr)(&sm.ring[wave][0][0]), skbuf = (lds_ptr)(&sm.sk[wave][0]);
    const unsigned gv = (lane / (DV / 16)) * D + col0 + 16 * (lane % (DV / 16));
    const int turn = part * (4 / DS);                            // which of its key tiles a wavefront begins with: step k is tile (k + turn) % 4 throughout
    int in = 0, slot = 0;
    auto issue = [&](auto k_, int w) {
        constexpr int k = decltype(k_)::value % EPW;
        const int key0 = (w * DEC_WAVES + wave) * BC;            // first key of this wavefront's block
        const lds_ptr dst = ring + in * (32 * D);
        in = in + 1 == R ? 0 : in + 1;
        if constexpr (k < 4) {
            const int key = key0 + 32 * ((k + turn) & 3), off = key < Nk ? key * D : NOWHERE;
            if constexpr (D == 128) {                            // (a run: 6 heads x 3 queries x 19608 keys 59.7 us, 58.1 piece by piece; d = 64 39.1 and 39.4)
#pragma unroll
                for (int i = 0; i < KS; ++i) lds_copy16_piece<KS>(i, rK, dst, lo.gk, lo.gk, off);
            } else lds_copy16_run<KS>(rK, dst, lo.gk, lo.gk, off);
            if constexpr (k == 0) {
#pragma unroll
                for (int i = 0; i < 2; ++i) lds_copy4(rSK, skbuf + 256 * i, 4 * lane, key0 + 64 * i < Nk ? (key0 + 64 * i) * 4 : NOWHERE);
            }
        } else {                                                 // (d = 64: the half of the block that the steps began with first)
            const int key = key0 + (VE == 2 ? (32 * DS * (k - 4) + 32 * turn) & (BC - 1) : 0), off = key < Nk ? key * D : NOWHERE;
#pragma unroll
            for (int i = 0; i < KS; ++i) lds_copy16(rV, dst + 1024 * i, gv, off + i * (1024 / DV) * D);
        }
    };
    for_each_int([&](auto k) { issue(k, 0); }, std::make_integer_sequence<int, R - 1>{});

    // line 5: column c is query c (past the last one: a copy of it, never stored)
    const int q = min(c, Nq - 1);
    const int8_t *qptr = Q + (static_cast<long>(head) * Nq + q) * D + 16 * G;
    v4i qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const v4i *>(qptr + 64 * kk);
    float nq2 = sQ[static_cast<long>(head) * Nq + q] * (-LOG2E * ACC_UNIT);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(qf[kk]));
    asm volatile("" : "+v"(nq2));
    const int first_limit = causal ? Nk - Nq : Nk - 1, klimit = causal ? q + Nk - Nq : Nk - 1;   // last key that the first query, that this one sees
    const v4i acc0 = {ACC_START_I, ACC_START_I, ACC_START_I, ACC_START_I};
    const unsigned k0 = c * D + 16 * (G ^ k_swz<D>(c));
    // transposing read of V, keys 4 G .. 4 G + 3 and 16 + 4 G .. of a key tile: the order in which a lane holds P
    const unsigned v0 = (16 * (c >> 3) + 4 * G + ((c >> 1) & 3)) * DV + 8 * (c & 1);

    const float *sVh = vblock ? sV + static_cast<long>(head) * T_c : sV + head;
    float carry = -INFINITY;                                     // m in front of the window (line 6)
    float o = 0.0f, l0 = 0.0f, l1 = 0.0f, sv_prev = 1.0f;        // of query tid / DV and column tid % DV
    const int fq = tid / DV, fc = tid % DV;

    for (int w = 0; w < windows; ++w) {
        const bool mine = w * DEC_WAVES + wave < T_c;            // (wave-uniform)
        auto advance = [&](auto k_, auto take) {
            constexpr int k = decltype(k_)::value;
            wait_vmcnt<P::behind(k)>();
            __builtin_amdgcn_sched_barrier(0);
            issue(std::integral_constant<int, k + R - 1>{}, w + (k + R - 1) / EPW);
            __builtin_amdgcn_sched_barrier(0);
            take(ring + slot * (32 * D));
            slot = slot + 1 == R ? 0 : slot + 1;
        };
        v4i sacc[4][2];
        float a[4][2][4], bmin = INFINITY;
        if (mine) {
            // line 9, integer part
            for_each_int([&](auto k_) {
                constexpr int k = decltype(k_)::value;
                v4i kop[2][KK];
                advance(k_, [&](lds_ptr ks) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int kk = 0; kk < KK; ++kk) kop[h][kk] = *reinterpret_cast<LDS_AS const v4i *>(lds_xor(ks, 64 * kk, k0) + 16 * D * h);
                });
#pragma unroll
                for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                    for (int h = 0; h < 2; ++h) sacc[k][h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(kop[h][kk], qf[kk], kk == 0 ? acc0 : sacc[k][h], 0, 0, 0);
            }, std::make_integer_sequence<int, 4>{});
            // line 9, fp32 part, and the extremum of the block
            const int key0 = (w * DEC_WAVES + wave) * BC;
            const bool masked = key0 + BC - 1 > min(first_limit, Nk - 1);                        // (wave-uniform)
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int at = 32 * ((k + turn) & 3) + 16 * h + 4 * G;                       // first of four keys, in the block
                    const v4f skv = *reinterpret_cast<const v4f *>(&sm.sk[wave][at]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float x = (ACC_START_F - __int_as_float(sacc[k][h][e])) * skv[e];
                        if (masked && key0 + at + e > klimit) x = INFINITY;
                        a[k][h][e] = x;
                        bmin = fminf(bmin, x);
                    }
                    if (h) __builtin_amdgcn_sched_barrier(0);
                }
            const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(bmin), __float_as_uint(bmin), false, false);
            bmin = pair_min(fminf(__uint_as_float(sw[0]), __uint_as_float(sw[1])));
        }
        if (G == 0) sm.ext[wave][c] = bmin;
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        // lines 10, 11 and the row sums of 12
        float before = INFINITY, total = INFINITY;               // over the blocks of the window in front of this wavefront's; over all
#pragma unroll
        for (int b = 0; b < DEC_WAVES; ++b) {
            if (b == wave) before = total;
            total = fminf(total, sm.ext[b][c]);
        }
        const float m_old = fmaxf(carry, before * nq2), m = fmaxf(m_old, bmin * nq2), mm = m - LOG2_R_NORM;
        carry = fmaxf(carry, total * nq2);
        __builtin_amdgcn_sched_barrier(0);
        if (mine) {
            v4i pf[2];                                           // two runs of 64 keys: steps 0 and 1, 2 and 3
            unsigned sum = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float y[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(a[k][h][e], nq2, -mm));
                    const uint32_t p = pack_p4(y);
                    sum = __builtin_amdgcn_sad_u8(p, 0u, sum);
                    pf[k >> 1][2 * (k & 1) + h] = static_cast<int>(p);
                }
            const auto sw = __builtin_amdgcn_permlane32_swap(sum, sum, false, false);            // lanes G and G + 2 hold the same half of the keys
            if (c < NQ && G < 2) sm.psum[c][wave][G] = static_cast<float>(sw[0] + sw[1]);
            if (c < NQ && G == 0) sm.alpha[c][wave] = __builtin_amdgcn_exp2f(m_old - m);
            // line 13, P V of the block
            v4i pacc[2];
            for_each_int([&](auto e_) {
                constexpr int e = decltype(e_)::value, N64 = DS / 2;                             // runs in an entry
                v4i vop[N64][2];
                advance(std::integral_constant<int, 4 + e>{}, [&](lds_ptr vs) {
#pragma unroll
                    for (int t = 0; t < N64; ++t)
#pragma unroll
                        for (int dt = 0; dt < 2; ++dt) {
                            // the run's two key tiles (d = 64: the entry holds them in order)
                            const int ta = VE == 2 ? 0 : (2 * t + turn) & 3, tb = VE == 2 ? 1 : (2 * t + 1 + turn) & 3;
                            const v2i t0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(vs + v0 + 32 * ta * DV + 16 * dt));
                            const v2i t1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(vs + v0 + 32 * tb * DV + 16 * dt));
                            vop[t][dt] = v4i{t0[0], t0[1], t1[0], t1[1]};
                        }
                });
#pragma unroll
                for (int t = 0; t < N64; ++t)
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt)
                        pacc[dt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vop[t][dt], pf[e * N64 + t], e + t == 0 ? acc0 : pacc[dt], 0, 0, 0);
            }, std::make_integer_sequence<int, VE>{});
            if (c < NQ) {
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) {
                    v4f t;
#pragma unroll
                    for (int i = 0; i < 4; ++i) t[i] = ACC_START_F - __int_as_float(pacc[dt][i]);
                    *reinterpret_cast<v4f *>(&sm.pv[wave][c][16 * dt + 4 * G]) = t;
                }
            }
        }
        __syncthreads();
        // lines 12, 13: the blocks of the window in order
        if (tid < NQ * DV) {
#pragma unroll
            for (int b0 = 0; b0 < DEC_WAVES; b0 += 8) {
                float t[8], al[8], ps[8][2];
#pragma unroll
                for (int b = 0; b < 8; ++b) { t[b] = sm.pv[b0 + b][fq][fc]; al[b] = sm.alpha[fq][b0 + b]; ps[b][0] = sm.psum[fq][b0 + b][0]; ps[b][1] = sm.psum[fq][b0 + b][1]; }
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const int jb = w * DEC_WAVES + b0 + b;
                    if (jb < T_c) {
                        float alpha_o = al[b];
                        if (vblock) {                            // one V scale per key block: the running output is kept in units of the current block's
                            const float sv_j = sVh[jb];
                            alpha_o = al[b] * (sv_prev * __builtin_amdgcn_rcpf(sv_j));
                            sv_prev = sv_j;
                        }
                        l0 = __builtin_fmaf(l0, al[b], ps[b][0]);
                        l1 = __builtin_fmaf(l1, al[b], ps[b][1]);
                        o = __builtin_fmaf(o, alpha_o, -t[b]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    wait_all_memory();                                           // requests past the last window: nothing of mine stays in flight

    // lines 15-17
    if (tid < NQ * DV && fq < Nq) {
        const float f = (vblock ? sv_prev : sVh[0]) * ACC_UNIT / (l0 + l1);
        float y = o * f;
        asm volatile("" : "+v"(y));                              // the fp32 product, rounded once more below
        const long at = (static_cast<long>(head) * Nq + fq) * D + col0 + fc;
        if (o_dtype == IFA_F32) static_cast<float *>(O)[at] = y;
        else if (o_dtype == IFA_F16) static_cast<uint16_t *>(O)[at] = static_cast<uint16_t>(Pack4<__half>::pack(y, 0.0f, 0.0f, 0.0f).x & 0xffffu);
        else static_cast<uint16_t *>(O)[at] = static_cast<uint16_t>(Pack4<__hip_bfloat16>::pack(y, 0.0f, 0.0f, 0.0f).x & 0xffffu);
    }
#endif
}

// ---- few queries, many keys, any number of heads: the key axis split across workgroups, exactly ----------------
// The narrow kernel cannot fill the chip when there are few heads, and walks a long key sequence at what one or two CUs take
// in.  Splitting the keys of a head over workgroups is not Algorithm 1 as
// long as each part rounds P on the grid of ITS OWN running maximum; it is Algorithm 1 once the maximum after every
// key block is known before any P is formed.  With at most SPLIT_MAX_Q queries per head the scores are small next to
// K and V (4 N_q bytes per key against 2 d), so they go through memory:
//   pass 1 (splitk_scores_kernel)  streams K, computes line 9 exactly as the other kernels do (same MFMA chain, same
//           scaling) and writes the scaled scores a, the minimum of every (32-key tile, query) -- the maxima of line 10
//           -- and the minimum of every (run of blocks, query);
//   pass 2 (splitk_pv_kernel)      streams V and the scores; the running maximum in front of a workgroup's first block
//           is the extremum over all earlier runs (max is exact and order-independent), so lines 10-13 give, block by
//           block, the same m, the same P bytes and the same int32 P V as the sequential walk; what a workgroup leaves
//           is the walk over its run of blocks started from O = 0, l = 0: a partial (m, l, O);
//   pass 3 (splitk_combine_kernel) O = sum over the runs of 2^(m_run - m_last) O_run, l likewise, then lines 15-17.
// P is bit-identical to the sequential kernels'; O and l differ from theirs only in the order of the fp32 additions
// (the sequential walk multiplies by e^{m_old - m} block after block, this one once per partial).
// In both streaming passes a workgroup takes a run of `cb` key blocks of one head and its wavefront w takes key tile w
// (keys 32w .. 32w + 31) of each of them: the rows of K, V, s_K and of the scores that a wavefront stages into LDS
// are exactly the rows it consumes itself, so the wavefronts of a workgroup never wait for one another -- no barrier
// in the loops; a wavefront's ring of staged blocks is ordered by its own counted s_waitcnt alone.  The four
// wavefronts meet once, after their loops: their minima (pass 1) and their partial (l, O) at the common m (pass 2)
// are combined through LDS.
constexpr int SPLIT_MAX_Q = 8;       // queries per head up to which the scores go through memory (a decode step, a few speculative tokens)
constexpr int SPLIT_MAX_Q_RECOMPUTE = 32;   // ... and up to which the second pass recomputes them from K instead (one column tile)
constexpr int SPLIT_NSTAGE_K = 4;    // pass 1: ring of K blocks, filled three ahead
constexpr int SPLIT_NSTAGE_V = 3;    // pass 2: ring of V blocks, filled two ahead
constexpr int SPLIT_LONG_RUN = 9;    // pass 2 with K, d = 64: blocks of a run from which the ring holds three blocks of K and V instead of two
[[maybe_unused]] constexpr bool SPLIT_NT = true;      // staging copies carry the non-temporal hint: every byte is read once (measured +7 % at 537 MB of K and V)

template <int D> struct SmemSplitK {
    alignas(4096) int8_t k[SPLIT_NSTAGE_K][BC * D];
    alignas(256) float sk[SPLIT_NSTAGE_K][4][64];             // per wavefront: the 32 s_K of its key tile (+ 32 unused)
    alignas(16) float red[4][SPLIT_MAX_Q_RECOMPUTE];
};
template <int D> struct SmemSplitV {
    alignas(4096) int8_t v[SPLIT_NSTAGE_V][BC * D];
    alignas(1024) float a[SPLIT_NSTAGE_V][4][SPLIT_MAX_Q][32];   // per wavefront: the scores of its key tile, query-major
    alignas(256) float tmin[SPLIT_NSTAGE_V][4][64];             // per wavefront: the block's [query][tile] minima (+ 32 unused)
    alignas(16) float red[4][SPLIT_MAX_Q];
    alignas(16) float pre[SPLIT_MAX_Q];
};
static_assert(2 * sizeof(SmemSplitK<128>) <= 160 * 1024 && 2 * sizeof(SmemSplitV<128>) <= 160 * 1024, "two workgroups per CU");
static_assert(offsetof(SmemSplitV<64>, v) % 4096 == 0 && (BC * 64) % 4096 == 0, "tile bases");

// Second pass for 9 .. 32 queries per head: the scores would be as many bytes as K and V, so they are not stored;
// the pass streams K once more and recomputes line 9 (same MFMA chain, same scaling: the same numbers).  A key tile is one chain from
// its scores to its share of O, so what a CU gets done is the wavefronts it holds: at d = 128 a ring of NS = 2 blocks, filled one ahead, leaves
// room for two workgroups (64 KB of copies in flight either way; with a ring of three, one per CU, half of a call's 512 workgroups
// waited for the other half).  Whole call, us, ring of three / two: 32 heads x 16 queries x 8192 keys 32.1 / 27.6, 60 x 16 x 8192 59 / 49, 32 x 32 x 32768
// 100 / 90, 8 x 16 x 16384 20.1 / 19.2.  At d = 64 two workgroups share a CU with either ring.  The smaller one starts sooner, the larger one
// has more in flight: runs of 4 blocks 24 x 9 x 16384 24.0 / 20.6, 32 x 16 x 8192 18.5 / 17.7, of 8 even (64 x 16 x 16384 45.3 / 45.4), of 13 24 x 9 x 65536 62.6 / 64.8, of
// 25 48 x 16 x 65536 120 / 128.
template <int D, int NS> struct SmemSplitKV {
    alignas(4096) int8_t k[NS][BC * D];
    alignas(4096) int8_t v[NS][BC * D];
    alignas(256) float sk[NS][4][64];
    alignas(1024) float tmin[NS][4][256];                       // per wavefront: the block's [query][tile] minima (512 B, + 512 unused)
    alignas(16) float pre[SPLIT_MAX_Q_RECOMPUTE];
};
static_assert(2 * sizeof(SmemSplitKV<128, 2>) <= 160 * 1024 && 2 * sizeof(SmemSplitKV<64, 3>) <= 160 * 1024, "two workgroups per CU");

// Layout of the workspace (fp32 words), shared by the host code and the kernels (MAXQ = 8 or 32, by Nq):
//   scores  [heads, T_c, 4 tiles, Nq, 32]     a of line 9 (masked keys: +inf); Nq <= 8 only
//   tmin    [heads, T_c, MAXQ, 4]             minimum of a per (block, query, tile); queries >= Nq unused
//   cmin    [heads, MAXQ, nchunks]            minimum of a per (run of blocks, query)
//   part_o  [heads, parts, Nq, d]             one partial per run of blocks
//   part_ml [heads, parts, Nq, 2]             m (log2 units) and l of the partial
struct SplitPlan {
    int cb, nchunks, T_c, maxq, parts;
    bool store;
    long off_tmin, off_cmin, off_part_o, off_part_ml, words;
};
inline SplitPlan split_plan(long heads, int Nq, int Nk, int d) {
    SplitPlan p;
    p.T_c = (Nk + BC - 1) / BC;
    p.store = Nq <= SPLIT_MAX_Q;
    p.maxq = p.store ? SPLIT_MAX_Q : SPLIT_MAX_Q_RECOMPUTE;
    long want = 1024 / heads;                    // about four workgroups per CU over the chip
    if (want < 1) want = 1;
    long cb = (p.T_c + want - 1) / want;
    const long cb_min = p.store ? 2 : 4;         // a run's partial (Nq x d floats) must stay small next to its K and V
    if (cb < cb_min) cb = cb_min;
    if (cb > p.T_c) cb = p.T_c;
    p.cb = static_cast<int>(cb);
    p.nchunks = (p.T_c + p.cb - 1) / p.cb;       // no run is empty
    p.parts = p.nchunks;
    auto up = [](long w) { return (w + 63) & ~63L; };            // 256-byte granules
    p.off_tmin = p.store ? up(heads * p.T_c * 4 * Nq * 32) : 0;
    p.off_cmin = p.off_tmin + up(heads * p.T_c * p.maxq * 4);
    p.off_part_o = p.off_cmin + up(heads * p.maxq * p.nchunks);
    p.off_part_ml = p.off_part_o + up(heads * p.parts * Nq * d);
    p.words = p.off_part_ml + up(heads * p.parts * Nq * 2);
    return p;
}

template <int D, bool CAUSAL, int MAXQ, bool STORE>
__global__ __launch_bounds__(THREADS, 2) void splitk_scores_kernel(
    const int8_t *__restrict__ Q, const int8_t *__restrict__ K, const float *__restrict__ sK, int Nq, int Nk, int cb,
    int nchunks, float *__restrict__ scores, float *__restrict__ tminG, float *__restrict__ cminG) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ SmemSplitK<D> sm;
    constexpr int KS = D / 32;
    constexpr int PER_BLOCK = KS + 1;                            // copy instructions per wavefront and block
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T_c = (Nk + BC - 1) / BC;
    const int head = blockIdx.x / nchunks, c = blockIdx.x % nchunks;
    const int jb0 = c * cb, jb1 = min(T_c, jb0 + cb);            // this workgroup's key blocks
    const int shift = CAUSAL ? Nk - Nq : 0;
    const int rq = min(r, Nq - 1);                               // columns past Nq: a copy of the last query, never stored

    const BufRsrc rK = make_rsrc(K + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const BufRsrc rSK = make_rsrc(sK + static_cast<long>(head) * Nk, static_cast<unsigned>(Nk) * 4);
    const lds_ptr kbuf = (lds_ptr)(&sm.k[0][0]);
    const lds_ptr skbuf = (lds_ptr)(&sm.sk[0][0][0]);
    const LaneOffsets<D> lo(lane, wave);
    // Line 8 for this wavefront's key tile of block jb (rows 32 wave .. + 31 of K_j: the pieces prefetch_k gives
    // this wavefront; its 32 s_K, lanes 32-63 repeating lanes 0-31) into stage (jb - jb0) % NSTAGE.  A block past the
    // run is requested nowhere, so that every block costs PER_BLOCK copy instructions and the counted waits stay valid.
    auto stage_block = [&](int jb) {
        const int st = (jb - jb0) % SPLIT_NSTAGE_K;
        const bool real = jb < jb1;
        const Prefetch pf = {rK, rK, rSK, real ? jb * BC * D : NOWHERE, real ? jb * BC * 4 : NOWHERE,
                             kbuf + st * BC * D, kbuf, skbuf + (st * 4 + wave) * 256};
        prefetch_k<D, SPLIT_NT>(pf, lo, wave);
        lds_copy4(pf.sk, pf.lsk, 4 * r + 128 * wave, pf.skoff);
    };
    stage_block(jb0);
    stage_block(jb0 + 1);
    stage_block(jb0 + 2);

    const int8_t *qptr = Q + (static_cast<long>(head) * Nq + rq) * D + 16 * g;
    v4i qf[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = *reinterpret_cast<const v4i *>(qptr + 32 * kk);
    // landed BEFORE the loop as far as the compiler is concerned: a wait of its own inside the loop would be a wait for
    // every outstanding vector-memory operation, the staged copies included
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(qf[kk]));
    v16i acc0;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc0[v] = ACC_START_I;
    float wmin = INFINITY;                                       // minimum over this wavefront's tiles of the whole run

    for (int jb = jb0; jb < jb1; ++jb) {
        const int st = (jb - jb0) % SPLIT_NSTAGE_K, j0 = jb * BC;
        // The counter retires in order.  Younger than the copies of block jb are those of blocks jb + 1 and jb + 2 and
        // the stores of earlier iterations: allowing 2 PER_BLOCK operations in flight means block jb has landed,
        // however many stores there are among them.
        wait_vmcnt<2 * PER_BLOCK>();
        stage_block(jb + 3);                                     // into the stage of block jb - 1, which this wavefront has left
        const lds_ptr ks = kbuf + st * BC * D;
        v4i kop[KS];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) kop[kk] = *reinterpret_cast<LDS_AS const v4i *>(k_operand<D>(ks, lo, kk) + 32 * wave * D);
        v4f skv[4];
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) skv[vq] = *reinterpret_cast<LDS_AS const v4f *>(skbuf + (st * 4 + wave) * 256 + lo.sk + 32 * vq);
        v16i sacc = acc0;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) sacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kop[kk], qf[kk], sacc, 0, 0, 0);
        // kept keys: index inside the block <= klimit (the causal diagonal, the ragged end of the sequence)
        const int tail = Nk - 1 - j0;
        const int klimit = CAUSAL ? min(rq + shift - j0, tail) : tail;
        const bool masked = CAUSAL ? (j0 + BC - 1 > min(shift, Nk - 1)) : (tail < BC - 1);   // wave-uniform
        float a[16], tmin = INFINITY;
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float x = (ACC_START_F - __int_as_float(sacc[4 * vq + e])) * skv[vq][e];
                if (masked && (32 * wave + 8 * vq + 4 * g + e > klimit)) x = INFINITY;
                a[4 * vq + e] = x;
                tmin = fminf(tmin, x);
            }
        tmin = pair_min(tmin);
        wmin = fminf(wmin, tmin);
        if (r < Nq) {
            if (STORE) {
                float *dst = scores + (((static_cast<long>(head) * T_c + jb) * 4 + wave) * Nq + r) * 32 + 4 * g;
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) *reinterpret_cast<v4f *>(dst + 8 * vq) = v4f{a[4 * vq], a[4 * vq + 1], a[4 * vq + 2], a[4 * vq + 3]};
            }
            if (g == 0) tminG[((static_cast<long>(head) * T_c + jb) * MAXQ + r) * 4 + wave] = tmin;
        }
    }
    wait_all_memory();                                           // requests past the run: nothing of mine stays in flight
    // the run's minimum per query, for the prefix the second pass needs: the only exchange between the wavefronts
    if (g == 0 && r < MAXQ) sm.red[wave][r] = wmin;
    __syncthreads();
    if (wave == 0 && g == 0 && r < Nq)
        cminG[(static_cast<long>(head) * MAXQ + r) * nchunks + c] = fminf(fminf(sm.red[0][r], sm.red[1][r]), fminf(sm.red[2][r], sm.red[3][r]));
#endif
}

template <int D>
__global__ __launch_bounds__(THREADS, 2) void splitk_pv_kernel(
    const int8_t *__restrict__ V, const float *__restrict__ sQ, int Nq, int Nk, int cb, int nchunks,
    const float *__restrict__ scores, const float *__restrict__ tminG, const float *__restrict__ cminG, float *__restrict__ part_o,
    float *__restrict__ part_ml) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ SmemSplitV<D> sm;
    constexpr int DT = D / 32;
    constexpr int PER_BLOCK = DT + 2;
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T_c = (Nk + BC - 1) / BC;
    const int head = blockIdx.x / nchunks, c = blockIdx.x % nchunks;
    const int jb0 = c * cb, jb1 = min(T_c, jb0 + cb);
    const int rq = min(r, Nq - 1);

    const BufRsrc rV = make_rsrc(V + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const BufRsrc rA = make_rsrc(scores + static_cast<long>(head) * T_c * 4 * Nq * 32, static_cast<unsigned>(T_c) * 4 * Nq * 32 * 4);
    const BufRsrc rT = make_rsrc(tminG + static_cast<long>(head) * T_c * SPLIT_MAX_Q * 4, static_cast<unsigned>(T_c) * SPLIT_MAX_Q * 4 * 4);
    const lds_ptr vbuf = (lds_ptr)(&sm.v[0][0]);
    const lds_ptr abuf = (lds_ptr)(&sm.a[0][0][0][0]);
    const lds_ptr tbuf = (lds_ptr)(&sm.tmin[0][0][0]);
    const LaneOffsets<D> lo(lane, wave);
    // This wavefront's key tile of V_j (the rows prefetch_v gives it), the scores of that tile (Nq x 32 floats,
    // contiguous; the copy moves 1 KB, whatever follows the record is not read) and the block's 32 tile minima.
    auto stage_block = [&](int jb) {
        const int st = (jb - jb0) % SPLIT_NSTAGE_V;
        const bool real = jb < jb1;
        const Prefetch pf = {rV, rV, rV, real ? jb * BC * D : NOWHERE, NOWHERE, vbuf, vbuf + st * BC * D, vbuf};
        prefetch_v<D, SPLIT_NT>(pf, lo, wave);
        lds_copy16(rA, abuf + (st * 4 + wave) * 1024, 16 * lane, real ? (jb * 4 + wave) * Nq * 128 : NOWHERE);
        lds_copy4(rT, tbuf + (st * 4 + wave) * 256, 4 * r, real ? jb * (SPLIT_MAX_Q * 4 * 4) : NOWHERE);
    };
    stage_block(jb0);
    stage_block(jb0 + 1);

    float nq2 = sQ[static_cast<long>(head) * Nq + rq] * (-LOG2E * ACC_UNIT);
    // Minimum of a over every block in front of this workgroup's first one: over the runs in front of this one.
    // 32 threads per query (wavefront w: queries 2w and 2w + 1).
    float pre = INFINITY;
    {
        const int q = tid >> 5;
        if (q < Nq)
            for (int cc = tid & 31; cc < c; cc += 32) pre = fminf(pre, cminG[(static_cast<long>(head) * SPLIT_MAX_Q + q) * nchunks + cc]);
#pragma unroll
        for (int s_ = 16; s_ >= 1; s_ >>= 1) pre = fminf(pre, __shfl_xor(pre, s_));
        if ((tid & 31) == 0) sm.pre[q] = pre;
    }
    asm volatile("" : "+v"(nq2));                                // as for Q above: no wait of the compiler's own inside the loop
    __syncthreads();
    pre = sm.pre[rq];
    float m2 = (pre == INFINITY) ? -INFINITY : pre * nq2;        // line 10 over all earlier blocks (no block: line 6)
    float l = 0.0f, o[DT][16];
    v16i acc0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        acc0[v] = ACC_START_I;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt][v] = 0.0f;
    }

    for (int jb = jb0; jb < jb1; ++jb) {
        const int st = (jb - jb0) % SPLIT_NSTAGE_V;
        wait_vmcnt<PER_BLOCK>();                                 // block jb has landed (block jb + 1 may be in flight)
        stage_block(jb + 2);                                     // into the stage of block jb - 1, which this wavefront has left
        const lds_ptr vs = vbuf + st * BC * D;
        // line 10 for the whole block: the four tile minima of this lane's query
        const v4f t4 = *reinterpret_cast<LDS_AS const v4f *>(tbuf + (st * 4 + wave) * 256 + rq * 16);
        const float bmin = fminf(fminf(t4[0], t4[1]), fminf(t4[2], t4[3]));
        const float m_new = fmaxf(m2, bmin * nq2);
        const float alpha = __builtin_amdgcn_exp2f(m2 - m_new);
        const float mm = m_new - LOG2_R_NORM;
        m2 = m_new;
        // line 11 for key tile `wave`
        v4i pw;
        uint32_t psum = 0;
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            const v4f av = *reinterpret_cast<LDS_AS const v4f *>(abuf + (st * 4 + wave) * 1024 + rq * 128 + (8 * vq + 4 * g) * 4);
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(av[e], nq2, -mm));
            const uint32_t w = pack_p4(x);
            psum = __builtin_amdgcn_sad_u8(w, 0u, psum);
            pw[vq] = static_cast<int>(w);
        }
        l = __builtin_fmaf(l, alpha, static_cast<float>(psum));  // line 12 over this lane's keys of this tile
        // line 13 over the keys of this tile, all d tiles
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const v2i t0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<D>(vs, lo, dt) + 32 * wave * D));
            const v2i t1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<D>(vs, lo, dt) + 16 * D + 32 * wave * D));
            const v4i vop = {t0[0], t0[1], t1[0], t1[1]};
            const v16i pacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(vop, pw, acc0, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) o[dt][v] = __builtin_fmaf(o[dt][v], alpha, -(ACC_START_F - __int_as_float(pacc[v])));
        }
    }
    wait_all_memory();
    // The four wavefronts hold partials of the same run of blocks at the same m: their sum is the workgroup's partial.
    // The V ring is free once every wavefront has left the loop; [wavefront][query][d] floats go through it.
    const float lt = l + swap32(l);
    __syncthreads();
    float *xo = reinterpret_cast<float *>(&sm.v[0][0]);          // 4 * 8 * D floats <= 16 KB
    if (r < Nq) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq)
                *reinterpret_cast<v4f *>(xo + (wave * SPLIT_MAX_Q + r) * D + 32 * dt + 8 * vq + 4 * g) = v4f{o[dt][4 * vq], o[dt][4 * vq + 1], o[dt][4 * vq + 2], o[dt][4 * vq + 3]};
        if (g == 0) sm.red[wave][r] = lt;
    }
    __syncthreads();
    const long slot0 = (static_cast<long>(head) * nchunks + c) * Nq;
    for (int idx = tid; idx < Nq * D; idx += THREADS) {
        const int q = idx / D, t = idx % D;
        part_o[(slot0 + q) * D + t] = (xo[(0 * SPLIT_MAX_Q + q) * D + t] + xo[(1 * SPLIT_MAX_Q + q) * D + t]) +
                                      (xo[(2 * SPLIT_MAX_Q + q) * D + t] + xo[(3 * SPLIT_MAX_Q + q) * D + t]);
    }
    if (wave == 0 && g == 0 && r < Nq) {
        part_ml[2 * (slot0 + r)] = m2;
        part_ml[2 * (slot0 + r) + 1] = (sm.red[0][r] + sm.red[1][r]) + (sm.red[2][r] + sm.red[3][r]);
    }
#endif
}

// Second pass for 9 .. 32 queries per head (see SmemSplitKV): lines 9-13 per key tile with m known beforehand.
template <int D, bool CAUSAL, int NS>
__global__ __launch_bounds__(THREADS, 2) void splitk_pv_recompute_kernel(
    const int8_t *__restrict__ Q, const int8_t *__restrict__ K, const int8_t *__restrict__ V, const float *__restrict__ sQ,
    const float *__restrict__ sK, int Nq, int Nk, int cb, int nchunks, const float *__restrict__ tminG,
    const float *__restrict__ cminG, float *__restrict__ part_o, float *__restrict__ part_ml) {
#if defined(__HIP_DEVICE_COMPILE__)
    using Smem = SmemSplitKV<D, NS>;
    __shared__ Smem sm;
    constexpr int KS = D / 32, DT = D / 32, MAXQ = SPLIT_MAX_Q_RECOMPUTE;
    constexpr int PER_BLOCK = KS + DT + 2;                       // copy instructions per wavefront and block
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T_c = (Nk + BC - 1) / BC;
    const int head = blockIdx.x / nchunks, c = blockIdx.x % nchunks;
    const int jb0 = c * cb, jb1 = min(T_c, jb0 + cb);
    const int shift = CAUSAL ? Nk - Nq : 0;
    const int rq = min(r, Nq - 1);

    const BufRsrc rK = make_rsrc(K + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const BufRsrc rV = make_rsrc(V + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
    const BufRsrc rSK = make_rsrc(sK + static_cast<long>(head) * Nk, static_cast<unsigned>(Nk) * 4);
    const BufRsrc rT = make_rsrc(tminG + static_cast<long>(head) * T_c * MAXQ * 4, static_cast<unsigned>(T_c) * MAXQ * 4 * 4);
    const lds_ptr kbuf = (lds_ptr)(&sm.k[0][0]);
    const lds_ptr vbuf = (lds_ptr)(&sm.v[0][0]);
    const lds_ptr skbuf = (lds_ptr)(&sm.sk[0][0][0]);
    const lds_ptr tbuf = (lds_ptr)(&sm.tmin[0][0][0]);
    const LaneOffsets<D> lo(lane, wave);
    // this wavefront's key tile of K_j and V_j, its 32 s_K, and the block's 128 tile minima (lanes 32-63 repeat 0-31)
    auto stage_block = [&](int jb) {
        const int st = (jb - jb0) % NS;
        const bool real = jb < jb1;
        const Prefetch pf = {rK, rV, rSK, real ? jb * BC * D : NOWHERE, real ? jb * BC * 4 : NOWHERE,
                             kbuf + st * BC * D, vbuf + st * BC * D, skbuf + (st * 4 + wave) * 256};
        prefetch_k<D, SPLIT_NT>(pf, lo, wave);
        prefetch_v<D, SPLIT_NT>(pf, lo, wave);
        lds_copy4(pf.sk, pf.lsk, 4 * r + 128 * wave, pf.skoff);
        lds_copy16(rT, tbuf + (st * 4 + wave) * 1024, 16 * r, real ? jb * (MAXQ * 4 * 4) : NOWHERE);
    };
    stage_block(jb0);
    if (NS > 2) stage_block(jb0 + 1);

    const int8_t *qptr = Q + (static_cast<long>(head) * Nq + rq) * D + 16 * g;
    v4i qf[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = *reinterpret_cast<const v4i *>(qptr + 32 * kk);
    float nq2 = sQ[static_cast<long>(head) * Nq + rq] * (-LOG2E * ACC_UNIT);
    // minimum of a over the runs in front of this one: 8 threads per query
    float pre = INFINITY;
    {
        const int q = tid >> 3;
        if (q < Nq)
            for (int cc = tid & 7; cc < c; cc += 8) pre = fminf(pre, cminG[(static_cast<long>(head) * MAXQ + q) * nchunks + cc]);
#pragma unroll
        for (int s_ = 4; s_ >= 1; s_ >>= 1) pre = fminf(pre, __shfl_xor(pre, s_));
        if ((tid & 7) == 0) sm.pre[q] = pre;
    }
    // landed BEFORE the loop as far as the compiler is concerned (no wait of its own for them inside the loop)
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(qf[kk]));
    asm volatile("" : "+v"(nq2));
    __syncthreads();
    pre = sm.pre[rq];
    float m2 = (pre == INFINITY) ? -INFINITY : pre * nq2;        // line 10 over all earlier blocks (no block: line 6)
    float l = 0.0f, o[DT][16];
    v16i acc0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        acc0[v] = ACC_START_I;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt][v] = 0.0f;
    }

    for (int jb = jb0; jb < jb1; ++jb) {
        const int st = (jb - jb0) % NS, j0 = jb * BC;
        wait_vmcnt<(NS - 2) * PER_BLOCK>();                      // block jb has landed (NS = 3: block jb + 1 may be in flight)
        stage_block(jb + NS - 1);                                // into the stage of block jb - 1, which this wavefront has left
        const lds_ptr ks = kbuf + st * BC * D, vs = vbuf + st * BC * D;
        // line 9 for key tile `wave`, as in the first pass
        v4i kop[KS];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) kop[kk] = *reinterpret_cast<LDS_AS const v4i *>(k_operand<D>(ks, lo, kk) + 32 * wave * D);
        v4f skv[4];
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) skv[vq] = *reinterpret_cast<LDS_AS const v4f *>(skbuf + (st * 4 + wave) * 256 + lo.sk + 32 * vq);
        v16i sacc = acc0;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) sacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kop[kk], qf[kk], sacc, 0, 0, 0);
        const int tail = Nk - 1 - j0;
        const int klimit = CAUSAL ? min(rq + shift - j0, tail) : tail;
        const bool masked = CAUSAL ? (j0 + BC - 1 > min(shift, Nk - 1)) : (tail < BC - 1);   // wave-uniform
        // line 10 for the whole block: the four tile minima of this lane's query
        const v4f t4 = *reinterpret_cast<LDS_AS const v4f *>(tbuf + (st * 4 + wave) * 1024 + rq * 16);
        const float bmin = fminf(fminf(t4[0], t4[1]), fminf(t4[2], t4[3]));
        const float m_new = fmaxf(m2, bmin * nq2);
        const float alpha = __builtin_amdgcn_exp2f(m2 - m_new);
        const float mm = m_new - LOG2_R_NORM;
        m2 = m_new;
        // line 11
        v4i pw;
        uint32_t psum = 0;
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float av = (ACC_START_F - __int_as_float(sacc[4 * vq + e])) * skv[vq][e];
                if (masked && (32 * wave + 8 * vq + 4 * g + e > klimit)) av = INFINITY;
                x[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(av, nq2, -mm));
            }
            const uint32_t w = pack_p4(x);
            psum = __builtin_amdgcn_sad_u8(w, 0u, psum);
            pw[vq] = static_cast<int>(w);
        }
        l = __builtin_fmaf(l, alpha, static_cast<float>(psum));  // line 12 over this lane's keys of this tile
        // line 13 over the keys of this tile, all d tiles
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const v2i t0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<D>(vs, lo, dt) + 32 * wave * D));
            const v2i t1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<LDS_AS v2i *>(v_operand<D>(vs, lo, dt) + 16 * D + 32 * wave * D));
            const v4i vop = {t0[0], t0[1], t1[0], t1[1]};
            const v16i pacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(vop, pw, acc0, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) o[dt][v] = __builtin_fmaf(o[dt][v], alpha, -(ACC_START_F - __int_as_float(pacc[v])));
        }
    }
    wait_all_memory();
    // The four wavefronts hold partials of the same run at the same m: their sum is the workgroup's partial.  The K
    // and V rings (contiguous) are free once every wavefront has left the loop; [wavefront][query][d] floats go through them.
    static_assert(offsetof(Smem, v) == sizeof(Smem::k) && 4 * MAXQ * D * 4 <= 2 * NS * BC * D, "exchange area");
    const float lt = l + swap32(l);
    __syncthreads();
    float *xo = reinterpret_cast<float *>(&sm.k[0][0]);
    float *xl = reinterpret_cast<float *>(&sm.sk[0][0][0]);      // [wavefront][query]
    if (r < Nq) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq)
                *reinterpret_cast<v4f *>(xo + (wave * MAXQ + r) * D + 32 * dt + 8 * vq + 4 * g) = v4f{o[dt][4 * vq], o[dt][4 * vq + 1], o[dt][4 * vq + 2], o[dt][4 * vq + 3]};
        if (g == 0) xl[wave * MAXQ + r] = lt;
    }
    __syncthreads();
    const long slot0 = (static_cast<long>(head) * nchunks + c) * Nq;
    for (int idx = tid; idx < Nq * D; idx += THREADS) {
        const int q = idx / D, t = idx % D;
        part_o[(slot0 + q) * D + t] = (xo[(0 * MAXQ + q) * D + t] + xo[(1 * MAXQ + q) * D + t]) + (xo[(2 * MAXQ + q) * D + t] + xo[(3 * MAXQ + q) * D + t]);
    }
    if (wave == 0 && g == 0 && r < Nq) {
        part_ml[2 * (slot0 + r)] = m2;
        part_ml[2 * (slot0 + r) + 1] = (xl[r] + xl[MAXQ + r]) + (xl[2 * MAXQ + r] + xl[3 * MAXQ + r]);
    }
#endif
}

// Lines 15-17 over the partial results of one (head, query).  256 threads: thread (pg, dq) sums the parts p = pg, pg + PG,
// ... for output columns 4 dq .. 4 dq + 3 (PG = 1024 / D groups of parts, D / 4 column quads), LDS adds the groups up.
template <int D, typename OutT>
__global__ __launch_bounds__(THREADS) void splitk_combine_kernel(const float *__restrict__ part_o, const float *__restrict__ part_ml,
                                                                 const float *__restrict__ sV, int Nq, int parts, OutT *__restrict__ O) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int DQ = D / 4, PG = THREADS / DQ;
    __shared__ float xo[PG][D];
    __shared__ float xl[PG];
    const long hq = blockIdx.x, head = hq / Nq, q = hq % Nq;
    const int dq = threadIdx.x % DQ, pg = threadIdx.x / DQ;
    const long slot0 = head * parts * Nq + q;
    const float m_last = part_ml[2 * (slot0 + static_cast<long>(parts - 1) * Nq)];   // the running maximum never decreases
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    float l = 0.0f;
    for (int p = pg; p < parts; p += PG) {
        const long slot = slot0 + static_cast<long>(p) * Nq;
        const float w = __builtin_amdgcn_exp2f(part_ml[2 * slot] - m_last);
        const v4f x = *reinterpret_cast<const v4f *>(part_o + slot * D + 4 * dq);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(x[e], w, acc[e]);
        l = __builtin_fmaf(part_ml[2 * slot + 1], w, l);
    }
    *reinterpret_cast<v4f *>(&xo[pg][4 * dq]) = acc;
    if (dq == 0) xl[pg] = l;
    __syncthreads();
    if (threadIdx.x < D) {
        const int t = threadIdx.x;
        float y = 0.0f, lsum = 0.0f;
#pragma unroll
        for (int i = 0; i < PG; ++i) { y += xo[i][t]; lsum += xl[i]; }
        y *= sV[head] * ACC_UNIT / lsum;
        asm volatile("" : "+v"(y));   // the fp32 product, rounded once more below: never a mixed-precision multiply that rounds straight to 16 bits
        if constexpr (sizeof(OutT) == 2) reinterpret_cast<uint16_t *>(O)[hq * D + t] = static_cast<uint16_t>(Pack4<OutT>::pack(y, 0.0f, 0.0f, 0.0f).x & 0xffffu);
        else O[hq * D + t] = y;
    }
#endif
}

// ---- host side ----------------------------------------------------------------------------------
template <int D, bool CAUSAL, bool VB, typename OutT>
int launch_packed(const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV,
                  int heads, int Nq, int Nk, void *O, hipStream_t st) {
    const long wgs = static_cast<long>(heads) * ((Nq + PACKED_BR - 1) / PACKED_BR);
    hipLaunchKernelGGL((int_flash_attn_fwd_packed_kernel<D, CAUSAL, VB, OutT>), dim3(static_cast<unsigned>(wgs)), dim3(THREADS), 0, st,
                       Q, K, V, sQ, sK, sV, heads, Nq, Nk, static_cast<OutT *>(O));
    return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
}

template <int D>
int launch_decode(const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV, int heads, int Nq, int Nk,
                  int causal, int vblock, int o_dtype, void *O, hipStream_t st) {
    constexpr int DS = D / 32;
    const dim3 grid(static_cast<unsigned>((heads + 7) / 8 * 8 * DS));
    if (Nq == 1) hipLaunchKernelGGL((int_flash_attn_fwd_decode_kernel<D, DS>), grid, dim3(DEC_THREADS), 0, st, Q, K, V, sQ, sK, sV, heads, Nk, vblock, o_dtype, O);
    else hipLaunchKernelGGL((int_flash_attn_fwd_draft_kernel<D, DS>), grid, dim3(DEC_THREADS), 0, st, Q, K, V, sQ, sK, sV, heads, Nq, Nk, causal, vblock, o_dtype, O);
    return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
}

template <int D, bool CAUSAL, bool VB, typename OutT>
int launch_narrow(IfaKernel kernel, const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV,
                  int heads, int Nq, int Nk, void *O, hipStream_t st) {
    if (kernel == IFA_KERNEL_PAIR) {
        const int T_r = (Nq + PAIR_BR - 1) / PAIR_BR;
        hipLaunchKernelGGL((int_flash_attn_fwd_pair_kernel<D, CAUSAL, VB, OutT>), dim3(static_cast<unsigned>(static_cast<long>(heads) * T_r)),
                           dim3(NARROW_THREADS), 0, st, Q, K, V, sQ, sK, sV, heads, Nq, Nk, head_group_for(CAUSAL, 2L * Nk * D, T_r), static_cast<OutT *>(O));
        return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
    }
    if (kernel == IFA_KERNEL_PACKED) return launch_packed<D, CAUSAL, VB, OutT>(Q, K, V, sQ, sK, sV, heads, Nq, Nk, O, st);
    const long qgroups = (Nq + NARROW_BR - 1) / NARROW_BR, padded = (heads * qgroups + 7) / 8 * 8;
    if (ifa_decode_query(heads, Nq, Nk, D))
        return launch_decode<D>(Q, K, V, sQ, sK, sV, heads, Nq, Nk, CAUSAL, VB, sizeof(OutT) == 4 ? IFA_F32 : std::is_same_v<OutT, __half> ? IFA_F16 : IFA_BF16, O, st);
    // K and V with the non-temporal hint where one workgroup reads each byte, and reads it once, and there are more of them than the
    // caches could keep for the next call; such a call runs with DS = 1.  (With the hint and DS = 2 the second workgroup of a pair may
    // find a line gone: right after K and V were written the call below fetched 730 - 790 MB, 545 with DS = 1.)  128 heads x 1 x 16384, 537 MB, us, after
    // the same call / after a read of 512 MB elsewhere / after a copy of 512 MB / right after K and V were quantized:
    //   hint, DS = 1 94 / 95 / 112 / 108;  hint, DS = 2 89 / 91 / 109 / 139;  no hint, DS = 2 100 / 100 / 120 / 122;  key split 100 / 103 / 112 / 112.
    // (At d = 128 the line matters from 65 heads on, at d = 64 from 129 on: fewer with one query run the decode kernel.)
    const int once = qgroups == 1 && 2L * heads * Nk * D > (64L << 20);
    auto launch = [&](auto ds) {
        constexpr int DS = decltype(ds)::value;
        hipLaunchKernelGGL((int_flash_attn_fwd_narrow_kernel<D, CAUSAL, VB, OutT, DS>), dim3(static_cast<unsigned>(padded * DS)), dim3(NARROW_THREADS), 0,
                           st, Q, K, V, sQ, sK, sV, heads, Nq, Nk, once, static_cast<OutT *>(O));
    };
    if constexpr (D == 128) {
        // two workgroups per query group as long as each then has a CU of its own
        if (heads * qgroups <= 128 && !once) launch(std::integral_constant<int, 2>{});
        else launch(std::integral_constant<int, 1>{});
    } else launch(std::integral_constant<int, 1>{});
    return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
}

// The three passes of the key-split path on one stream; `ws` is the workspace laid out by split_plan().
template <int D, bool CAUSAL, typename OutT>
int launch_splitk(const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV,
                  int heads, int Nq, int Nk, void *O, float *ws, hipStream_t st) {
    const SplitPlan p = split_plan(heads, Nq, Nk, D);
    float *scores = ws, *tmin = ws + p.off_tmin, *cmin = ws + p.off_cmin, *part_o = ws + p.off_part_o, *part_ml = ws + p.off_part_ml;
    const dim3 grid(static_cast<unsigned>(static_cast<long>(heads) * p.nchunks));
    if (p.store) {
        hipLaunchKernelGGL((splitk_scores_kernel<D, CAUSAL, SPLIT_MAX_Q, true>), grid, dim3(THREADS), 0, st, Q, K, sK, Nq, Nk, p.cb, p.nchunks,
                           scores, tmin, cmin);
        hipLaunchKernelGGL((splitk_pv_kernel<D>), grid, dim3(THREADS), 0, st, V, sQ, Nq, Nk, p.cb, p.nchunks, scores, tmin, cmin, part_o, part_ml);
    } else {
        hipLaunchKernelGGL((splitk_scores_kernel<D, CAUSAL, SPLIT_MAX_Q_RECOMPUTE, false>), grid, dim3(THREADS), 0, st, Q, K, sK, Nq, Nk, p.cb,
                           p.nchunks, scores, tmin, cmin);
        auto launch = [&](auto ns) {
            hipLaunchKernelGGL((splitk_pv_recompute_kernel<D, CAUSAL, decltype(ns)::value>), grid, dim3(THREADS), 0, st, Q, K, V, sQ, sK, Nq, Nk, p.cb,
                               p.nchunks, tmin, cmin, part_o, part_ml);
        };
        if constexpr (D == 64) {
            if (p.cb >= SPLIT_LONG_RUN) launch(std::integral_constant<int, 3>{});
            else launch(std::integral_constant<int, 2>{});
        } else launch(std::integral_constant<int, 2>{});
    }
    hipLaunchKernelGGL((splitk_combine_kernel<D, OutT>), dim3(static_cast<unsigned>(heads * Nq)), dim3(THREADS), 0, st, part_o, part_ml, sV,
                       Nq, p.parts, static_cast<OutT *>(O));
    return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
}

template <int D, bool CAUSAL>
int launch_splitk_dtype(const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV,
                        int heads, int Nq, int Nk, void *O, int o_dtype, float *ws, hipStream_t st) {
    switch (o_dtype) {
    case IFA_F32: return launch_splitk<D, CAUSAL, float>(Q, K, V, sQ, sK, sV, heads, Nq, Nk, O, ws, st);
    case IFA_F16: return launch_splitk<D, CAUSAL, __half>(Q, K, V, sQ, sK, sV, heads, Nq, Nk, O, ws, st);
    default: return launch_splitk<D, CAUSAL, __hip_bfloat16>(Q, K, V, sQ, sK, sV, heads, Nq, Nk, O, ws, st);
    }
}

// argument checks of the key-split path that do not concern the workspace
int splitk_args(const signed char *Q_i8, const signed char *K_i8, const signed char *V_i8, const float *s_Q, const float *s_K,
                const float *s_V, int B, int H, int Nq, int Nk, int d, int causal, const void *O, int o_dtype) {
    if (!Q_i8 || !K_i8 || !V_i8 || !s_Q || !s_K || !s_V || !O) return IFA_ERR_NULL;
    if (B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0 || d <= 0) return IFA_ERR_SHAPE;
    const long heads = static_cast<long>(B) * H;
    if (heads > (1L << 40) / Nk / d) return IFA_ERR_SHAPE;
    if (causal && Nk < Nq) return IFA_ERR_UNSUPPORTED;           // a query with no visible key
    if (o_dtype < IFA_F32 || o_dtype > IFA_BF16) return IFA_ERR_DTYPE;
    if ((d != 64 && d != 128) || Nq > SPLIT_MAX_Q_RECOMPUTE) return IFA_ERR_UNSUPPORTED;
    if (static_cast<long>(Nk) * d > 0x7ff00000L) return IFA_ERR_UNSUPPORTED;      // a head's K (or V) stays below NOWHERE
    const SplitPlan p = split_plan(heads, Nq, Nk, d);
    if (static_cast<long>(p.T_c) * 4 * p.maxq * 128 > 0x7ff00000L ||               // so do a head's scores and minima arrays
        heads * p.nchunks > 0x7fffffffL || heads * Nq > 0x7fffffffL) return IFA_ERR_UNSUPPORTED;
    if (!ifa_aligned16(Q_i8) || !ifa_aligned16(K_i8) || !ifa_aligned16(V_i8) || !ifa_aligned16(O) ||
        (reinterpret_cast<uintptr_t>(s_Q) & 3) || (reinterpret_cast<uintptr_t>(s_K) & 3) || (reinterpret_cast<uintptr_t>(s_V) & 3))
        return IFA_ERR_UNSUPPORTED;
    return IFA_OK;
}

int splitk_dispatch(const signed char *Q_i8, const signed char *K_i8, const signed char *V_i8, const float *s_Q, const float *s_K,
                    const float *s_V, int B, int H, int Nq, int Nk, int d, int causal, void *O, int o_dtype, float *ws,
                    hipStream_t st) {
    const int8_t *Q = reinterpret_cast<const int8_t *>(Q_i8);
    const int8_t *K = reinterpret_cast<const int8_t *>(K_i8);
    const int8_t *V = reinterpret_cast<const int8_t *>(V_i8);
    const int hd = B * H;
    if (ifa_unsplit_queries(hd, Nq, Nk, d)) return ifa_launch_fwd(Q, K, V, s_Q, s_K, s_V, hd, Nq, Nk, d, causal, O, o_dtype, st);
    if (d == 128)
        return causal ? launch_splitk_dtype<128, true>(Q, K, V, s_Q, s_K, s_V, hd, Nq, Nk, O, o_dtype, ws, st)
                      : launch_splitk_dtype<128, false>(Q, K, V, s_Q, s_K, s_V, hd, Nq, Nk, O, o_dtype, ws, st);
    return causal ? launch_splitk_dtype<64, true>(Q, K, V, s_Q, s_K, s_V, hd, Nq, Nk, O, o_dtype, ws, st)
                  : launch_splitk_dtype<64, false>(Q, K, V, s_Q, s_K, s_V, hd, Nq, Nk, O, o_dtype, ws, st);
}

}  // namespace

// The narrow kernel for the dispatcher of the fused kernel's entry points (arguments already validated there).
int ifa_launch_narrow(IfaKernel kernel, const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV, int heads,
                      int Nq, int Nk, int d, int causal, int vblock, void *O, int o_dtype, hipStream_t st) {
    auto by_dtype = [&](auto D_, auto C_, auto VB_) {
        constexpr int D = decltype(D_)::value;
        constexpr bool C = decltype(C_)::value, VB = decltype(VB_)::value;
        switch (o_dtype) {
        case IFA_F32: return launch_narrow<D, C, VB, float>(kernel, Q, K, V, sQ, sK, sV, heads, Nq, Nk, O, st);
        case IFA_F16: return launch_narrow<D, C, VB, __half>(kernel, Q, K, V, sQ, sK, sV, heads, Nq, Nk, O, st);
        default: return launch_narrow<D, C, VB, __hip_bfloat16>(kernel, Q, K, V, sQ, sK, sV, heads, Nq, Nk, O, st);
        }
    };
    using I64 = std::integral_constant<int, 64>;
    using I128 = std::integral_constant<int, 128>;
    auto by_flags = [&](auto D_) {
        if (causal) return vblock ? by_dtype(D_, std::true_type{}, std::true_type{}) : by_dtype(D_, std::true_type{}, std::false_type{});
        return vblock ? by_dtype(D_, std::false_type{}, std::true_type{}) : by_dtype(D_, std::false_type{}, std::false_type{});
    };
    return d == 128 ? by_flags(I128{}) : by_flags(I64{});
}

extern "C" long ifa_splitk_workspace_bytes(int B, int H, int Nq, int Nk, int d) {
    if (B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0 || (d != 64 && d != 128) || Nq > SPLIT_MAX_Q_RECOMPUTE) return 0;
    const long heads = static_cast<long>(B) * H;
    if (heads > (1L << 40) / Nk / d) return 0;
    return split_plan(heads, Nq, Nk, d).words * 4;
}

extern "C" int int_flash_attn_fwd_splitk(const signed char *Q_i8, const signed char *K_i8, const signed char *V_i8,
                                         const float *s_Q, const float *s_K, const float *s_V, int B, int H, int Nq, int Nk,
                                         int d, int causal, void *O, int o_dtype, void *workspace, long workspace_bytes,
                                         void *hip_stream) {
    const int rc = splitk_args(Q_i8, K_i8, V_i8, s_Q, s_K, s_V, B, H, Nq, Nk, d, causal, O, o_dtype);
    if (rc != IFA_OK) return rc;
    if (!workspace) return IFA_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(workspace) & 255) return IFA_ERR_UNSUPPORTED;
    if (workspace_bytes < ifa_splitk_workspace_bytes(B, H, Nq, Nk, d)) return IFA_ERR_WORKSPACE;
    return splitk_dispatch(Q_i8, K_i8, V_i8, s_Q, s_K, s_V, B, H, Nq, Nk, d, causal, O, o_dtype, static_cast<float *>(workspace),
                           static_cast<hipStream_t>(hip_stream));
}

// ---- the key-split path for callers that cannot allocate -------------------------------------------------------
// The same launches with the workspace in a file-scope device array instead of a buffer of the caller's.  In
// host code the array's name is only a stand-in for the symbol: the device address is asked for once per device
// (hipGetSymbolAddress, with that device current) and kept; every GPU holds its own copy of the array.
constexpr long STATIC_WORKSPACE_BYTES = 16L << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_WORKSPACE_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
void *g_scratch_ptr[MAX_DEVICES];
std::mutex g_scratch_mutex;

// device address of `scratch` on the current device, or null
void *static_workspace() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

// Also the set-up call: it resolves the array's address on the current device, so that a later
// int_flash_attn_fwd_splitk_static on this device (under graph capture, say) has no set-up left to do.
extern "C" long ifa_static_workspace_bytes(void) {
    (void)static_workspace();
    return STATIC_WORKSPACE_BYTES;
}

extern "C" int int_flash_attn_fwd_splitk_static(const signed char *Q_i8, const signed char *K_i8, const signed char *V_i8,
                                                const float *s_Q, const float *s_K, const float *s_V, int B, int H, int Nq,
                                                int Nk, int d, int causal, void *O, int o_dtype, void *hip_stream) {
    const int rc = splitk_args(Q_i8, K_i8, V_i8, s_Q, s_K, s_V, B, H, Nq, Nk, d, causal, O, o_dtype);
    if (rc != IFA_OK) return rc;
    if (ifa_splitk_workspace_bytes(B, H, Nq, Nk, d) > STATIC_WORKSPACE_BYTES) return IFA_ERR_WORKSPACE;
    void *ws = static_workspace();
    if (!ws) return IFA_ERR_HIP;
    return splitk_dispatch(Q_i8, K_i8, V_i8, s_Q, s_K, s_V, B, H, Nq, Nk, d, causal, O, o_dtype, static_cast<float *>(ws),
                           static_cast<hipStream_t>(hip_stream));
}


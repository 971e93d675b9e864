// Half-INT8 variant of the INT-FlashAttention forward pass for gfx950 (Section 4 of arXiv 2409.16997: INT8 Q and K
// with token-level scales, V kept in FP16).  The first GEMM and everything up to the running max are those of
// Algorithm 1; the softmax weights then stay real, are rounded to FP16 and meet the caller's FP16 V on
// v_mfma_f32_32x32x16_f16:
//     S^T = K_j Q_i^T                 v_mfma_i32_32x32x32_i8, fp32 scales             (lines 9-10)
//     P~  = fp16(exp(S - m))          no factor R; round to nearest even, subnormals kept
//     l   = alpha l + rowsum(P~)      the rounded weights, summed in fp32 (v_dot2_f32_f16 with ones)
//     O^T = alpha O^T + V_j^T P~^T    the MFMA accumulates straight onto the rescaled fp32 output
//     O   = O / l
//
// Same orientation and work split as the INT8 kernel (workgroup = 4 wavefronts = 128 queries, a lane owns one
// query), but the key block is B_c = 64: an FP16 V tile is twice the bytes of an INT8 one, and 64 keys keep
// K (2 x 8 KB) + V (2 x 16 KB) double-buffered at two workgroups per CU.  In the 32x32 accumulator layout a lane
// holds keys 8*(v/4) + 4*g + v%4 of a 32-key tile; two consecutive v/4 groups are the 8 contraction halves one
// lane feeds to a 32x32x16 MFMA, so P~ never leaves registers here either.  The matching V^T operand (8 keys of
// one d column per lane, V being [keys, d]) is gathered by the LDS with ds_read_b64_tr_b16: within 16 lanes,
// lane 4k+j addresses 4 halves (d = d0+4j .. +3) of key k, and lane i receives d column d0+i of keys 0..3.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <hip/hip_bf16.h>
#include <stdint.h>
#include <type_traits>

#include "intfa.h"
#include "intfa_internal.h"
#include "intfa_device.h"

namespace {

using namespace ifa_dev;

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef short s4 __attribute__((ext_vector_type(4)));

constexpr int BCH = 64;       // keys per block of this variant
[[maybe_unused]] constexpr int NT = BCH / 32;  // 32-key tiles per block

template <int D> struct SmemH {
    alignas(4096) int8_t k[2][BCH * D];        // K_j int8, row = key, 16-byte slots XOR-swizzled by row
    alignas(1024) int8_t v[2][BCH * D * 2];    // V_j fp16, row = key (2 D bytes), 64-byte chunks XOR-swizzled by row
    alignas(256) float sk[2][BCH];             // s_K of the block
};
// lds_xor() wants every K / V tile at a multiple of 4096 bytes
static_assert((BCH * 64) % 4096 == 0 && offsetof(SmemH<64>, v) % 4096 == 0 && offsetof(SmemH<128>, v) % 4096 == 0, "tile bases");

template <int D> __device__ __forceinline__ int kh_swz(int row) {
    return (D == 128) ? (row & 7) : ((row >> 1) & 3);
}
// V rows are read 4 consecutive keys at a time at one 64-byte chunk: the low key bits pick the chunk slot
template <int D> __device__ __forceinline__ int vh_swz(int row) {
    return (D == 128) ? (row & 3) : (row & 1);
}

#if defined(__HIP_DEVICE_COMPILE__)

template <int D> struct LaneOffsetsH {
    static constexpr int KS = D / 32, DT = D / 32, KP = D / 64, VP = D / 32;
    // A operand of S^T: row r, 16-byte chunk 2*kk + g.  The swizzle XORs the chunk index and 2*kk + g = 2*kk ^ g,
    // so step kk is at k0 ^ (32*kk)   (+ 32*mt*D per key tile, an immediate)
    unsigned k0;
    // A operand of O^T: keys 4g + (i/4) of a 16-key step, d tile dt at v0 ^ (64*dt); the keys 8 further on, which the
    // swizzle does not see, at + 8 * 2D   (+ (32*mt + 16*s) * 2D per step)
    unsigned v0;
    // staging: byte offset inside the K / V block in HBM of the chunk this lane moves in piece 0 of its wavefront;
    // piece i is 1024 bytes further on (whole rows, which the swizzles do not see)
    unsigned gk, gv;
    __device__ __forceinline__ LaneOffsetsH(int lane, int wave) {
        const int r = lane & 31, g = lane >> 5;
        constexpr int CH = D / 16, CHV = D / 8;      // 16-byte slots per K row / per V row
        {
            const int p = wave * KP * 64 + lane, row = p / CH, slot = p % CH;      // a piece is 1024 / D >= 8 rows
            gk = row * D + 16 * (slot ^ kh_swz<D>(row));
        }
        {
            const int p = wave * VP * 64 + lane, row = p / CHV, slot = p % CHV;    // a piece is 512 / D >= 4 rows
            gv = row * (2 * D) + 16 * (slot ^ (vh_swz<D>(row) << 2));
        }
        k0 = r * D + ((g ^ kh_swz<D>(r)) * 16);
        const int i = lane & 15, G = lane >> 4, kq = i >> 2, j = i & 3;
        const int key = 4 * g + kq;
        v0 = key * (2 * D) + (vh_swz<D>(key) * 64) + 32 * (G & 1) + 8 * j;
    }
};

struct PrefetchH {
    BufRsrc k, v, sk;                // one head's K [N, d] int8, V [N, d] fp16 and s_K [N] fp32
    int koff, voff, skoff;           // byte offsets of the next block inside K, V and s_K
    lds_ptr lk, lv, lsk;             // LDS destinations
};
// Block offset of a request that must fetch nothing (no block follows): past the end of any tensor, so every lane
// is out of range (the scalar offset takes part in the range check) and the copy moves no data.
constexpr int NOWHERE_H = 0x7fff0000;

template <int D>
__device__ __forceinline__ void prefetch_block(const PrefetchH &nx, const LaneOffsetsH<D> &lo, int wave, int lane) {
    constexpr int KP = D / 64, VP = D / 32;
#pragma unroll
    for (int i = 0; i < KP; ++i) lds_copy16_piece<KP>(i, nx.k, nx.lk + wave * KP * 1024, lo.gk, lo.gk, nx.koff);
#pragma unroll
    for (int i = 0; i < VP; ++i) lds_copy16_piece<VP>(i, nx.v, nx.lv + wave * VP * 1024, lo.gv, lo.gv, nx.voff);
    if (wave == 3) lds_copy4(nx.sk, nx.lsk, 4 * lane, nx.skoff);       // 64 lanes x 4 bytes = the 64 scales of the block
}

template <int D> struct RowStateH {
    float m2;             // running max in log2 units (identical in lanes r and r + 32)
    float l;              // running sum of the rounded weights over this lane's keys
    v16f o[D / 32];       // running output, d = 32*dt + 8*(v/4) + 4*g + v%4: the MFMA accumulator itself
};

// One key block already resident in LDS.  MASKED: a block with masked keys (on or past the causal diagonal, or the
// ragged last block): a key of the block is kept iff its index inside the block is <= klimit (per lane, may be
// negative); the first `clear_tiles` 32-key tiles (wave-uniform) hold no masked key for any lane of the wavefront;
// 32-key tiles after tile `last` (wave-uniform, -1: none) are masked for every lane and skipped.
template <int D, bool MASKED>
__device__ __forceinline__ void process_block_half(lds_ptr ks, lds_ptr vs, lds_ptr sk, const LaneOffsetsH<D> &lo,
                                                   const v4i (&qf)[D / 32], float sq2, int klimit, int last_tile, int clear_tiles, int g,
                                                   const v16i &bias, RowStateH<D> &st) {
    constexpr int KS = D / 32, DT = D / 32;
    const int last = MASKED ? last_tile : NT - 1;
    float a[NT][16];
    float bmax = -INFINITY;

    // The source is software-pipelined like the INT8 kernel's: LDS operands of the next MFMA group are requested
    // before the current group is issued, and the vector work on tile t-1 follows the MFMAs of tile t.
    v4i kop[2][KS];
    v4f skr[2][4];
    auto load_k = [&](int buf, int mt) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) kop[buf][kk] = *reinterpret_cast<LDS_AS const v4i *>(lds_xor(ks, 32 * kk, lo.k0) + 32 * mt * D);
    };
    auto load_sk = [&](int buf, int mt) {
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) skr[buf][vq] = *reinterpret_cast<LDS_AS const v4f *>(sk + 16 * g + 128 * mt + 32 * vq);
    };
    auto scale_elems = [&](int mt, const v16i &acc, const v4f (&skv)[4], auto masked) {   // line 9, fp32 part: a = acc * s_K
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float x = (__int_as_float(acc[4 * vq + e]) - ACC_BIAS_F) * skv[vq][e];
                if (decltype(masked)::value && (32 * mt + 8 * vq + 4 * g + e > klimit)) x = -INFINITY;   // masked key
                a[mt][4 * vq + e] = x;
                bmax = fmaxf(bmax, x);
            }
    };
    // only the tiles the mask boundary crosses pay for the comparisons (wave-uniform choice)
    auto scale_tile = [&](int mt, const v16i &acc, const v4f (&skv)[4]) {
        if (MASKED && mt >= clear_tiles) scale_elems(mt, acc, skv, std::true_type{});
        else scale_elems(mt, acc, skv, std::false_type{});
    };
    // V^T operands of d tile dt: one h8 per 16-key step of the active tiles
    h8 vop[2][2 * NT];
    auto load_v = [&](int buf, int dt) {
#pragma unroll
        for (int mt = 0; mt < NT; ++mt)
            if (mt <= last) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int koff = (32 * mt + 16 * s) * (2 * D);
                    const h4 t0 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s4 *>(lds_xor(vs, 64 * dt, lo.v0) + koff)));
                    const h4 t1 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s4 *>(lds_xor(vs, 64 * dt, lo.v0) + 8 * (2 * D) + koff)));
                    vop[buf][2 * mt + s] = h8{t0[0], t0[1], t0[2], t0[3], t1[0], t1[1], t1[2], t1[3]};
                }
            }
    };

    // ---- S^T = K Q^T, tile by tile
    v16i sacc[2];
    load_k(0, 0);
    load_sk(0, 0);
#pragma unroll
    for (int mt = 0; mt < NT; ++mt) {
        if (mt <= last) {
            if (mt + 1 <= last) load_k((mt + 1) & 1, mt + 1);
            sacc[mt & 1] = bias;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
                sacc[mt & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kop[mt & 1][kk], qf[kk], sacc[mt & 1], 0, 0, 0);
            if (mt > 0) scale_tile(mt - 1, sacc[(mt - 1) & 1], skr[(mt - 1) & 1]);
            if (mt + 1 <= last) load_sk((mt + 1) & 1, mt + 1);
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) a[mt][v] = -INFINITY;
        }
    }
    if constexpr (MASKED) load_v(0, 0);                           // first V^T operands go out before the last tile is scaled
#pragma unroll
    for (int mt = 0; mt < NT; ++mt)
        if (mt == last) scale_tile(mt, sacc[mt & 1], skr[mt & 1]);

    bmax = pair_max(bmax);
    const float m_new = fmaxf(st.m2, bmax * sq2);                 // finite from the first block on (key 0 is never masked)
    const float alpha = __builtin_amdgcn_exp2f(st.m2 - m_new);    // exp2(-inf) = 0 on the first block
    st.m2 = m_new;

    // ---- P~ = fp16(2^(a s_Q' - m)), two keys per register in accumulator order; l sums the rounded values
    h2 ph[NT][8];
    float psum = 0.0f;
    const h2 ones = {(_Float16)1.0f, (_Float16)1.0f};
    auto p_pair = [&](int mt, int c) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(a[mt][2 * c], sq2, -m_new));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(a[mt][2 * c + 1], sq2, -m_new));
        const h2 w = {(_Float16)p0, (_Float16)p1};
        ph[mt][c] = w;
        psum = __builtin_amdgcn_fdot2(w, ones, psum, false);
    };
    if constexpr (!MASKED) {
        // Unmasked blocks: the second GEMM runs key tile by key tile over all d tiles, with the weights of the NEXT key
        // tile computed between its MFMAs at raised wave priority (two exps per MFMA hide behind it); each V^T operand
        // is re-requested for the next key tile right after the MFMA that read it has issued.
        h8 vt[DT][2];
        auto load_v1 = [&](int mt, int dt, int s_) {
            const int koff = (32 * mt + 16 * s_) * (2 * D);
            const h4 t0 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s4 *>(lds_xor(vs, 64 * dt, lo.v0) + koff)));
            const h4 t1 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s4 *>(lds_xor(vs, 64 * dt, lo.v0) + 8 * (2 * D) + koff)));
            vt[dt][s_] = h8{t0[0], t0[1], t0[2], t0[3], t1[0], t1[1], t1[2], t1[3]};
        };
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) { load_v1(0, dt, 0); load_v1(0, dt, 1); }
#pragma unroll
        for (int c = 0; c < 8; ++c) p_pair(0, c);
        __builtin_amdgcn_s_setprio(3);
#pragma unroll
        for (int mt = 0; mt < NT; ++mt) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                if (mt == 0) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) st.o[dt][v] *= alpha;
                }
#pragma unroll
                for (int s_ = 0; s_ < 2; ++s_) {
                    const h8 pb = {ph[mt][4 * s_][0], ph[mt][4 * s_][1], ph[mt][4 * s_ + 1][0], ph[mt][4 * s_ + 1][1],
                                   ph[mt][4 * s_ + 2][0], ph[mt][4 * s_ + 2][1], ph[mt][4 * s_ + 3][0], ph[mt][4 * s_ + 3][1]};
                    st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vt[dt][s_], pb, st.o[dt], 0, 0, 0);
                    if (mt + 1 < NT) load_v1(mt + 1, dt, s_);
                }
                if (mt + 1 < NT) {
#pragma unroll
                    for (int q = 0; q < 8 / DT; ++q) p_pair(mt + 1, dt * (8 / DT) + q);
                }
            }
        }
        __builtin_amdgcn_s_setprio(0);
        st.l = __builtin_fmaf(st.l, alpha, psum);
        return;
    }
#pragma unroll
    for (int mt = 0; mt < NT; ++mt) {
        if (mt <= last) {
#pragma unroll
            for (int c = 0; c < 8; ++c) p_pair(mt, c);
        }
    }
    st.l = __builtin_fmaf(st.l, alpha, psum);

    // ---- O^T = alpha O^T + V^T P~^T: each d tile is rescaled in place, then the fp16 MFMAs accumulate onto it
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        if (dt + 1 < DT) load_v((dt + 1) & 1, dt + 1);
#pragma unroll
        for (int v = 0; v < 16; ++v) st.o[dt][v] *= alpha;
#pragma unroll
        for (int mt = 0; mt < NT; ++mt) {
            if (mt <= last) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {                       // 16-key steps of the tile
                    const h8 pb = {ph[mt][4 * s][0], ph[mt][4 * s][1], ph[mt][4 * s + 1][0], ph[mt][4 * s + 1][1],
                                   ph[mt][4 * s + 2][0], ph[mt][4 * s + 2][1], ph[mt][4 * s + 3][0], ph[mt][4 * s + 3][1]};
                    st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vop[dt & 1][2 * mt + s], pb, st.o[dt], 0, 0, 0);
                }
            }
        }
    }
}

// The same block, same results, in registers for three wavefronts per SIMD (d = 64: four), for calls with enough workgroups.  Two wavefronts
// take turns at matrix and vector instructions and wait out each other's row maximum, LDS reads and barrier, every 64 keys; a third one fills in.  168
// registers (d = 64: 116) hold the block without the 16 the S^T accumulators start from (the MFMA's inline constant; a is carried in units of
// 2^26, a power of two, so the numbers are the same as long as neither it nor s_Q times that leaves the range: FAR_SQ), with the scores in the accumulators' place and the s_K of one key tile, reloaded as
// they are used.  Two / three or four, us: d = 64, 32 x 8192 causal 350 / 302, 64 x 4096 340 / 303, 128 x 4096 causal 359 / 326, 300 x 200 12.7 / 10.2;
// d = 128, 32 x 16384 causal 1874 / 1811, 96 x 1724 154 / 151, 300 x 200 18.0 / 15.6, 600 x 128 causal 15.0 / 12.5.  With few workgroups the order of the function
// above is faster, which has all of its LDS operands requested earlier: 24 x 1400 at d = 128 36.8 / 38.5.
// FAR: for a wavefront with a row whose s_Q is beyond FAR_SQ: s_Q 2^26 log2 e could be infinite from 2^101 on, and s_K 2^-26 loses bits that such a row can see.
// Up to FAR_SQ what is lost below 2^-149 is less than 2^-33 of a score.
constexpr float FAR_SQ = 1.2379400392853803e27f;                 // 2^90
template <int D, bool MASKED, bool FAR>
__device__ __forceinline__ void process_block_half_lean(lds_ptr ks, lds_ptr vs, lds_ptr sk, const LaneOffsetsH<D> &lo,
                                                        const v4i (&qf)[D / 32], float sq2, int klimit, int last_tile, int clear_tiles, int g,
                                                        RowStateH<D> &st) {
    constexpr int KS = D / 32, DT = D / 32;
    const int last = MASKED ? last_tile : NT - 1;
    v16i sacc[NT];
    float a[NT][16];
    float bmax = -INFINITY;
    v4i kop[NT][KS];
    v4f skr[4];
    auto load_k = [&](int mt) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) kop[mt][kk] = *reinterpret_cast<LDS_AS const v4i *>(lds_xor(ks, 32 * kk, lo.k0) + 32 * mt * D);
    };
    auto load_sk = [&](int mt, int vq) { skr[vq] = *reinterpret_cast<LDS_AS const v4f *>(sk + 16 * g + 128 * mt + 32 * vq); };

    // ---- S^T = K Q^T, tile by tile
    load_k(0);
#pragma unroll
    for (int mt = 0; mt < NT; ++mt) {
        if (mt <= last) {
            if (mt + 1 <= last) load_k(mt + 1);
            if (mt == last) {
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) load_sk(0, vq);
            }
            sacc[mt] = mfma_i8_start(kop[mt][0], qf[0]);
#pragma unroll
            for (int kk = 1; kk < KS; ++kk) sacc[mt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kop[mt][kk], qf[kk], sacc[mt], 0, 0, 0);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // line 9, fp32 part, in place: a = acc * s_K in units of 2^26
#pragma unroll
    for (int mt = 0; mt < NT; ++mt) {
        if (mt <= last) {
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float x = __int_as_float(sacc[mt][4 * vq + e]) - ACC_START_F;
                    if (FAR) x *= ACC_UNIT;
                    x *= skr[vq][e];
                    if (MASKED && mt >= clear_tiles && 32 * mt + 8 * vq + 4 * g + e > klimit) x = -INFINITY;
                    a[mt][4 * vq + e] = x;
                    bmax = fmaxf(bmax, x);
                }
                if (mt + 1 <= last) load_sk(mt + 1, vq);
            }
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) a[mt][v] = -INFINITY;
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    bmax = pair_max(bmax);
    const float m_new = fmaxf(st.m2, bmax * sq2);                 // finite from the first block on (key 0 is never masked)
    const float alpha = __builtin_amdgcn_exp2f(st.m2 - m_new);    // exp2(-inf) = 0 on the first block
    st.m2 = m_new;

    // ---- P~ = fp16(2^(a s_Q' - m)), two keys per register in accumulator order; l sums the rounded values
    h2 ph[NT][8];
    float psum = 0.0f;
    const h2 ones = {(_Float16)1.0f, (_Float16)1.0f};
    auto p_pair = [&](int mt, int c) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(a[mt][2 * c], sq2, -m_new));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(a[mt][2 * c + 1], sq2, -m_new));
        const h2 w = {(_Float16)p0, (_Float16)p1};
        ph[mt][c] = w;
        psum = __builtin_amdgcn_fdot2(w, ones, psum, false);
    };
    h8 vt[DT][2];
    auto load_v1 = [&](int mt, int dt, int s_) {
        const int koff = (32 * mt + 16 * s_) * (2 * D);
        const h4 t0 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s4 *>(lds_xor(vs, 64 * dt, lo.v0) + koff)));
        const h4 t1 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s4 *>(lds_xor(vs, 64 * dt, lo.v0) + 8 * (2 * D) + koff)));
        vt[dt][s_] = h8{t0[0], t0[1], t0[2], t0[3], t1[0], t1[1], t1[2], t1[3]};
    };
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) { load_v1(0, dt, 0); load_v1(0, dt, 1); }
#pragma unroll
    for (int c = 0; c < 8; ++c) p_pair(0, c);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(3);
#pragma unroll
    for (int mt = 0; mt < NT; ++mt) {
        if (mt <= last) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                if (mt == 0) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) st.o[dt][v] *= alpha;
                }
#pragma unroll
                for (int s_ = 0; s_ < 2; ++s_) {
                    const h8 pb = {ph[mt][4 * s_][0], ph[mt][4 * s_][1], ph[mt][4 * s_ + 1][0], ph[mt][4 * s_ + 1][1],
                                   ph[mt][4 * s_ + 2][0], ph[mt][4 * s_ + 2][1], ph[mt][4 * s_ + 3][0], ph[mt][4 * s_ + 3][1]};
                    st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vt[dt][s_], pb, st.o[dt], 0, 0, 0);
                    if (mt + 1 <= last) load_v1(mt + 1, dt, s_);
                }
                if (mt + 1 <= last) {
#pragma unroll
                    for (int q = 0; q < 8 / DT; ++q) p_pair(mt + 1, dt * (8 / DT) + q);
                }
            }
        }
    }
    __builtin_amdgcn_s_setprio(0);
    st.l = __builtin_fmaf(st.l, alpha, psum);
}

#endif  // __HIP_DEVICE_COMPILE__

// W wavefronts per SIMD: 2, or as many as the lean form of a block allows
template <int D, int W, bool CAUSAL, typename OutT>
__global__ __launch_bounds__(THREADS, W) void int_flash_attn_fwd_half_kernel(
    const int8_t *__restrict__ Q, const int8_t *__restrict__ K, const _Float16 *__restrict__ V,
    const float *__restrict__ sQ, const float *__restrict__ sK, int heads, int Nq, int Nk, int head_group, OutT *__restrict__ O) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ SmemH<D> sm;
    constexpr int DT = D / 32;

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T_r = (Nq + BR - 1) / BR;
    const int T_c = (Nk + BCH - 1) / BCH;
    // Under the mask the queries are the LAST Nq positions of the key sequence: query i sees keys <= i + shift.
    const int shift = CAUSAL ? Nk - Nq : 0;

    int head, qord;
    map_workgroup(blockIdx.x, heads, T_r, head_group, CAUSAL, head, qord);
    const int qb = CAUSAL ? (T_r - 1 - qord) : qord;
    const int q_local = 32 * wave + r;
    const int q_head = qb * BR + q_local;
    // rows past Nq are computed on a clamped copy of the last row and never stored
    const long qrow = static_cast<long>(head) * Nq + min(q_head, Nq - 1);

    const int8_t *Kh = K + static_cast<long>(head) * Nk * D;
    const _Float16 *Vh = V + static_cast<long>(head) * Nk * D;
    const float *sKh = sK + static_cast<long>(head) * Nk;
    const lds_ptr kbuf = (lds_ptr)(&sm.k[0][0]);
    const lds_ptr vbuf = (lds_ptr)(&sm.v[0][0]);
    const lds_ptr skbuf = (lds_ptr)(&sm.sk[0][0]);
    // key blocks this workgroup walks: up to the last key any of its queries sees
    const int first_q = qb * BR;
    const int nblocks = CAUSAL ? min(Nk - 1, first_q + BR - 1 + shift) / BCH + 1 : T_c;

    const BufRsrc rK = make_rsrc(Kh, static_cast<unsigned>(Nk) * D);
    const BufRsrc rV = make_rsrc(Vh, static_cast<unsigned>(Nk) * D * 2);
    const BufRsrc rSK = make_rsrc(sKh, static_cast<unsigned>(Nk) * 4);

    v4i qf[D / 32];
#pragma unroll
    for (int kk = 0; kk < D / 32; ++kk)
        qf[kk] = *reinterpret_cast<const v4i *>(Q + qrow * D + 32 * kk + 16 * g);
    const float sq = sQ[qrow];
    const bool far = W > 2 && __any(sq > FAR_SQ);                // (wave-uniform)
    const float sq2 = sq * (W == 2 || far ? LOG2E : LOG2E * ACC_UNIT);
    const LaneOffsetsH<D> lo(lane, wave);
    {
        const PrefetchH first = {rK, rV, rSK, 0, 0, 0, kbuf, vbuf, skbuf};
        prefetch_block<D>(first, lo, wave, lane);
    }

    [[maybe_unused]] v16i bias;                                  // (W = 2) constant registers the S^T accumulators start from
#pragma unroll
    for (int v = 0; v < 16; ++v) bias[v] = ACC_BIAS_I;
    if constexpr (W == 2) asm volatile("" : "+v"(bias));                               // opaque: kept in registers, not re-materialised per use

    auto lane_late = [&]() { return W == 2 ? lane : lane_index(); };   // after the loop over the unmasked blocks

    RowStateH<D> st;
    st.m2 = -INFINITY;
    st.l = 0.0f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) st.o[dt][v] = 0.0f;

    wait_all_memory();
    __syncthreads();

    // Blocks in which every key counts for every query of the workgroup come first; the rest (the two blocks that
    // meet the causal diagonal band of the workgroup's 128 queries, or the ragged last block) run the masked code.
    const int nfull = min(nblocks, CAUSAL ? min(Nk / BCH, (first_q + shift + 1) / BCH) : Nk / BCH);
    const int wave_last_q = first_q + 32 * wave + 31;            // last query of this wavefront
    auto next_block = [&](int jb) {                              // what block jb + 1 needs staged, into the other buffers
        const int nxt = (jb & 1) ^ 1, j1 = (jb + 1) * BCH;
        const bool more = jb + 1 < nblocks;
        return PrefetchH{rK, rV, rSK, more ? j1 * D : NOWHERE_H, more ? j1 * D * 2 : NOWHERE_H, more ? j1 * 4 : NOWHERE_H,
                         kbuf + nxt * BCH * D, vbuf + nxt * BCH * D * 2, skbuf + nxt * BCH * 4};
    };
    auto walk = [&](auto far_) {                                 // (as many barriers either way)
    [[maybe_unused]] constexpr bool FAR = decltype(far_)::value;
    for (int jb = 0; jb < nfull; ++jb) {
        const int cur = jb & 1;
        prefetch_block<D>(next_block(jb), lo, wave, lane);
        if constexpr (W == 2) process_block_half<D, false>(kbuf + cur * BCH * D, vbuf + cur * BCH * D * 2, skbuf + cur * BCH * 4, lo, qf, sq2,
                                                           0, NT - 1, NT, g, bias, st);
        else process_block_half_lean<D, false, FAR>(kbuf + cur * BCH * D, vbuf + cur * BCH * D * 2, skbuf + cur * BCH * 4, lo, qf, sq2, 0, NT - 1, NT, g, st);
        wait_all_memory();                                       // my part of the next block has landed in LDS
        __syncthreads();                                         // everyone's has, and `cur` is free again
    }
    for (int jb = nfull; jb < nblocks; ++jb) {
        const int cur = jb & 1;
        prefetch_block<D>(next_block(jb), lo, wave, lane_late());
        const int j0 = jb * BCH;
        const int tail = Nk - 1 - j0;                                              // last valid key of the block
        const int ln = lane_late(), g = ln >> 5;
        const int klimit = CAUSAL ? min(first_q + 32 * wave + (ln & 31) + shift - j0, tail) : tail;     // < 0: nothing kept
        const int wlim = CAUSAL ? min(wave_last_q + shift - j0, tail) : tail;
        const int last_tile = wlim < 0 ? -1 : min(NT - 1, wlim >> 5);
        const int wmin = CAUSAL ? min(wave_last_q - 31 + shift - j0, tail) : tail;   // klimit of the wavefront's first row
        if (last_tile >= 0) {                                                      // wave-uniform
            if constexpr (W == 2) process_block_half<D, true>(kbuf + cur * BCH * D, vbuf + cur * BCH * D * 2, skbuf + cur * BCH * 4, lo, qf, sq2,
                                                              klimit, last_tile, max(0, (wmin + 1) >> 5), g, bias, st);
            else process_block_half_lean<D, true, FAR>(kbuf + cur * BCH * D, vbuf + cur * BCH * D * 2, skbuf + cur * BCH * 4, lo, qf, sq2,
                                                  klimit, last_tile, max(0, (wmin + 1) >> 5), g, st);
        }
        wait_all_memory();
        __syncthreads();
    }
    };
    if (W > 2 && far) walk(std::bool_constant<(W > 2)>{});
    else walk(std::false_type{});

    const float l = st.l + swap32(st.l);
    const float f = 1.0f / l;
    // Every block ends with a barrier, so all of LDS is free here: each wavefront stages its 32 x D tile in its own
    // 64 D bytes of the V buffers and stores whole (fp32: half) rows.
    const int row0 = qb * BR + 32 * wave;                        // first query row of this wavefront
    OutT *orow0 = O + (static_cast<long>(head) * Nq + row0) * D;
    store_tile_staged<D, OutT>(vbuf + wave * (64 * D), orow0, Nq - row0, lane_late(), [&](int dt, int v) { return st.o[dt][v] * f; });
#endif
}

// ---- few queries, many keys -------------------------------------------------------------------------------------
// The half-INT8 counterpart of the few-query kernel of intfa_attention_fewq.hip: the wavefronts of a workgroup share one
// group of 32 queries and take FEW_NB key blocks of 64 keys at a time, in two roles that run one group of blocks apart.
//   2 FEW_NB S wavefronts (block b of the group, key tile t): lines 9-11 for that tile.  A wavefront copies the
//       K rows it reads itself, two groups ahead, and holds the operands of the next group in registers; the extrema of the tiles
//       meet in LDS (first barrier), then the weights go to LDS (second barrier);
//   four PV wavefronts (d tile): O = alpha O + P~ V and l for the group before, block by block in order, on weights and V^T operands
//       they have taken to registers by the first barrier; they also copy V, a group ahead.
// The running maximum in front of each block of 64 keys is that of the sequential walk and a lane's weights and sums are those of a lane
// of the kernel above, so the rows are the same, bit for bit: what a head gives does not depend on how many heads the call has.  (l in
// the S wavefronts, each its tile's part, was another order of that sum, and 32 x 1 x 4099 29.0 us against 27.0.)
// What bounds it is what one CU takes in (about 60 GB/s: 48 KB per group in 0.8 us at d = 128) and the chain of a group next to
// it.  Three blocks per group fill LDS and measure 4-8 % slower from 128 heads on.  DS = 2 (d = 128): two workgroups per query
// group, each with half of the d columns, as in the INT8 kernel (32 KB per group and CU).  One query against 4096 keys: 128
// heads 33.2 us = 6.1 TB/s (DS = 1: 38.6; 73.9 on the kernel above, which gives such a call one busy wavefront in four), 32 heads
// of 4099 28.9 (30.7, 73.9), 512 heads (DS = 1) 117 (144).
constexpr int FEW_BR = 32;         // queries per workgroup
constexpr int FEW_NB = 2;          // key blocks per group
constexpr int FEW_S_WAVES = 2 * FEW_NB;
constexpr int FEW_THREADS = (FEW_S_WAVES + 4) * 64;

template <int D, int DS> struct SmemFewH {
    alignas(4096) int8_t k[2][FEW_NB][BCH * D];
    alignas(4096) int8_t v[2][FEW_NB][BCH * (D / DS) * 2];
    alignas(128) float sk[2][FEW_S_WAVES][32];            // per S wavefront: the s_K of its key tile
    alignas(16) v4i p[FEW_NB][NT][2][64];                 // per block, key tile, 16-key step and lane: 8 weights
    alignas(16) float ext[2][FEW_NB][32][NT];             // per block, query and key tile: the maximum of a (line 10)
};
static_assert(sizeof(SmemFewH<128, 1>) <= 160 * 1024, "LDS budget");

template <int D, bool CAUSAL, typename OutT, int DS>
__global__ __launch_bounds__(FEW_THREADS) void int_flash_attn_fwd_half_few_kernel(
    const int8_t *__restrict__ Q, const int8_t *__restrict__ K, const _Float16 *__restrict__ V,
    const float *__restrict__ sQ, const float *__restrict__ sK, int heads, int Nq, int Nk, int once, OutT *__restrict__ O) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ SmemFewH<D, DS> sm;
    constexpr int KS = D / 32, NB = FEW_NB, DV = D / DS;

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qgroups = (Nq + FEW_BR - 1) / FEW_BR;
    const int shift = CAUSAL ? Nk - Nq : 0;
    int head, qg, half;
    if (!map_query_group<DS>(blockIdx.x, heads, qgroups, head, qg, half)) return;
    const int col0 = half * DV;                                  // first column of V and O
    const int first_q = qg * FEW_BR;
    const int q_head = first_q + r;
    const long qrow = static_cast<long>(head) * Nq + min(q_head, Nq - 1);   // rows past Nq: a clamped copy, never stored
    const float sq2 = sQ[qrow] * LOG2E;
    const int last_key = CAUSAL ? min(Nk - 1, min(first_q + FEW_BR, Nq) - 1 + shift) : Nk - 1;   // ... of any query of the group
    const int nblocks = last_key / BCH + 1;
    const int ngroups = (nblocks + NB - 1) / NB;
    float m2 = -INFINITY;                                        // running maximum in log2 units, kept in step by both roles
    struct Maxima { float v[NB]; };
    auto maxima = [&](int parity) {                              // line 10: the running maximum after each block of a group
        Maxima m;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float2 e = *reinterpret_cast<const float2 *>(&sm.ext[parity][b][r][0]);
            m2 = fmaxf(m2, fmaxf(e.x, e.y) * sq2);
            m.v[b] = m2;
        }
        return m;
    };

    if (wave < FEW_S_WAVES) {
        // ---- S wavefront: key tile t of block `blk` of every group
        constexpr int PER_GROUP = KS + 1;                        // copy instructions per group
        const int t = wave & 1, blk = wave >> 1;
        const BufRsrc rK = make_rsrc(K + static_cast<long>(head) * Nk * D, static_cast<unsigned>(Nk) * D);
        const BufRsrc rSK = make_rsrc(sK + static_cast<long>(head) * Nk, static_cast<unsigned>(Nk) * 4);
        const lds_ptr kbuf = (lds_ptr)(&sm.k[0][blk][0]);
        const lds_ptr skbuf = (lds_ptr)(&sm.sk[0][wave][0]);
        const LaneOffsetsH<D> lo(lane, 2 * t);                   // the pieces of tile t are those of wavefronts 2t, 2t + 1 of the kernel above
        // this wavefront's 32 rows of K and their s_K: it alone reads what it copies, so its own counted wait orders the
        // two.  Rows past the end come as zeros and are masked below; a group past the last one is requested nowhere, so
        // that every group costs PER_GROUP copies.
        auto stage_group = [&](int gi) {
            const int jb = gi * NB + blk;
            const bool real = jb < nblocks;
            const int koff = real ? jb * BCH * D : NOWHERE_H;
            const lds_ptr dst = kbuf + (gi & 1) * (NB * BCH * D) + t * (32 * D);
            if (once) lds_copy16_run<KS, true>(rK, dst, lo.gk, lo.gk, koff);
            else lds_copy16_run<KS>(rK, dst, lo.gk, lo.gk, koff);
            if (g == 0) lds_copy4(rSK, skbuf + (gi & 1) * (FEW_S_WAVES * 128), 4 * r + 128 * t, real ? jb * BCH * 4 : NOWHERE_H);
        };
        stage_group(0);
        stage_group(1);
        const int8_t *qptr = Q + qrow * D + 16 * g;
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
            const lds_ptr ks = kbuf + (gi & 1) * (NB * BCH * D), sk = skbuf + (gi & 1) * (FEW_S_WAVES * 128);
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) kop[kk] = *reinterpret_cast<LDS_AS const v4i *>(lds_xor(ks, 32 * kk, lo.k0) + 32 * t * D);
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) skv[vq] = *reinterpret_cast<LDS_AS const v4f *>(sk + 16 * g + 32 * vq);
        };
        v16i bias;
#pragma unroll
        for (int v = 0; v < 16; ++v) bias[v] = ACC_BIAS_I;
        wait_vmcnt<PER_GROUP>();
        __builtin_amdgcn_sched_barrier(0);
        read_group(0);
        wait_lds();
        for (int gi = 0; gi < ngroups; ++gi) {
            v16i sacc = bias;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) sacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kop[kk], qf[kk], sacc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            stage_group(gi + 2);                                 // under the MFMAs, into the place group gi has left
            __builtin_amdgcn_sched_barrier(0);
            const int j0 = (gi * NB + blk) * BCH;
            const int tail = Nk - 1 - j0;
            const int klimit = CAUSAL ? min(q_head + shift - j0, tail) : tail;         // kept keys: index inside the block <= klimit
            const bool masked = CAUSAL ? (j0 + BCH - 1 > min(first_q + shift, Nk - 1)) : (tail < BCH - 1);   // wave-uniform
            float a[16], bmax = -INFINITY;
            auto scale = [&](auto with_mask) {
#pragma unroll
                for (int vq = 0; vq < 4; ++vq)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float x = (__int_as_float(sacc[4 * vq + e]) - ACC_BIAS_F) * skv[vq][e];
                        if (decltype(with_mask)::value && (32 * t + 8 * vq + 4 * g + e > klimit)) x = -INFINITY;
                        a[4 * vq + e] = x;
                        bmax = fmaxf(bmax, x);
                    }
            };
            if (masked) scale(std::true_type{});
            else scale(std::false_type{});
            bmax = pair_max(bmax);
            if (g == 0) sm.ext[gi & 1][blk][r][t] = bmax;
            __syncthreads();
            const Maxima m = maxima(gi & 1);
            wait_vmcnt<PER_GROUP>();                        // group gi + 1 has landed (group gi + 2 may be in flight)
            __builtin_amdgcn_sched_barrier(0);
            read_group(gi + 1);
            float mb = m.v[0];
#pragma unroll
            for (int b = 1; b < NB; ++b) mb = blk == b ? m.v[b] : mb;
            h2 ph[8];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                ph[c] = h2{(_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(a[2 * c], sq2, -mb)),
                           (_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(a[2 * c + 1], sq2, -mb))};
#pragma unroll
            for (int s_ = 0; s_ < 2; ++s_) {
                const h8 pb = {ph[4 * s_][0], ph[4 * s_][1], ph[4 * s_ + 1][0], ph[4 * s_ + 1][1], ph[4 * s_ + 2][0], ph[4 * s_ + 2][1], ph[4 * s_ + 3][0], ph[4 * s_ + 3][1]};
                sm.p[blk][t][s_][lane] = __builtin_bit_cast(v4i, pb);
            }
            wait_lds();                                          // (the operands of group gi + 1 are in registers too)
            __syncthreads();
        }
        wait_all_memory();                                       // requests past the last group: nothing of mine stays in flight
        __syncthreads();                                         // the PV wavefronts' last group
        return;
    }

    // ---- PV wavefront: d tile dt of O^T = V^T P~^T, one group of blocks behind
    const int dt = wave - FEW_S_WAVES;
    // V ends for this workgroup with the last key tile that a query of the group sees: what lies behind comes as zeros.  Its
    // weights are 0, but 0 times an infinity or a NaN of the caller's V is not (the kernel above leaves such a tile out).
    const BufRsrc rV = make_rsrc(V + static_cast<long>(head) * Nk * D, static_cast<unsigned>(min(Nk, (last_key | 31) + 1)) * D * 2);
    const lds_ptr vbuf = (lds_ptr)(&sm.v[0][0][0]);
    const LaneOffsetsH<DV> lo(lane, dt);
    // With DS = 2 a row of the tile is a half row of V: the copies of LaneOffsetsH<DV> with the row stride of V (a piece is
    // 512 / DV = 8 rows, which its swizzle does not see).
    constexpr int PIECES = DV / 32;
    const int srow = dt * 16 + lane / (DV / 8);
    const unsigned gvs = DS == 1 ? lo.gv : srow * (2 * D) + 2 * col0 + 16 * ((lane % (DV / 8)) ^ (vh_swz<DV>(srow) << 2));
    // V of group gi (this wavefront's quarter of every block); a block past the last one is requested nowhere and comes as
    // zeros, so that every group costs NB * PIECES copies
    auto stage_group = [&](int gi) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int jb = gi * NB + b;
            const int voff = jb < nblocks ? jb * BCH * D * 2 : NOWHERE_H;
            const lds_ptr dst = vbuf + ((gi & 1) * NB + b) * (BCH * DV * 2) + dt * PIECES * 1024;
            auto copy = [&](auto nt) {
                if constexpr (DS == 1) lds_copy16_run<PIECES, decltype(nt)::value>(rV, dst, gvs, gvs, voff);
                else {
#pragma unroll
                    for (int i = 0; i < PIECES; ++i) lds_copy16<decltype(nt)::value>(rV, dst + i * 1024, gvs, voff + 1024 * DS * i);
                }
            };
            if (once) copy(std::true_type{});
            else copy(std::false_type{});
        }
    };
    v16f o;
#pragma unroll
    for (int v = 0; v < 16; ++v) o[v] = 0.0f;
    const bool works = dt < PIECES;                              // two d tiles in a half (or D = 64): the other wavefronts only copy
    h8 vop[NB][4], pf[NB][4];
    float l = 0.0f;                                              // of this lane's keys, added up in the order of the kernel above
    const h2 ones = {(_Float16)1.0f, (_Float16)1.0f};
    auto block = [&](int b, float m_prev, float m_new) {         // (a block past the last one: the maximum stays, the weights are 0)
        const float alpha = __builtin_amdgcn_exp2f(m_prev - m_new);
        float psum = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) psum = __builtin_amdgcn_fdot2(h2{pf[b][i][2 * j], pf[b][i][2 * j + 1]}, ones, psum, false);
        l = __builtin_fmaf(l, alpha, psum);
#pragma unroll
        for (int v = 0; v < 16; ++v) o[v] *= alpha;
#pragma unroll
        for (int i = 0; i < 4; ++i) o = __builtin_amdgcn_mfma_f32_32x32x16_f16(vop[b][i], pf[b][i], o, 0, 0, 0);
    };
    stage_group(0);
    for (int gi = 0; gi <= ngroups; ++gi) {
        const float m_before = m2;
        Maxima m = {};
        if (gi > 0 && works) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const lds_ptr vs = vbuf + (((gi - 1) & 1) * NB + b) * (BCH * DV * 2);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const h4 t0 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s4 *>(lds_xor(vs, 64 * dt, lo.v0) + 16 * i * (2 * DV))));
                    const h4 t1 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s4 *>(lds_xor(vs, 64 * dt, lo.v0) + (16 * i + 8) * (2 * DV))));
                    vop[b][i] = h8{t0[0], t0[1], t0[2], t0[3], t1[0], t1[1], t1[2], t1[3]};
                    pf[b][i] = __builtin_bit_cast(h8, sm.p[b][i >> 1][i & 1][lane]);
                }
            }
            m = maxima((gi - 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            block(0, m_before, m.v[0]);
        }
        __syncthreads();
        if (gi < ngroups) stage_group(gi + 1);
        if (gi > 0 && works) {
#pragma unroll
            for (int b = 1; b < NB; ++b) block(b, m.v[b - 1], m.v[b]);
        }
        if (gi < ngroups) {
            wait_vmcnt<NB * PIECES>();                        // my part of V of group gi has landed (group gi + 1 may be in flight)
            __syncthreads();                                     // everyone's has, and the weights of group gi are in LDS
        }
    }
    wait_all_memory();

    if (q_head < Nq && works) {
        const float f = 1.0f / (l + swap32(l));
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

template <int D, bool CAUSAL, typename OutT>
int launch_half(const int8_t *Q, const int8_t *K, const _Float16 *V, const float *sQ, const float *sK, int heads, int Nq, int Nk,
                void *O, hipStream_t st) {
    // as for INT8, this kernel / the one below, us.  d = 128: 32 heads x 256 queries x 8192 keys 64 / 145, x 512 119 / 145, x 700 184 / 146;
    // 512 x 32 x 2048 66 / 79, x 64 94 / 81; short keys 512 x 1 x 128 9.6 / 8.8, 2000 x 32 x 256 53 / 51, 2000 x 1 x 384 54 / 62.
    // d = 64: 2000 x 1 x 64 15.0 / 13.1, x 128 17.4 / 19.2, 32 x 512 x 2048 20 / 33.
    if (ifa_few_queries(heads, Nq, Nk, D, true)) {
        const long qgroups = (Nq + FEW_BR - 1) / FEW_BR, padded = (heads * qgroups + 7) / 8 * 8;
        // the non-temporal hint where K and V are read once and do not stay in the caches, here with DS = 2 as well, us after the same call /
        // after a copy of 512 MB / right after K was quantized and V written: 128 x 1 x 4096, 101 MB, 32 / 41 / 36, without it 32 / 61 / 41;
        // 128 x 1 x 16384 138 / 157 / 174 and 141 / 167 / 172
        const int once = qgroups == 1 && 3L * heads * Nk * D > (64L << 20);
        auto launch = [&](auto ds) {
            constexpr int DS = decltype(ds)::value;
            hipLaunchKernelGGL((int_flash_attn_fwd_half_few_kernel<D, CAUSAL, OutT, DS>), dim3(static_cast<unsigned>(padded * DS)), dim3(FEW_THREADS), 0,
                               st, Q, K, V, sQ, sK, heads, Nq, Nk, once, static_cast<OutT *>(O));
        };
        if constexpr (D == 128) {
            // two workgroups per query group as long as each then has a CU of its own (160 heads x 1 x 4096: 40 us with one, 57 with two)
            if (heads * qgroups <= 128) launch(std::integral_constant<int, 2>{});
            else launch(std::integral_constant<int, 1>{});
        } else launch(std::integral_constant<int, 1>{});
        return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
    }
    const int T_r = (Nq + BR - 1) / BR;
    const long wgs = static_cast<long>(heads) * T_r;
    // T_r = 0: under the mask this kernel keeps 4 heads per group (8 measured 4-17 % slower here at N = 1280 .. 2048)
    const int head_group = head_group_for(CAUSAL, 3L * Nk * D, 0);
    auto launch = [&](auto w) {
        hipLaunchKernelGGL((int_flash_attn_fwd_half_kernel<D, decltype(w)::value, CAUSAL, OutT>), dim3(static_cast<unsigned>(wgs)), dim3(THREADS), 0,
                           st, Q, K, V, sQ, sK, heads, Nq, Nk, head_group, static_cast<OutT *>(O));
    };
    if (ifa_half_wavefronts(heads, Nq, Nk, D, CAUSAL, head_group) > 2) launch(std::integral_constant<int, D == 64 ? 4 : 3>{});
    else launch(std::integral_constant<int, 2>{});
    return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
}

template <int D, bool CAUSAL>
int launch_half_dtype(const int8_t *Q, const int8_t *K, const _Float16 *V, const float *sQ, const float *sK, int heads,
                      int Nq, int Nk, void *O, int o_dtype, hipStream_t st) {
    switch (o_dtype) {
    case IFA_F32: return launch_half<D, CAUSAL, float>(Q, K, V, sQ, sK, heads, Nq, Nk, O, st);
    case IFA_F16: return launch_half<D, CAUSAL, __half>(Q, K, V, sQ, sK, heads, Nq, Nk, O, st);
    default: return launch_half<D, CAUSAL, __hip_bfloat16>(Q, K, V, sQ, sK, heads, Nq, Nk, O, st);
    }
}

}  // namespace

extern "C" int ifa_block_cols_half(int d, int causal) {
    (void)causal;
    return (d == 64 || d == 128) ? BCH : 0;
}

namespace {
int half_entry(const signed char *Q_i8, const signed char *K_i8, const void *V_f16, const float *s_Q, const float *s_K,
               int B, int H, int Nq, int Nk, int d, int causal, void *O, int o_dtype, void *hip_stream) {
    if (!Q_i8 || !K_i8 || !V_f16 || !s_Q || !s_K || !O) return IFA_ERR_NULL;
    if (B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0 || d <= 0) return IFA_ERR_SHAPE;
    const long heads = static_cast<long>(B) * H;
    const int N = Nq > Nk ? Nq : Nk;
    if (heads > (1L << 40) / N / d) return IFA_ERR_SHAPE;
    if (o_dtype < IFA_F32 || o_dtype > IFA_BF16) return IFA_ERR_DTYPE;
    if (d != 64 && d != 128) return IFA_ERR_UNSUPPORTED;
    if (causal && Nk < Nq) return IFA_ERR_UNSUPPORTED;           // a query with no visible key
    if (static_cast<long>(N) * d * 2 > 0x7ff00000L || heads * ((N + BR - 1) / BR) > 0x7fffffffL) return IFA_ERR_UNSUPPORTED;
    if (!ifa_aligned16(Q_i8) || !ifa_aligned16(K_i8) || !ifa_aligned16(V_f16) || !ifa_aligned16(O) ||
        (reinterpret_cast<uintptr_t>(s_Q) & 3) || (reinterpret_cast<uintptr_t>(s_K) & 3))
        return IFA_ERR_UNSUPPORTED;
    const int8_t *Q = reinterpret_cast<const int8_t *>(Q_i8);
    const int8_t *K = reinterpret_cast<const int8_t *>(K_i8);
    const _Float16 *V = reinterpret_cast<const _Float16 *>(V_f16);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int hd = static_cast<int>(heads);
    if (d == 128)
        return causal ? launch_half_dtype<128, true>(Q, K, V, s_Q, s_K, hd, Nq, Nk, O, o_dtype, st)
                      : launch_half_dtype<128, false>(Q, K, V, s_Q, s_K, hd, Nq, Nk, O, o_dtype, st);
    return causal ? launch_half_dtype<64, true>(Q, K, V, s_Q, s_K, hd, Nq, Nk, O, o_dtype, st)
                  : launch_half_dtype<64, false>(Q, K, V, s_Q, s_K, hd, Nq, Nk, O, o_dtype, st);
}
}  // namespace

extern "C" int int_flash_attn_fwd_half(const signed char *Q_i8, const signed char *K_i8, const void *V_f16,
                                       const float *s_Q, const float *s_K, int B, int H, int N, int d, int causal,
                                       void *O, int o_dtype, void *hip_stream) {
    return half_entry(Q_i8, K_i8, V_f16, s_Q, s_K, B, H, N, N, d, causal, O, o_dtype, hip_stream);
}

extern "C" int int_flash_attn_fwd_half_rect(const signed char *Q_i8, const signed char *K_i8, const void *V_f16,
                                            const float *s_Q, const float *s_K, int B, int H, int Nq, int Nk, int d,
                                            int causal, void *O, int o_dtype, void *hip_stream) {
    return half_entry(Q_i8, K_i8, V_f16, s_Q, s_K, B, H, Nq, Nk, d, causal, O, o_dtype, hip_stream);
}

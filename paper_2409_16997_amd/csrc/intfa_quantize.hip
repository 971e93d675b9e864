// Symmetric INT8 quantizers of Section 3.2 (S = absmax / R, R = 127), gfx950.
//
// Both are HBM-streaming kernels: every element is read once (twice for V, whose scale needs
// the whole head first) and written once as a byte.  A lane owns 8 consecutive elements, so
// loads are 128-bit for fp16/bf16 and 2 x 128-bit for fp32, stores are 64-bit, and a row of
// d elements is d/8 adjacent lanes whose absmax is combined with DPP lane shuffles.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <hip/hip_bf16.h>
#include <stdint.h>
#include <type_traits>

#include "intfa.h"
#include "intfa_internal.h"

namespace {

// ---- 8 consecutive elements of any supported dtype, as loaded and widened exactly to fp32 -------
template <typename T> struct Raw8 {                   // fp16, bf16: one 128-bit load
    uint4 raw;
    // held as loaded: the compiler may not keep the widened values (twice the registers) in its place
    __device__ __forceinline__ void hold() { asm volatile("" : "+v"(raw.x), "+v"(raw.y), "+v"(raw.z), "+v"(raw.w)); }
    template <typename I> __device__ __forceinline__ void load(const void *p, I idx) { raw = *reinterpret_cast<const uint4 *>(static_cast<const T *>(p) + idx); }
    template <typename I> __device__ __forceinline__ void load_once(const void *p, I idx) {      // with the non-temporal hint
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        const u4 v = __builtin_nontemporal_load(reinterpret_cast<const u4 *>(static_cast<const T *>(p) + idx));
        raw = make_uint4(v[0], v[1], v[2], v[3]);
    }
    __device__ __forceinline__ void widen(float (&x)[8]) const {
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (std::is_same_v<T, __half>) {
                const float2 f = __half22float2(__builtin_bit_cast(__half2, w[i]));
                x[2 * i] = f.x;
                x[2 * i + 1] = f.y;
            } else {                                  // bf16 -> fp32 is a 16-bit shift
                x[2 * i] = __uint_as_float(w[i] << 16);
                x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
            }
        }
    }
};
template <> struct Raw8<float> {
    float4 a, b;
    __device__ __forceinline__ void hold() {
        asm volatile("" : "+v"(a.x), "+v"(a.y), "+v"(a.z), "+v"(a.w), "+v"(b.x), "+v"(b.y), "+v"(b.z), "+v"(b.w));
    }
    template <typename I> __device__ __forceinline__ void load_once(const void *p, I idx) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        const f4 *q = reinterpret_cast<const f4 *>(static_cast<const float *>(p) + idx);
        const f4 v = __builtin_nontemporal_load(q), w = __builtin_nontemporal_load(q + 1);
        a = make_float4(v[0], v[1], v[2], v[3]);
        b = make_float4(w[0], w[1], w[2], w[3]);
    }
    template <typename I> __device__ __forceinline__ void load(const void *p, I idx) {
        const float4 *q = reinterpret_cast<const float4 *>(static_cast<const float *>(p) + idx);
        a = q[0];
        b = q[1];
    }
    __device__ __forceinline__ void widen(float (&x)[8]) const {
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    }
};
template <typename T, typename I> __device__ __forceinline__ void load8(const void *p, I idx, float (&x)[8]) {
    Raw8<T> r;
    r.load(p, idx);
    r.widen(x);
}

__device__ __forceinline__ float absmax8(const float (&x)[8]) {
    float a = fmaxf(fabsf(x[0]), fabsf(x[1]));
#pragma unroll
    for (int i = 2; i < 8; ++i) a = fmaxf(a, fabsf(x[i]));
    return a;
}

// q = clamp(rint(x * inv), -127, 127) for 8 values, packed little-endian into two dwords.
__device__ __forceinline__ uint2 quant8(const float (&x)[8], float inv) {
    uint32_t w[2] = {0u, 0u};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float t = rintf(x[i] * inv);
        t = fminf(fmaxf(t, -127.0f), 127.0f);
        w[i >> 2] |= (static_cast<uint32_t>(static_cast<int>(t)) & 0xffu) << (8 * (i & 3));
    }
    return make_uint2(w[0], w[1]);
}

// max over the aligned group of `LPR` adjacent lanes (LPR a power of two <= 64), result in all.
template <int LPR>
__device__ __forceinline__ float group_max(float a) {
    // quad_perm [1,0,3,2] and [2,3,0,1], then mirrors inside 8 and 16 lanes: DPP, no LDS.
    if (LPR >= 2) a = fmaxf(a, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a), 0xB1, 0xf, 0xf, true)));
    if (LPR >= 4) a = fmaxf(a, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a), 0x4E, 0xf, 0xf, true)));
    if (LPR >= 8) a = fmaxf(a, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a), 0x141, 0xf, 0xf, true)));  // row_half_mirror
    if (LPR >= 16) a = fmaxf(a, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a), 0x140, 0xf, 0xf, true))); // row_mirror
    if (LPR >= 32) a = fmaxf(a, __shfl_xor(a, 16));
    if (LPR >= 64) a = fmaxf(a, __shfl_xor(a, 32));
    return a;
}

// value held by lane ^ M (M a power of two < 64): DPP inside a quad, the LDS crossbar (no memory access) beyond
template <int M> __device__ __forceinline__ float lane_xor(float x) {
    const int v = __float_as_int(x);
    if (M == 1) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true));        // quad_perm [1,0,3,2]
    if (M == 2) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true));        // quad_perm [2,3,0,1]
    if (M == 4) return __int_as_float(__builtin_amdgcn_ds_swizzle(v, 0x101F));                   // bit mode: xor 4
    if (M == 8) return __int_as_float(__builtin_amdgcn_ds_swizzle(v, 0x201F));
    if (M == 16) return __int_as_float(__builtin_amdgcn_ds_swizzle(v, 0x401F));
    return __shfl_xor(x, 32);
}

// One butterfly stage of the Walsh-Hadamard transform across lanes: elements 8*sub + i and 8*(sub ^ M) + i.
// The lane with bit M clear holds a and keeps a + b, the other holds b and keeps a - b.
template <int M, int LPR> __device__ __forceinline__ void hadamard_lane_stage(float (&x)[8], int sub) {
    if (M < LPR) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float p = lane_xor<M>(x[i]);
            x[i] = (sub & M) ? (p - x[i]) : (x[i] + p);
        }
    }
}

// Unnormalized Walsh-Hadamard transform (Sylvester order) of a row of 8*LPR elements spread over LPR lanes,
// stages h = 1, 2, 4 inside the lane's 8 registers, then h = 8, 16, ... across lanes, all in fp32.
template <int LPR> __device__ __forceinline__ void hadamard_row(float (&x)[8], int sub) {
#pragma unroll
    for (int h = 1; h < 8; h <<= 1)
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if ((i & h) == 0) {
                const float a = x[i], b = x[i + h];
                x[i] = a + b;
                x[i + h] = a - b;
            }
    hadamard_lane_stage<1, LPR>(x, sub);
    hadamard_lane_stage<2, LPR>(x, sub);
    hadamard_lane_stage<4, LPR>(x, sub);
    hadamard_lane_stage<8, LPR>(x, sub);
    hadamard_lane_stage<16, LPR>(x, sub);
    hadamard_lane_stage<32, LPR>(x, sub);
}

// ---- token-level: one row = LPR lanes ---------------------------------------------------------
struct TokenJob {
    const void *X;
    int8_t *Xq;
    float *scale;
    float scale_mul;
};
// Rows row0, row0 + row_stride, ... of one tensor; the caller's LPR adjacent lanes `sub` = 0 .. LPR - 1 share a row.
// ONCE: the loads carry the non-temporal hint.
template <typename T, int LPR, bool HADAMARD, bool ONCE = false>
__device__ __forceinline__ void quantize_token_rows(const TokenJob &job, long rows, long row0, long row_stride, int sub) {
    for (long row = row0; row < rows; row += row_stride) {
        float x[8];
        const long idx = row * (LPR * 8) + sub * 8;
        Raw8<T> raw;
        if (ONCE) raw.load_once(job.X, idx);
        else raw.load(job.X, idx);
        raw.widen(x);
        if (HADAMARD) hadamard_row<LPR>(x, sub);
        const float a = group_max<LPR>(absmax8(x));
        const float inv = (a == 0.0f) ? 0.0f : 127.0f / a;
        *reinterpret_cast<uint2 *>(job.Xq + idx) = quant8(x, inv);
        if (sub == 0) job.scale[row] = ((a == 0.0f) ? 1.0f : a / 127.0f) * job.scale_mul;
    }
}

// One launch serves up to two tensors of the same shape (Q and K of a step): blockIdx.y picks the job.
template <typename T, int LPR, bool HADAMARD>
__global__ __launch_bounds__(256) void quantize_tokenwise_kernel(TokenJob j0, TokenJob j1, long rows) {
    constexpr int ROWS_PER_BLOCK = 256 / LPR;
    const TokenJob job = blockIdx.y == 0 ? j0 : j1;
    quantize_token_rows<T, LPR, HADAMARD>(job, rows, static_cast<long>(blockIdx.x) * ROWS_PER_BLOCK + threadIdx.x / LPR,
                                          static_cast<long>(gridDim.x) * ROWS_PER_BLOCK, threadIdx.x % LPR);
}

// ---- tensor-level, one scale per head ----------------------------------------------------------
// A head's absmax has to be known before its first code.  Three ways, none with atomics or slots to clear:
//   shares several workgroups per head take the absmax of all of it, each writes the codes of its share; one launch;
//   whole  one workgroup of HEAD_THREADS takes the whole head, keeps its first KEEP_BYTES in registers and reads the rest a
//          second time right after the first, out of the caches; one launch;
//   parts  `parts` workgroups per head leave the absmax of their part (fp32 bits) at the START of each of the `regions`
//          the second launch cuts the head's codes into: a workgroup of that launch reads the words in front of its own
//          region before it writes its codes over them, so nobody else's words are touched and no third launch is needed.
constexpr int HEAD_THREADS = 1024, SHORT_HEAD_THREADS = 256;
template <typename T> constexpr int LOADS_IN_FLIGHT = sizeof(T) == 2 ? 4 : 2;   // chunks of 8 per thread
constexpr int KEEP_BYTES = 96 << 10;   // 24 registers per thread: two workgroups per CU
struct HeadJob {
    const void *X;                 // [heads, per_head]
    int8_t *Xq;
    float *scale;                  // [heads]
    long per_head;
    int heads, parts, regions;     // parts = 0: whole heads, by `shares` workgroups each
    int shares;
    long chunks_per_part, chunks_per_region;   // in chunks of 8 elements; the last part and region take the remainder (shares: chunks_per_region each)
};

template <int THREADS> __device__ __forceinline__ float workgroup_max(float a) {
    __shared__ float wmax[THREADS / 64];
    a = group_max<64>(a);
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = a;
    __syncthreads();
    a = wmax[0];
#pragma unroll
    for (int i = 1; i < THREADS / 64; ++i) a = fmaxf(a, wmax[i]);
    return a;
}

template <typename T, int THREADS> __device__ __forceinline__ void head_whole(const HeadJob &hj, long head) {
    constexpr int KEEP = sizeof(T) == 2 ? KEEP_BYTES / 16384 : KEEP_BYTES / 32768;   // chunks per thread
    constexpr int U = LOADS_IN_FLIGHT<T>;
    const T *X = static_cast<const T *>(hj.X) + head * hj.per_head;
    int8_t *Xq = hj.Xq + head * hj.per_head;
    const int chunks = static_cast<int>(hj.per_head / 8), tid = threadIdx.x;   // 32-bit offsets from a uniform base
    Raw8<T> keep[KEEP];
    float a = 0.0f, x[8];
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
        if (tid + i * THREADS < chunks) keep[i].load(X, 8 * (tid + i * THREADS));
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
        if (tid + i * THREADS < chunks) {
            keep[i].widen(x);
            a = fmaxf(a, absmax8(x));
        }
    const int first = KEEP * THREADS + tid;
    int c = first;
    for (; c + (U - 1) * THREADS < chunks; c += U * THREADS) {
        Raw8<T> r[U];
#pragma unroll
        for (int i = 0; i < U; ++i) r[i].load(X, 8 * (c + i * THREADS));
#pragma unroll
        for (int i = 0; i < U; ++i) {
            r[i].widen(x);
            a = fmaxf(a, absmax8(x));
        }
    }
    for (; c < chunks; c += THREADS) {
        load8<T>(X, 8 * c, x);
        a = fmaxf(a, absmax8(x));
    }
    a = workgroup_max<THREADS>(a);
#pragma unroll
    for (int i = 0; i < KEEP; ++i) keep[i].hold();
    const float inv = (a == 0.0f) ? 0.0f : 127.0f / a;
    if (tid == 0) hj.scale[head] = (a == 0.0f) ? 1.0f : a / 127.0f;
    // backwards: what was read last is nearest
    for (c -= THREADS; c - (U - 1) * THREADS >= first; c -= U * THREADS) {
        Raw8<T> r[U];
#pragma unroll
        for (int i = 0; i < U; ++i) r[i].load(X, 8 * (c - i * THREADS));
#pragma unroll
        for (int i = 0; i < U; ++i) {
            r[i].widen(x);
            *reinterpret_cast<uint2 *>(Xq + 8 * (c - i * THREADS)) = quant8(x, inv);
        }
    }
    for (; c >= first; c -= THREADS) {
        load8<T>(X, 8 * c, x);
        *reinterpret_cast<uint2 *>(Xq + 8 * c) = quant8(x, inv);
    }
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
        if (tid + i * THREADS < chunks) {
            keep[i].widen(x);
            *reinterpret_cast<uint2 *>(Xq + 8 * (tid + i * THREADS)) = quant8(x, inv);
        }
}

// shares > 1: every one of a head's workgroups takes the absmax of the whole head, beginning with the share whose codes it writes, which stays in
// registers.  They run on one XCD (8 apart), so what one brings in the others find in its L2: a CU takes in 59 GB/s from beyond it, 120 - 140 out of it.
// (What it measures: plan_heads().)
template <typename T> __device__ __forceinline__ void head_share(const HeadJob &hj, long head, int share) {
    constexpr int KEEP = sizeof(T) == 2 ? KEEP_BYTES / 16384 : KEEP_BYTES / 32768;   // chunks per thread
    constexpr int U = LOADS_IN_FLIGHT<T>;
    const T *X = static_cast<const T *>(hj.X) + head * hj.per_head;
    int8_t *Xq = hj.Xq + head * hj.per_head;
    const int chunks = static_cast<int>(hj.per_head / 8), tid = threadIdx.x, size = static_cast<int>(hj.chunks_per_region);
    const int c0 = share * size, c1 = min(chunks, c0 + size);
    Raw8<T> keep[KEEP];
    float a = 0.0f, x[8];
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
        if (c0 + tid + i * HEAD_THREADS < c1) keep[i].load(X, 8 * (c0 + tid + i * HEAD_THREADS));
    // the rest of the head, from the end of the share on and round to its beginning
    const int rest = chunks - (c1 - c0);
    auto place = [&](int j) { return c1 + j < chunks ? c1 + j : c1 + j - chunks; };
    int j = tid;
    for (; j + (U - 1) * HEAD_THREADS < rest; j += U * HEAD_THREADS) {
        Raw8<T> r[U];
#pragma unroll
        for (int i = 0; i < U; ++i) r[i].load(X, 8 * place(j + i * HEAD_THREADS));
#pragma unroll
        for (int i = 0; i < U; ++i) {
            r[i].widen(x);
            a = fmaxf(a, absmax8(x));
        }
    }
    for (; j < rest; j += HEAD_THREADS) {
        load8<T>(X, 8 * place(j), x);
        a = fmaxf(a, absmax8(x));
    }
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
        if (c0 + tid + i * HEAD_THREADS < c1) {
            keep[i].widen(x);
            a = fmaxf(a, absmax8(x));
        }
    a = workgroup_max<HEAD_THREADS>(a);
#pragma unroll
    for (int i = 0; i < KEEP; ++i) keep[i].hold();
    const float inv = (a == 0.0f) ? 0.0f : 127.0f / a;
    if (share == 0 && tid == 0) hj.scale[head] = (a == 0.0f) ? 1.0f : a / 127.0f;
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
        if (c0 + tid + i * HEAD_THREADS < c1) {
            keep[i].widen(x);
            *reinterpret_cast<uint2 *>(Xq + 8 * (c0 + tid + i * HEAD_THREADS)) = quant8(x, inv);
        }
}

template <typename T> __device__ __forceinline__ void head_part_absmax(const HeadJob &hj, long head, int part) {
    constexpr int U = LOADS_IN_FLIGHT<T>;
    const long base = head * hj.per_head, chunks = hj.per_head / 8;
    const long c1 = part + 1 < hj.parts ? (part + 1) * hj.chunks_per_part : chunks;
    float a = 0.0f, x[8];
    long c = part * hj.chunks_per_part + threadIdx.x;
    for (; c + (U - 1) * HEAD_THREADS < c1; c += U * HEAD_THREADS) {
        Raw8<T> r[U];
#pragma unroll
        for (int i = 0; i < U; ++i) r[i].load(hj.X, base + 8 * (c + i * HEAD_THREADS));
#pragma unroll
        for (int i = 0; i < U; ++i) {
            r[i].widen(x);
            a = fmaxf(a, absmax8(x));
        }
    }
    for (; c < c1; c += HEAD_THREADS) {
        load8<T>(hj.X, base + 8 * c, x);
        a = fmaxf(a, absmax8(x));
    }
    a = workgroup_max<HEAD_THREADS>(a);
    for (int r = threadIdx.x; r < hj.regions; r += HEAD_THREADS)
        reinterpret_cast<float *>(hj.Xq + base + 8 * r * hj.chunks_per_region)[part] = a;
}

// What workgroup `wg` of a launch does for V before any row of Q and K is touched; the number of such workgroups is head_workgroups().
template <typename T> __device__ __forceinline__ void head_first_pass(const HeadJob &hj, int wg) {
    if (hj.shares > 1) {
        const int unit = wg >> 3, head = unit / hj.shares * 8 + (wg & 7);
        if (head < hj.heads) head_share<T>(hj, head, unit % hj.shares);
    } else if (hj.parts == 0) head_whole<T, HEAD_THREADS>(hj, wg);
    else head_part_absmax<T>(hj, wg / hj.parts, wg % hj.parts);
}
template <typename T> __global__ __launch_bounds__(HEAD_THREADS, 8) void head_first_pass_kernel(HeadJob hj) {
    head_first_pass<T>(hj, static_cast<int>(blockIdx.x));
}

template <typename T> __global__ __launch_bounds__(SHORT_HEAD_THREADS, 8) void short_head_kernel(HeadJob hj) {
    head_whole<T, SHORT_HEAD_THREADS>(hj, blockIdx.x);
}

// Second launch of `parts`: one workgroup per (region, head).
template <typename T> __global__ __launch_bounds__(256) void head_quantize_regions_kernel(HeadJob hj) {
    const long head = blockIdx.y, base = head * hj.per_head, chunks = hj.per_head / 8;
    const long c0 = blockIdx.x * hj.chunks_per_region, c1 = static_cast<int>(blockIdx.x) + 1 < hj.regions ? c0 + hj.chunks_per_region : chunks;
    const float *words = reinterpret_cast<const float *>(hj.Xq + base + 8 * c0);
    float a = 0.0f;
    for (int p = 0; p < hj.parts; ++p) a = fmaxf(a, words[p]);
    const float inv = (a == 0.0f) ? 0.0f : 127.0f / a;
    __syncthreads();                                             // every thread has read the words its workgroup now overwrites
    for (long c = c0 + threadIdx.x; c < c1; c += 256) {
        float x[8];
        load8<T>(hj.X, base + 8 * c, x);
        *reinterpret_cast<uint2 *>(hj.Xq + base + 8 * c) = quant8(x, inv);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) hj.scale[head] = (a == 0.0f) ? 1.0f : a / 127.0f;
}

// Q and K token-level and the first pass of V in one launch.  Bound by HBM: 3 elements in and 3 bytes out each, and V a
// second time as far as the caches do not hold it.  The workgroups of V come first: a whole head is the longest piece of
// work in the launch, and the rows of Q and K fill in around it.  `once`: Q and K are read past the caches, which leaves
// more of V there for its second read.  128 heads x 4096 x 128 fp16: 124 us (4.9 TB/s of 604 MB; a plain copy of 1 GiB
// reaches 5.0 on this card), 135 as three launches with V's passes apart; without the hint 130; 64 heads x 1024 x 64: 10.4 us,
// before 13.9; one head of 128 x 64 fp32: 5 us, before 14.4.
template <typename T, int LPR>
__global__ __launch_bounds__(HEAD_THREADS, 8) void quantize_qkv_kernel(TokenJob jq, TokenJob jk, long rows, HeadJob hj, int head_wgs, int once) {
    constexpr int ROWS_PER_BLOCK = HEAD_THREADS / LPR;
    if (static_cast<int>(blockIdx.x) < head_wgs) {
        head_first_pass<T>(hj, static_cast<int>(blockIdx.x));
        return;
    }
    const int wg = static_cast<int>(blockIdx.x) - head_wgs, per_tensor = (static_cast<int>(gridDim.x) - head_wgs) / 2;
    const TokenJob job = wg < per_tensor ? jq : jk;
    const long row0 = static_cast<long>(wg < per_tensor ? wg : wg - per_tensor) * ROWS_PER_BLOCK + threadIdx.x / LPR;
    const long stride = static_cast<long>(per_tensor) * ROWS_PER_BLOCK;
    if (once) quantize_token_rows<T, LPR, false, true>(job, rows, row0, stride, threadIdx.x % LPR);
    else quantize_token_rows<T, LPR, false>(job, rows, row0, stride, threadIdx.x % LPR);
}

// ---- tensor-level, one scale for the whole array -------------------------------------------------
// |x| >= 0, so the fp32 bit pattern orders like the value and an integer atomic max works.
template <typename T>
__global__ __launch_bounds__(256) void array_absmax_kernel(const void *__restrict__ X, long n, unsigned *__restrict__ slot) {
    float a = 0.0f;
    for (long i = (static_cast<long>(blockIdx.x) * 256 + threadIdx.x) * 8; i < n; i += static_cast<long>(gridDim.x) * 256 * 8) {
        float x[8];
        load8<T>(X, i, x);
        a = fmaxf(a, absmax8(x));
    }
    a = workgroup_max<256>(a);
    // Atomics on one address serialise: look first.  The slot only grows, so a value read here, however stale, is a
    // lower bound of the final one and skipping below it loses nothing.
    if (threadIdx.x == 0 && __float_as_uint(a) > __builtin_nontemporal_load(slot)) atomicMax(slot, __float_as_uint(a));
}

template <typename T>
__global__ __launch_bounds__(256) void array_quantize_kernel(const void *__restrict__ X, long n, const unsigned *__restrict__ slot,
                                                             int8_t *__restrict__ Xq) {
    const float a = __uint_as_float(*slot);
    const float inv = (a == 0.0f) ? 0.0f : 127.0f / a;
    for (long i = (static_cast<long>(blockIdx.x) * 256 + threadIdx.x) * 8; i < n; i += static_cast<long>(gridDim.x) * 256 * 8) {
        float x[8];
        load8<T>(X, i, x);
        *reinterpret_cast<uint2 *>(Xq + i) = quant8(x, inv);
    }
}

// ---- block-level: one scale per (head, block of `block` keys), single pass -----------------------
// A workgroup owns one block: at most 128 keys x 128 channels = 16384 elements = 8 chunks of 8 per thread,
// held in registers between the absmax and the rounding, so the activations are read once.
template <typename T>
__global__ __launch_bounds__(256) void block_quantize_kernel(const void *__restrict__ X, long N, int d, int block,
                                                             int8_t *__restrict__ Xq, float *__restrict__ scale) {
    const long head = blockIdx.y, jb = blockIdx.x;
    const long first = head * N * d + jb * static_cast<long>(block) * d;     // first element of the block
    const long keys = (N - jb * block < block) ? (N - jb * block) : block;
    const int chunks = static_cast<int>(keys * d / 8);
    float x[8][8];
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = threadIdx.x + 256 * i;
        if (c < chunks) {
            load8<T>(X, first + 8L * c, x[i]);
            a = fmaxf(a, absmax8(x[i]));
        }
    }
    a = group_max<64>(a);
    __shared__ float wmax[4];
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = a;
    __syncthreads();
    a = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    const float inv = (a == 0.0f) ? 0.0f : 127.0f / a;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = threadIdx.x + 256 * i;
        if (c < chunks) *reinterpret_cast<uint2 *>(Xq + first + 8L * c) = quant8(x[i], inv);
    }
    if (threadIdx.x == 0) scale[head * gridDim.x + jb] = (a == 0.0f) ? 1.0f : a / 127.0f;
}

__global__ void zero_word_kernel(unsigned *p) { *p = 0u; }

// absmax bits in slot 0 -> the scale in every slot.  One block; slot 0 is read by every thread before any write.
__global__ void array_scale_finalize_kernel(float *scale, long heads) {
    const float a = __uint_as_float(reinterpret_cast<const unsigned *>(scale)[0]);
    __syncthreads();
    for (long h = threadIdx.x; h < heads; h += blockDim.x) scale[h] = (a == 0.0f) ? 1.0f : a / 127.0f;
}

// fn.template operator()<LPR>() for the row length d = 8 LPR
template <typename F> int by_row_lanes(int d, F fn) {
    switch (d / 8) {
    case 4: fn(std::integral_constant<int, 4>{}); break;
    case 8: fn(std::integral_constant<int, 8>{}); break;
    case 16: fn(std::integral_constant<int, 16>{}); break;
    case 32: fn(std::integral_constant<int, 32>{}); break;
    case 64: fn(std::integral_constant<int, 64>{}); break;
    default: return IFA_ERR_UNSUPPORTED;
    }
    return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
}

template <typename T, bool HADAMARD>
int launch_tokenwise(const TokenJob &j0, const TokenJob &j1, int jobs, long rows, int d, hipStream_t st) {
    const long rows_per_block = 256 / (d / 8);
    long blocks = (rows + rows_per_block - 1) / rows_per_block;
    const long cap = 256L * 64 / jobs;                   // grid-stride beyond 64 blocks per CU (4 to 64 measured alike)
    if (blocks > cap) blocks = cap;
    const dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>(jobs)), block(256);
    return by_row_lanes(d, [&](auto lpr) {
        hipLaunchKernelGGL((quantize_tokenwise_kernel<T, decltype(lpr)::value, HADAMARD>), grid, block, 0, st, j0, j1, rows);
    });
}

// Shares, whole heads or parts.  From 96 heads on, whole heads keep enough workgroups busy and the second read of V is partly a
// cache hit (Q, K, V of 96 x 2048 x 128 fp16: 47 us whole, 55 in parts; 128 x 4096 x 128: 124 and 145).  With fewer heads one workgroup walks its head at about 40 GB/s next to the fixed 4 us, and what
// the second launch costs (2.5 us) only buys the chip's bandwidth for heads that are long: 4 heads of 256 KB 10.7 us whole
// and 7.6 in parts, 64 heads of 128 KB 10.2 and 12.0.
// Next to the rows of Q and K the line lies lower for heads of up to 1 MB, which an extra launch delays more than it speeds up (Q, K, V in rotation, parts /
// whole, us: 64 x 1777 x 128 fp16 34.5 / 27.4, 64 x 4096 x 128 72.5 / 68.2, 64 x 6000 x 64 53 / 43.6, 80 x 2600 x 128 56.5 / 49.4, 80 x 1300 x 128 fp32 45.3 / 37.3;
// beyond it 64 x 8192 x 128 fp16 147 / 160, and below 64 heads or, in fp32, 80 they even out: 48 x 1777 x 128 fp16 27.7 / 29.7, 64 x 1777 x 128 fp32 48.1 / 51.7).
// `alone`: no rows of Q and K to fill in around the heads, so long heads that leave CUs without one (256 take a head each, then the
// next 256) go in parts as well.  V alone, whole / in parts, us, repeated and with inputs in rotation: 96 x 8192 x 128 fp16 101, 121 / 84, 103, fp32 220, 232 /
// 174, 186; 128 x 4096 x 128 fp32 108, 127 / 95, 108; 260 x 2048 x 128 fp16 60, 71 / 56, 66, fp32 121, 135 / 105, 121; 300 x 8192 x 64 fp16 155, 166 / 149, 157;
// on the other side 128 x 4096 x 128 fp16 49, 67 / 54, 62, 128 x 1024 x 128 fp32 19, 27 / 25, 28, 160 x 4096 x 128 fp16 59, 78 / 66, 78, 256 x 4096 x 128 fp16 101, 117 / 118, 133.
HeadJob plan_heads(const void *X, long heads, long per_head, int elem_bytes, int8_t *Xq, float *scale, bool alone) {
    HeadJob hj = {X, Xq, scale, per_head, static_cast<int>(heads), 0, 0, 1, 0, 0};
    const long head_bytes = per_head * elem_bytes, rounds = (heads + 255) / 256;
    // Up to 64 heads of up to 256 KB (fp32, or 8 to 48 heads beside the rows of Q and K: 384 KB): in shares, one launch instead of two, or of 16 KB and more
    // per share instead of a whole head, and about as many workgroups as CUs.  Before (whole or parts) / shares, us, Q, K, V in rotation, fp16: 1 x 96 KB
    // 5.6 / 3.8, 4 x 128 6.8 / 4.9, 8 x 64 5.3 / 4.1, 8 x 192 7.5 / 6.0, 16 x 128 8.8 / 5.5, 32 x 192 13.9 / 9.2, 32 x 384 18.2 / 15.8, 48 x 256 18.7 / 14.6, 64 x 256 20.3 / 18.7; beyond
    // 1 x 384 7.3 / 7.9, 4 x 384 8.3 / 8.6, 64 x 384 24.2 / 26.9, 80 x 256 20.8 / 22.0.  V alone: 8 x 96 5.5 / 3.8, 32 x 128 8.4 / 5.1, 48 x 256 13.2 / 9.0; 16 x 384 8.2 / 8.7.
    const long share_limit = elem_bytes == 4 || (!alone && heads >= 8 && heads <= 48) ? 384L << 10 : 256L << 10;
    if (heads <= 64 && head_bytes <= share_limit) {
        long n = head_bytes / (16L << 10);
        if (n > 12) n = 12;
        if (n > 224 / heads) n = 224 / heads;
        if (n >= 2 && head_bytes <= n * KEEP_BYTES) {
            hj.shares = static_cast<int>(n);
            hj.chunks_per_region = (per_head / 8 + n - 1) / n;
            return hj;
        }
    }
    const bool uneven = alone && 8 * heads < 5 * 256 * rounds && head_bytes > (heads > 256 ? 256L << 10 : 1L << 20);
    const bool beside = !alone && heads >= (elem_bytes == 2 ? 64 : 80) && head_bytes <= (1L << 20);
    if (beside || (heads >= 96 && per_head < (1L << 29) && !uneven) || head_bytes <= (64L << 10) + (heads < 96 ? heads * (4L << 10) : 0)) return hj;
    const long chunks = per_head / 8;
    auto split = [&](long want, long &per) {             // at most `want` pieces of at least HEAD_THREADS chunks
        long n = chunks / HEAD_THREADS < want ? chunks / HEAD_THREADS : want;
        if (n < 1) n = 1;
        per = chunks / n;
        return static_cast<int>(n);
    };
    hj.parts = split((512 + heads - 1) / heads < 64 ? (512 + heads - 1) / heads : 64, hj.chunks_per_part);
    hj.regions = split((1024 + heads - 1) / heads, hj.chunks_per_region);   // 8 KB of codes or more: the words of 64 parts fit
    return hj;
}
int head_workgroups(const HeadJob &hj) {
    if (hj.shares > 1) return (hj.heads + 7) / 8 * 8 * hj.shares;
    return hj.parts == 0 ? hj.heads : hj.heads * hj.parts;
}

template <typename T> int launch_head_second(const HeadJob &hj, hipStream_t st) {
    if (hj.parts > 0)
        hipLaunchKernelGGL((head_quantize_regions_kernel<T>), dim3(static_cast<unsigned>(hj.regions), static_cast<unsigned>(hj.heads)), dim3(256),
                           0, st, hj);
    return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
}

template <typename T>
int launch_headwise(const void *X, long heads, long per_head, int8_t *Xq, float *scale, int global_scale, hipStream_t st) {
    if (!global_scale) {
        const HeadJob hj = plan_heads(X, heads, per_head, sizeof(T), Xq, scale, true);
        // Many short heads: four workgroups of 256 in the place of one of 1024, most of whose threads have nothing to do (8192 heads of 2 KB
        // 8.6 us, 25 with 1024; 8192 of 8 KB 17 and 29; 4096 of 32 KB, beyond the line, 34 and 32).
        if (hj.parts == 0 && heads > 512 && per_head * static_cast<long>(sizeof(T)) <= (16L << 10)) {
            hipLaunchKernelGGL((short_head_kernel<T>), dim3(static_cast<unsigned>(heads)), dim3(SHORT_HEAD_THREADS), 0, st, hj);
            return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
        }
        hipLaunchKernelGGL((head_first_pass_kernel<T>), dim3(static_cast<unsigned>(head_workgroups(hj))), dim3(HEAD_THREADS), 0, st, hj);
        return launch_head_second<T>(hj, st);
    }
    unsigned *slot = reinterpret_cast<unsigned *>(scale);
    const long n = heads * per_head;
    long bx = (n / 8 + 255) / 256;
    if (bx > 1024) bx = 1024;                            // about 4 workgroups per CU: more only add atomics on the slot
    hipLaunchKernelGGL(zero_word_kernel, dim3(1), dim3(1), 0, st, slot);
    hipLaunchKernelGGL((array_absmax_kernel<T>), dim3(static_cast<unsigned>(bx)), dim3(256), 0, st, X, n, slot);
    hipLaunchKernelGGL((array_quantize_kernel<T>), dim3(static_cast<unsigned>(bx)), dim3(256), 0, st, X, n, slot, Xq);
    hipLaunchKernelGGL(array_scale_finalize_kernel, dim3(1), dim3(256), 0, st, scale, heads);
    return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
}

template <typename T>
int launch_qkv(const TokenJob &jq, const TokenJob &jk, const void *V, long heads, long N, int d, int8_t *Vq, float *sV, hipStream_t st) {
    const HeadJob hj = plan_heads(V, heads, N * d, sizeof(T), Vq, sV, false);
    const int head_wgs = head_workgroups(hj);
    const long rows = heads * N, rows_per_block = HEAD_THREADS / (d / 8);
    long per_tensor = (rows + rows_per_block - 1) / rows_per_block;
    // grid-stride beyond 32 (whole heads) or 16 workgroups per CU for Q and K together (128 x 4096 x 128: 124 us at 32, 128 at
    // 16, 132 at 64; in parts, 32 x 16384 x 128: 144 at 16, 154 at 64)
    const long cap = 256L * (hj.parts == 0 ? 16 : 8);
    if (per_tensor > cap) per_tensor = cap;
    // below 64 MB the caches hold V whatever Q and K do (64 x 1024 x 64, 25 MB: 10.7 us with the hint, 10.4 without)
    const int once = hj.parts == 0 && 3 * heads * N * d * static_cast<long>(sizeof(T)) > (64L << 20);
    const int rc = by_row_lanes(d, [&](auto lpr) {
        hipLaunchKernelGGL((quantize_qkv_kernel<T, decltype(lpr)::value>), dim3(static_cast<unsigned>(head_wgs + 2 * per_tensor)), dim3(HEAD_THREADS),
                           0, st, jq, jk, rows, hj, head_wgs, once);
    });
    return rc == IFA_OK ? launch_head_second<T>(hj, st) : rc;
}

}  // namespace

namespace {
int tokenwise_args(const void *X, int x_dtype, long rows, int d, const signed char *Xq, const float *scale, float scale_mul) {
    if (!X || !Xq || !scale) return IFA_ERR_NULL;
    if (rows <= 0 || d <= 0 || rows > (1L << 40) / d) return IFA_ERR_SHAPE;
    if (x_dtype < IFA_F32 || x_dtype > IFA_BF16) return IFA_ERR_DTYPE;
    if (d != 32 && d != 64 && d != 128 && d != 256 && d != 512) return IFA_ERR_UNSUPPORTED;
    if (!ifa_aligned16(X) || !ifa_aligned16(Xq) || (reinterpret_cast<uintptr_t>(scale) & 3)) return IFA_ERR_UNSUPPORTED;
    if (!(scale_mul > 0.0f) || scale_mul > 3.0e38f) return IFA_ERR_SHAPE;
    return IFA_OK;
}

template <bool HADAMARD>
int tokenwise_launch(const TokenJob &j0, const TokenJob &j1, int jobs, int x_dtype, long rows, int d, hipStream_t st) {
    switch (x_dtype) {
    case IFA_F32: return launch_tokenwise<float, HADAMARD>(j0, j1, jobs, rows, d, st);
    case IFA_F16: return launch_tokenwise<__half, HADAMARD>(j0, j1, jobs, rows, d, st);
    default: return launch_tokenwise<__hip_bfloat16, HADAMARD>(j0, j1, jobs, rows, d, st);
    }
}

template <bool HADAMARD>
int tokenwise_entry(const void *X, int x_dtype, long rows, int d, signed char *Xq, float *scale, float scale_mul,
                    void *hip_stream) {
    const int rc = tokenwise_args(X, x_dtype, rows, d, Xq, scale, scale_mul);
    if (rc != IFA_OK) return rc;
    const TokenJob job = {X, reinterpret_cast<int8_t *>(Xq), scale, scale_mul};
    return tokenwise_launch<HADAMARD>(job, job, 1, x_dtype, rows, d, static_cast<hipStream_t>(hip_stream));
}

int headwise_args(const void *X, int x_dtype, long heads, long N, int d, const signed char *Xq, const float *scale) {
    if (!X || !Xq || !scale) return IFA_ERR_NULL;
    if (heads <= 0 || N <= 0 || d <= 0 || heads > 65535 || N > (1L << 40) / d / heads) return IFA_ERR_SHAPE;
    if (x_dtype < IFA_F32 || x_dtype > IFA_BF16) return IFA_ERR_DTYPE;
    if ((N * d) % 8 != 0) return IFA_ERR_UNSUPPORTED;
    if (!ifa_aligned16(X) || !ifa_aligned16(Xq) || (reinterpret_cast<uintptr_t>(scale) & 3)) return IFA_ERR_UNSUPPORTED;
    return IFA_OK;
}

}  // namespace

extern "C" int quantize_tokenwise_ex(const void *X, int x_dtype, long rows, int d, signed char *Xq, float *scale,
                                     float scale_mul, void *hip_stream) {
    return tokenwise_entry<false>(X, x_dtype, rows, d, Xq, scale, scale_mul, hip_stream);
}

extern "C" int quantize_tokenwise_hadamard(const void *X, int x_dtype, long rows, int d, signed char *Xq, float *scale,
                                           float scale_mul, void *hip_stream) {
    return tokenwise_entry<true>(X, x_dtype, rows, d, Xq, scale, scale_mul, hip_stream);
}

extern "C" int quantize_tokenwise(const void *X, int x_dtype, long rows, int d, signed char *Xq, float *scale) {
    return quantize_tokenwise_ex(X, x_dtype, rows, d, Xq, scale, 1.0f, ifa_current_stream());
}

extern "C" int quantize_blockwise(const void *X, int x_dtype, long heads, long N, int d, int block_keys,
                                  signed char *Xq, float *scale, void *hip_stream) {
    if (!X || !Xq || !scale) return IFA_ERR_NULL;
    if (heads <= 0 || N <= 0 || d <= 0 || block_keys <= 0 || heads > 65535 || N > (1L << 40) / d / heads) return IFA_ERR_SHAPE;
    if (x_dtype < IFA_F32 || x_dtype > IFA_BF16) return IFA_ERR_DTYPE;
    if (d % 8 != 0 || static_cast<long>(block_keys) * d > 16384) return IFA_ERR_UNSUPPORTED;
    const long blocks = (N + block_keys - 1) / block_keys;
    if (blocks > 0x7fffffffL) return IFA_ERR_UNSUPPORTED;
    if (!ifa_aligned16(X) || !ifa_aligned16(Xq) || (reinterpret_cast<uintptr_t>(scale) & 3)) return IFA_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    int8_t *q = reinterpret_cast<int8_t *>(Xq);
    const dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>(heads)), block(256);
    switch (x_dtype) {
    case IFA_F32: hipLaunchKernelGGL((block_quantize_kernel<float>), grid, block, 0, st, X, N, d, block_keys, q, scale); break;
    case IFA_F16: hipLaunchKernelGGL((block_quantize_kernel<__half>), grid, block, 0, st, X, N, d, block_keys, q, scale); break;
    default: hipLaunchKernelGGL((block_quantize_kernel<__hip_bfloat16>), grid, block, 0, st, X, N, d, block_keys, q, scale); break;
    }
    return hipGetLastError() == hipSuccess ? IFA_OK : IFA_ERR_HIP;
}

extern "C" int quantize_headwise_ex(const void *X, int x_dtype, long heads, long N, int d, signed char *Xq,
                                    float *scale, int global_scale, void *hip_stream) {
    const int rc = headwise_args(X, x_dtype, heads, N, d, Xq, scale);
    if (rc != IFA_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    int8_t *q = reinterpret_cast<int8_t *>(Xq);
    switch (x_dtype) {
    case IFA_F32: return launch_headwise<float>(X, heads, N * d, q, scale, global_scale, st);
    case IFA_F16: return launch_headwise<__half>(X, heads, N * d, q, scale, global_scale, st);
    default: return launch_headwise<__hip_bfloat16>(X, heads, N * d, q, scale, global_scale, st);
    }
}

extern "C" int quantize_headwise(const void *X, int x_dtype, long heads, long N, int d, signed char *Xq,
                                 float *scale, int global_scale) {
    return quantize_headwise_ex(X, x_dtype, heads, N, d, Xq, scale, global_scale, ifa_current_stream());
}

extern "C" int quantize_qk(const void *Q, const void *K, int x_dtype, long rows, int d, signed char *Q_i8, signed char *K_i8,
                           float *s_Q, float *s_K, float s_Q_mul, int hadamard, void *hip_stream) {
    int rc = tokenwise_args(Q, x_dtype, rows, d, Q_i8, s_Q, s_Q_mul);
    if (rc == IFA_OK) rc = tokenwise_args(K, x_dtype, rows, d, K_i8, s_K, 1.0f);
    if (rc != IFA_OK) return rc;
    const TokenJob jq = {Q, reinterpret_cast<int8_t *>(Q_i8), s_Q, s_Q_mul}, jk = {K, reinterpret_cast<int8_t *>(K_i8), s_K, 1.0f};
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    return hadamard ? tokenwise_launch<true>(jq, jk, 2, x_dtype, rows, d, st) : tokenwise_launch<false>(jq, jk, 2, x_dtype, rows, d, st);
}

extern "C" int quantize_qkv(const void *Q, const void *K, const void *V, int x_dtype, long heads, long N, int d,
                            signed char *Q_i8, signed char *K_i8, signed char *V_i8, float *s_Q, float *s_K, float *s_V,
                            float s_Q_mul, void *hip_stream) {
    int rc = headwise_args(V, x_dtype, heads, N, d, V_i8, s_V);             // bounds heads * N * d first
    if (rc == IFA_OK) rc = tokenwise_args(Q, x_dtype, heads * N, d, Q_i8, s_Q, s_Q_mul);
    if (rc == IFA_OK) rc = tokenwise_args(K, x_dtype, heads * N, d, K_i8, s_K, 1.0f);
    if (rc != IFA_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const TokenJob jq = {Q, reinterpret_cast<int8_t *>(Q_i8), s_Q, s_Q_mul}, jk = {K, reinterpret_cast<int8_t *>(K_i8), s_K, 1.0f};
    int8_t *vq = reinterpret_cast<int8_t *>(V_i8);
    switch (x_dtype) {
    case IFA_F32: return launch_qkv<float>(jq, jk, V, heads, N, d, vq, s_V, st);
    case IFA_F16: return launch_qkv<__half>(jq, jk, V, heads, N, d, vq, s_V, st);
    default: return launch_qkv<__hip_bfloat16>(jq, jk, V, heads, N, d, vq, s_V, st);
    }
}

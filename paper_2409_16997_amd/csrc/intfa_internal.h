// Host-side helpers shared by the translation units of libintfa.so (not part of the C ABI).
#ifndef INTFA_INTERNAL_H
#define INTFA_INTERNAL_H

#include <hip/hip_runtime.h>
#include <stdint.h>

// Stream set by ifa_set_stream(); the null stream until then.
hipStream_t ifa_current_stream();

// Groups of 32 queries that one launch of a few-query kernel holds: a launch has less than 2^32 threads and their workgroups up to
// 768 (the other kernels have 256, which is three times as many heads).
constexpr long IFA_FEW_MAX_GROUPS = 5L << 20;

// Which calls the few-query kernels take (INT8 with one V scale per head: the same results, bit for bit): those that would leave the
// fused kernel's two workgroups per CU mostly empty.  They have four workgroups of 32 queries where the fused kernel has one of
// 128, one per CU at a time, and walk 256 keys in 1.0 - 1.5 us where a fused workgroup alone on its CU takes 3.3.  Few-query / fused, us,
// d = 128 unless stated:
//   up to 256 workgroups, one wave   32 heads x 256 queries x 8192 keys 49 / 106, 4 x 1024 x 1024 9.0 / 16.6, 32 x 256 x 256 6.6 / 7.4;
//                                    d = 64, 8 x 1024 x 1024 7.4 / 13.3, 16 x 512 x 512 5.7 / 8.1, 8 x 256 x 256 4.6 / 5.4
//   more, up to 32 queries per head  the fused kernel has a wavefront in four busy, but twice the workgroups on a CU and less to start:
//                                    up to `short_keys` keys it wins (INT8: 512 x 32 x 256 14.4 / 12.8, 1000 x 1 x 256 23.8 / 22.1, x 384 28.4 / 28.2,
//                                    x 512 31.3 / 34.2; 4096 x 1 x 128 70 / 42), beyond it does not (1000 x 1 x 1024 48 / 56, 768 x 32 x 1024 41 / 52)
//   more, longer ones                two waves win on long key sequences (32 x 512 x 8192 79 / 106, 256 x 64 x 2048 37 / 37) and lose on short ones
//                                    (64 x 200 x 200 7.5 / 5.9), more lose (32 x 700 x 8192 120 / 107, 512 x 64 x 2048 71 / 59)
static inline long ifa_query_groups(int heads, int Nq) { return static_cast<long>(heads) * ((Nq + 31) / 32); }
static inline bool ifa_few_queries(int heads, int Nq, int Nk, int d, bool half) {
    const int short_keys = half ? (d == 128 ? 256 : 64) : (d == 128 ? 384 : 0);   // (INT8, d = 64: the packed kernel's)
    const long groups = ifa_query_groups(heads, Nq);
    if (groups > IFA_FEW_MAX_GROUPS) return false;
    if (groups <= 256) return true;
    return Nq <= 32 ? Nk > short_keys : groups <= 512 && Nk >= 2048;
}

// Which INT8 calls the packed kernel takes before either of them, us (calls in a graph, K and V in rotation):
//   one key block                    packed / few-query: 32 x 1 x 128 4.3 / 4.9, 128 x 32 x 64 5.0 / 5.8; d = 64, 32 x 1 x 128 3.7 / 4.3
//   d = 64, more than 256 workgroups and up to 1024 or 1280 keys, packed / few-query / fused: 264 x 1 x 256 6.7 / 8.5 / 7.5, 512 x 32 x 128
//                                    5.9 / 9.4 / 6.8, 1000 x 1 x 512 20.5 / 24.1 / 22.8, 4096 x 1 x 128 30 / 62 / 33, 400 x 8 x 1025 16.8 / 18.4 / 20;
//                                    beyond that 400 x 8 x 1500 21.6 / 19.7 / 27.6, 768 x 32 x 1024 26.3 / 25.4 / 33.  With 33 to 64 queries packed / fused: 256 x 33 x 128 5.2 / 5.7,
//                                    x 1500 19.9 / 21.5, but 140 x 64 x 64 4.9 / 4.5 and above 512 workgroups 300 x 64 x 512 15.2 / 11.7
static inline bool ifa_packed_queries(int heads, int Nq, int Nk, int d) {
    const long groups = ifa_query_groups(heads, Nq);
    if (groups <= 256) return Nk <= 128;
    if (d != 64) return false;
    return Nq <= 32 ? Nk <= (groups <= 512 ? 1280 : 1024) : Nq <= 64 && groups <= 512 && Nk >= 128 && Nk < 2048;
}

// The packed or the twelve-wavefront few-query kernel of intfa_attention_fewq.hip, for the dispatcher of the entry points in
// intfa_attention.hip; arguments already validated.
int ifa_launch_narrow(const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV, int heads,
                      int Nq, int Nk, int d, int causal, int vblock, void *O, int o_dtype, hipStream_t st);

// That dispatcher, one V scale per head: the kernel int_flash_attn_fwd_rect runs; arguments already validated.
int ifa_launch_fwd(const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV, int heads,
                   int Nq, int Nk, int d, int causal, void *O, int o_dtype, hipStream_t st);

static inline bool ifa_aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

#endif

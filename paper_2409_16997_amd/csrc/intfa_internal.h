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

// Which calls the few-query kernels take (INT8: same results, bit for bit): up to 32 queries per head, and longer ones that
// would leave the fused kernel's two workgroups per CU mostly empty.  They have four workgroups of 32 queries where the
// fused kernel has one of 128, one per CU at a time, and walk 256 keys in 1.0 - 1.5 us where a fused workgroup alone on its
// CU takes 3.3: one wave of 256 workgroups always wins (32 heads x 256 queries x 8192 keys 49 us against 106,
// 4 x 1024 x 1024 9.0 against 16.6, 32 x 256 x 256 6.6 against 7.4), two waves win on long key sequences (32 x 512 x 8192: 79
// against 106, 256 x 64 x 2048: 37 and 37) and lose on short ones (64 x 200 x 200: 7.5 against 5.9), more lose
// (32 x 700 x 8192: 120 against 107, 512 x 64 x 2048: 71 against 59).
static inline bool ifa_few_queries(int heads, int Nq, int Nk) {
    const long wgs = static_cast<long>(heads) * ((Nq + 31) / 32);
    if (wgs > IFA_FEW_MAX_GROUPS) return false;
    return Nq <= 32 || wgs <= 256 || (wgs <= 512 && Nk >= 2048);
}

// The few-query kernel of intfa_attention_fewq.hip (one workgroup per head and 32 queries), for the dispatcher of the
// entry points in intfa_attention.hip; arguments already validated.
int ifa_launch_narrow(const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV, int heads,
                      int Nq, int Nk, int d, int causal, int vblock, void *O, int o_dtype, hipStream_t st);

static inline bool ifa_aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

#endif

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
//   more, longer ones                (those that ifa_pair_queries() leaves) two waves win on long key sequences (2 x 5000 x 5000 33 / 65) and lose on short ones
//                                    (64 x 200 x 200 7.5 / 5.9), more lose (32 x 700 x 8192 120 / 107, 512 x 64 x 2048 71 / 59)
static inline long ifa_query_groups(int heads, int Nq) { return static_cast<long>(heads) * ((Nq + 31) / 32); }
static inline bool ifa_few_queries(int heads, int Nq, int Nk, int d, bool half) {
    const int short_keys = half ? (d == 128 ? 256 : 64) : (d == 128 ? 384 : 0);   // (INT8, d = 64: the packed kernel's)
    const long groups = ifa_query_groups(heads, Nq);
    if (groups > IFA_FEW_MAX_GROUPS) return false;
    if (groups <= 256) return true;
    return Nq <= 32 ? Nk > short_keys : groups <= 512 && Nk >= 2048;
}

// Which of the few-query kernel's INT8 calls the decode kernel (one query per head) and its form for two to eight take: as long as its workgroups (four per head,
// d = 64: two) each have a CU of their own.  Few-query / decode kernel, us, K and V in rotation: 1 x 300 keys 5.2 / 3.9, 32 x 1024 8.1 / 6.5, 64 x 1500 .88 of the time,
// 64 x 32800 .81, 8 x 24600 .58; d = 64, 128 x 200 .94, 128 x 4100 .90, 128 x 16500 .80.  Beyond the line, at d = 128: 65 heads x 257 1.21, x 4100 1.38, 128 x 1024 1.32.
// Two to eight queries, repeated: 32 x 4 x 4900 23.9 / 19.1, 8 x 5 x 2048 10.6 / 7.8, 64 x 8 x 16384 81 / 62, 64 x 8 x 600 6.6 / 6.0; d = 64, 64 x 8 x 4900 20.3 / 15.2, 128 x 8 x 600 5.6 /
// 5.2; on fewer keys all that is there to do is start and end: 64 x 8 x 200 4.7 / 5.0, d = 64 128 x 5 x 200 4.0 / 4.5.
static inline bool ifa_decode_query(long heads, int Nq, int Nk, int d) { return heads <= (d == 128 ? 64 : 128) && (Nq == 1 || (Nq <= 8 && Nk > 384)); }

// Which INT8 calls the packed kernel takes before either of them, us (calls in a graph, K and V in rotation):
//   one key block                    packed / few-query: 32 x 1 x 128 4.3 / 4.9, 128 x 32 x 64 5.0 / 5.8; d = 64, 32 x 1 x 128 3.7 / 4.3
//   d = 64, more than 256 workgroups and up to 768 keys (1152 from 1025 on), packed / few-query: 400 x 8 x 768 13.0 / 13.4, 1000 x 1 x 640 22.7 / 24.2,
//                                    1500 x 1 x 1152 47.9 / 47.6, 2000 x 32 x 1024 60.1 / 60.9; and fused, on the same K and V: 260 x 1 x 256 5.1 / 6.6 / 6.3, 512 x 32 x 128 4.5 / 7.6 /
//                                    5.6, 1000 x 1 x 512 18.7 / 20.9 / 21.6.  Beyond that 600 x 1 x 900 23.5 / 20.8, 512 x 32 x 1280 21.0 / 19.1, 1000 x 1 x 1280
//                                    36.7 / 33.4, 2000 x 8 x 1280 69.0 / 64.3.  With 33 to 64 queries packed / fused: 256 x 33 x 128 5.2 / 5.7,
//                                    but 140 x 64 x 64 4.9 / 4.5 and above 512 workgroups 300 x 64 x 512 15.2 / 11.7; from 384 keys on the two-group kernel's
static inline bool ifa_packed_queries(int heads, int Nq, int Nk, int d) {
    const long groups = ifa_query_groups(heads, Nq);
    if (groups <= 256) return Nk <= 128;
    if (d != 64) return false;
    return Nq <= 32 ? Nk <= (groups <= 1024 ? 768 : 1152) : Nq <= 64 && groups <= 512 && Nk >= 128 && Nk < 384;
}

// Which INT8 calls the two-group kernel takes before all of them: more groups of 32 queries than CUs, two of one head to a workgroup.
// It walks 256 keys of 64 queries in 1.7 - 1.9 us, one workgroup per CU; the few-query kernel takes 1.15 for 32 queries, a fused workgroup of 128
// alone on its CU 3.3, two 5.1.  Before (which kernel) / now, us, d = 128 unless stated:
//   up to 256 workgroups, one wave  32 heads x 512 queries x 8192 keys 79 (few-query) / 60, 65 x 128 x 3000 45 (few-query) / 26, 32 x 512 x 1500 25 (fused) / 18,
//                                   x 700 15.1 (fused) / 12.4; d = 64, 256 x 64 x 1000 14.9 (packed) / 11.5.  On fewer keys start and end outweigh it:
//                                   32 x 448 x 448 10.6 (fused) / 10.8, 160 x 64 x 300 10.0 / 10.8; d = 64, 24 x 384 x 450 9.7 / 7.8, 130 x 64 x 300 7.2 / 7.5.
//                                   Half of the key blocks masked: the heaviest workgroup decides, and the two waves of the few-query kernel, which
//                                   takes such calls from 2048 keys on, even out: 2 x 5000 33 (few-query) / 37, 1 x 14000 87 / 89; but 3 x 5000 45 / 38, 8 x 2048 22.8 / 20.4
//   more, some of the blocks masked twice as many and smaller workgroups than the fused kernel's even out better, up to 512 of them the sooner the fewer they are: the
//                                   other one's heaviest workgroup decides, this one's second wave is light and short.  How light falls with the keys in front of
//                                   the queries, where all blocks are visible, and so does the line, in Nk / Nq.  Over 1550 causal calls a head size it is within .2 % of the
//                                   faster kernel on average; 2 of the 943 taken more than 2 % slower.  Fused / this one: 10 x 1996 d = 64 24.5 / 15.5,
//                                   12 x 1518 d = 64 19.3 / 12.6, 12 x 1444 22.8 / 17.6, 3 x 5898 x 14531 187 / 132, 8 x 4096 56 / 41, 4 x 8192 107 / 69; not 24 x 757 14.3 / 15.9,
//                                   32 x 892 x 1979 31.5 / 33.6, 23 x 995 x 1791 27.5 / 30.2, 27 x 1099 x 3885 58.2 / 61.6, d = 64 39 x 565 x 922 14.0 / 15.7, 43 x 526 x 2081 26.2 / 29.6.
//                                   Beyond 512, half of the blocks masked, up to 8 (10) heads: 1 x 32768 410 / 236, 5 x 8192 115 / 99, 10 x 3380 d = 64 39.9 / 32.8; then not:
//                                   20 x 1600 25.8 / 25.9, 12 x 3200 45.5 / 45.5, 12 x 3047 x 4490 71.5 / 74.3, 7 x 8192 112 / 119; beyond `keys`
//                                   8 x 5612 x 8418 126 / 127 (d = 64 99 / 101), 8 x 6124 x 12248 195 / 206 (147 / 161), 4 x 12268 x 24536 382 / 394 (287 / 310)
//   ... with per-block V scales     (`vblock`) the change of unit per block costs this kernel's few wavefronts more, and the second wave has to be lighter still: within .1 %
//                                   of the faster, 14 of 798 more than 2 % slower.  2 x 8419 d = 64 92.9 / 61.7, 5 x 3562 x 5755 65.3 / 46.0, d = 128 2 x 8214 110 / 66, 12 x 1444 23.0 / 18.0; not 43 x 526 x 2081 d = 64 27.3 / 34.7, 12 x 3047 x 4490 58.2 / 69.9,
//                                   41 x 661 x 1156 17.4 / 20.8, 5 x 9696 110 / 122, d = 128 26 x 846 x 1479 24.9 / 28.6, 12 x 3047 x 4490 74 / 85
//   more, all blocks visible        two waves of workgroups against one of the fused kernel's: 48 x 512 x 8192 107 (fused) / 111
static inline bool ifa_pair_queries(int heads, int Nq, int Nk, int d, bool causal, bool vblock = false) {
    if (Nq <= 32 || ifa_query_groups(heads, Nq) <= 256) return false;
    const long wgs = static_cast<long>(heads) * ((Nq + 63) / 64), keys = heads * static_cast<long>(Nk);
    const bool uneven = causal && 2L * Nq >= Nk;
    if (wgs <= 256) return Nk >= (d == 128 ? 512 : 384) && !(uneven && Nk >= 2048 && (heads == 1 || wgs <= 192));
    if (!causal || 4L * Nq < Nk) return false;
    if (vblock && (d == 128 ? 7L : 6L) * Nq < 2L * Nk) return false;
    if (wgs <= 512) {                                            // Nk >= wgs (a + b max(0, Nk / Nq - 9 / 8)) - c
        const long a2 = d == 64 ? 6 : vblock ? 9 : 8, b2 = d == 64 ? (vblock ? 14 : 5) : (vblock ? 10 : 6), c = d == 64 ? 200 : vblock ? 400 : 100;   // 2 a, 2 b
        const long front = 8L * Nk - 9L * Nq;
        return 16 * (Nk + c) * Nq >= wgs * (8 * a2 * Nq + b2 * (front > 0 ? front : 0));
    }
    if (vblock) return wgs <= (heads <= 8 ? (d == 128 ? 680 : 640) : heads <= 10 ? 576 : 0) && 4L * Nk <= (d == 128 ? 6L : 5L) * Nq && keys <= (d == 128 ? 48L : 40L) << 10;
    return uneven && Nk >= 2048 && keys <= 56L << 10 && ((heads <= 8 && wgs <= 768) || (wgs <= 576 && Nk >= (d == 128 ? 4000 : 3000) && (heads <= 10 || 4L * Nk <= 5L * Nq)));
}

// ---- wavefronts per SIMD of the fused kernels ------------------------------------------------------------------------
// Workgroups have 128 queries and two, three or four of them share a CU.  Calls with more than 512 of them have work for a third (half-INT8, d = 64: a fourth); calls that
// two to a CU hold in one round keep two, whose way to the operands is shorter.
//   Even calls (no mask, few keys masked, or up to three workgroups a head): rounds decide.  769 to 1024 are two rounds of 512 and two of 768.
//   Uneven ones (under the mask, at most twice as many keys as queries): an XCD takes its heads in groups, the heaviest workgroups of a group first (map_workgroup()), and a workgroup
// runs the slower the more share its CU.  With one whole group and part of a second, the heavy ones of the second start when the light ones of the first end, and there is little
// left to even them out: two to a CU end sooner.  `groups` = heads / 8 / heads of a group.  Each line with what it measured, us, two / three (four), from 2024 and 1762 uneven calls
// a head size.
static inline bool ifa_even_workgroups(int Nq, int Nk, bool causal) { return !causal || 2L * Nq < Nk || Nq <= 3 * 128; }
// INT8, d = 64: from 865 workgroups (12 to 15 a head: 2251, 16 and more: 1251) on, without one and a half groups of heads that have 20 to 49 each.  96 x 800 causal 16.9 / 20.0 (672),
// 100 x 900 20.2 / 23.3 (800); 110 x 1024 25.6 / 25.1 (880), 100 x 1732 49.0 / 54.6 (1400, 14 a head), 215 x 1732 106.7 / 99.6 (3010), 83 x 2116 66.6 / 61.2 (1411, 17 a head); in one and a
// half groups 45 x 5740 197 / 214, 50 x 6174 242 / 255, 50 x 4446 135 / 143, 88 x 3016 118 / 124.  The calls so taken: .956 of two everywhere (with the better of both .947), 17 of 2024
// more than 3 % slower than with two, 37 without the last condition; off by most 109 x 1293 x 2061 62.6 / 69.1.  Even: 300 x 250 9.5 / 8.6 (600), 230 x 300 11.3 / 9.5; 70 x 1516 x 3308 80.6 / 83.7 (840), 31 x 3216 100 / 102 (806).
static inline int ifa_fused_wavefronts(int heads, int Nq, int Nk, int d, bool causal, int head_group) {
    if (d != 64) return 2;                                       // (256 registers a wavefront)
    const long T_r = (Nq + 127) / 128, wgs = heads * T_r, group = 8L * head_group;
    if (ifa_even_workgroups(Nq, Nk, causal)) return wgs > 512 && !(T_r > 3 && wgs > 768 && wgs <= 1024) ? 3 : 2;
    if (wgs <= (T_r <= 11 ? 864 : T_r <= 15 ? 2250 : 1250)) return 2;
    return T_r >= 20 && T_r < 50 && 8L * heads >= 11 * group && 4L * heads < 7 * group ? 2 : 3;
}
// Half-INT8, d = 64, four: from 1025 on, without one and a quarter to two groups (of four heads here) of 30 to 41 a head: 35 x 4446 ... 50 x 4446 180 / 208, 40 x 4948 192 / 214, 42 x 4770 185 / 205; but
// 82 x 2008 84 / 65 (1312), 144 x 1152 47.4 / 41.1 (1296).  .939 of two everywhere (.930), 18 of 1762 more than 3 % slower, 51 without; off by most 69 x 1831 (1035).
//   d = 128, three: with up to 6 a head from 1251 on, with more from 2251 on with five groups of heads and more; one group of 35 and more a head from 1101 on.  192 x 668 39.3 / 43.0 (1152), 87 x 3837
// 313 / 332 (2610), 46 x 8099 684 / 713 (2944, one and a half groups); 267 x 768 61.0 / 58.8, 222 x 2204 310 / 295 (3996), 32 x 8192 488 / 472 (2048, one group), 32 x 16384 1874 / 1811.  .985 of two
// everywhere (.973), 1 of 1768 more than 3 % slower.  Even: 71 x 1792 3 % slower (994), 490 x 180 x 685 50.2 / 54.4 (980), 264 x 258 x 697 45.6 / 48.2 (792); 32 x 5120 11 % faster (1280).
static inline int ifa_half_wavefronts(int heads, int Nq, int Nk, int d, bool causal, int head_group) {
    const long T_r = (Nq + 127) / 128, wgs = heads * T_r, group = 8L * head_group, h8 = 8L * heads;
    const int more = d == 64 ? 4 : 3;
    if (ifa_even_workgroups(Nq, Nk, causal)) return wgs > 512 && !(d == 128 && wgs > 768 && wgs <= 1024) ? more : 2;
    if (d == 64) return wgs > 1024 && !(T_r >= 30 && T_r < 42 && h8 >= 10 * group && 16L * heads < 33 * group) ? more : 2;
    if (T_r <= 6) return wgs > 1250 ? more : 2;
    return (heads >= 5 * group && wgs > 2250) || (T_r >= 35 && wgs > 1100 && h8 >= (T_r >= 46 ? 5 : 6) * group && h8 < 9 * group) ? more : 2;
}

// Which calls of the key-split entry points do without the split: they run the kernel that int_flash_attn_fwd_rect picks.  The
// few-query kernel walks 1000 keys of every head in 5 us (d = 64: 3.5) however many heads there are, until the chip is full, and
// starts 7 us sooner (from 9 queries on 10); the split passes stream K, V and the scores (or K twice) of all heads, so they win while heads are few and keys are many:
//     few-query  u + v Nk,   split  u' + w heads (Nk + E),   the same at heads (Nk + E) = H (Nk - S).
// S is the start in keys; H falls with Nq, whose scores and partial outputs only the split moves through memory.  Fitted to 3590 calls, each repeated on the same K and V
// and on K and V in rotation; it decides the calls that the decode kernel and its form for two to eight do not take (below): of those of up to eight queries the ones of
// more than 64 heads, at d = 64 128, where only one or two queries on more than 34000 keys still split.
// Both sides of the line, heads x queries x keys, few-query / split, us, repeated; (in rotation):
//   d = 128   80 x 1 x 8192 45.4 / 41.6, 88 45.6 / 43.5;  112 x 1 x 32768 178 / 177, 128 181 / 194;  72 x 8 x 16384 85 / 78, 80 85 / 86;  56 x 9 x 8192 43.2 / 43.9, 64 43.6 / 46.6;
//             64 x 16 x 16384 83.8 / 80.4, 72 84.8 / 89.4;  24 x 32 x 4096 19.1 / 20.0 (22.9 / 21.5), 32 20.4 / 21.1;  64 x 32 x 32768 164 / 154, 72 166 / 177
//   d = 64    144 x 1 x 32768 114 / 131;  72 x 9 x 8192 30.9 / 29.6, 80 31.4 / 32.7;  80 x 16 x 16384 57.9 / 55.3, 88 58.2 / 59.0;  80 x 32 x 32768 112 / 109, 88 114 / 118
// Off by most: 8 x 16 x 2500 at d = 128 (12.5 us split, 15.7 taken; in rotation 15.1 and 15.8), 32 x 16 x 4096 (18.4 split, 19.8 taken).
// One query: the decode kernel's own line, decode kernel / split, K and V in rotation: 1 x 3000 .97 of the time, x 4100 1.26; 16 x 4100 .97, x 6200 1.19; 32 x 6200 1.01; 56 x 6200 .96,
// x 8200 1.09; 64 x 8200 .92; d = 64, 1 x 3000 .87, x 4100 1.21; 32 x 6200 .91, x 8200 1.26; 64 x 6200 .87, x 8200 1.08; 96 x 8200 1.00; 112 x 8200 .93, x 16500 .77, x 32800 1.06; 128 x 4100 .75, x 32800 .93.
// Two to eight: its form's line, the same way: 8 queries x 8 heads x 2100 keys 11.6 / 13.4, 32 x 4100 21.2 / 24.4, x 6200 29.4 / 30.3, x 8200 37.5 / 31.1, 48 x 6200 31.9 / 35.7, x 8200
// 40.1 / 39.7, 64 x 8200 39.2 / 46.1, x 16500 71.0 / 72.4; 2 queries, 16 x 3000 13.0 / 13.4, 48 x 4100 23.1 / 26.4, x 6200 31.6 / 31.3; d = 64, 2 queries, 64 x 6200 22.1 / 23.6, 96 x 12300 1.06;
// 8 queries, 64 x 6200 21.9 / 27.2, x 12300 39.6 / 40.5, 96 x 32800 106 / 121.
static inline bool ifa_unsplit_queries(int heads, int Nq, int Nk, int d) {
    if (ifa_decode_query(heads, Nq, Nk, d))
        return Nq == 1 ? Nk <= 3000 + 75 * heads || heads >= 108 : Nk <= 2000 + (86 + 4 * Nq) * heads || heads >= 120 - 3 * Nq;
    const bool stored = Nq <= 8;                                 // the scores go through memory (more queries: K is read again)
    const long E = stored && d == 128 ? 2048 : 1024, S = stored ? 1536 : 2304;
    const long H = stored ? (d == 128 ? 134 - 5 * Nq : 146 - 7 * Nq) : (d == 128 ? 104 : 122) - Nq;
    return Nk <= 2048 || heads * (Nk + E) >= H * (Nk - S);
}

// The kernel of an INT8 call
enum IfaKernel { IFA_KERNEL_FUSED, IFA_KERNEL_PAIR, IFA_KERNEL_PACKED, IFA_KERNEL_FEW };
static inline IfaKernel ifa_fwd_kernel(int heads, int Nq, int Nk, int d, bool causal, bool vblock = false) {
    return ifa_pair_queries(heads, Nq, Nk, d, causal, vblock) ? IFA_KERNEL_PAIR : ifa_packed_queries(heads, Nq, Nk, d) ? IFA_KERNEL_PACKED :
           ifa_few_queries(heads, Nq, Nk, d, false) ? IFA_KERNEL_FEW : IFA_KERNEL_FUSED;
}

// One of the kernels of intfa_attention_fewq.hip (not IFA_KERNEL_FUSED), for the dispatcher of the entry points in
// intfa_attention.hip; arguments already validated.
int ifa_launch_narrow(IfaKernel kernel, const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV, int heads,
                      int Nq, int Nk, int d, int causal, int vblock, void *O, int o_dtype, hipStream_t st);

// That dispatcher, one V scale per head: the kernel int_flash_attn_fwd_rect runs; arguments already validated.
int ifa_launch_fwd(const int8_t *Q, const int8_t *K, const int8_t *V, const float *sQ, const float *sK, const float *sV, int heads,
                   int Nq, int Nk, int d, int causal, void *O, int o_dtype, hipStream_t st);

static inline bool ifa_aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

#endif

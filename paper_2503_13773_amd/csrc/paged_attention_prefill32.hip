// Causal attention of many query positions per sequence over the block-allocated KV cache on
// 32x32x16 matrix-core tiles (gfx950, bf16, head_dim 128, positive scale): the
// recomputation path of a preempted request (prefill re-run over prompt + generated tokens,
// quadratic in the sequence length: paper Section 2.5 and 3.5) and chunked prefill.
//
// Why 32x32 tiles.  Measured on this chip, a vector instruction holds a SIMD's vector issue
// port for 4 cycles, an exponential for 8 and a matrix instruction for 8, whatever its shape;
// a 16x16x32 tile then runs 16 cycles in the matrix pipe, a 32x32x16 tile 32 cycles with twice
// the work.  Attention at head_dim 128 needs per 32 tokens x 32 score columns about 60 vector
// instructions and 16 exponentials of softmax arithmetic (16 scores per lane).  With 34 small
// tiles that adds up to about 800 port cycles against 544 matrix cycles; with 16 large tiles it
// is about 500 port cycles against 512.
//
// One workgroup = (sequence, 2 query heads sharing one KV head, 64 or 128 consecutive query
// rows); each of its 4 or 8 wavefronts owns 16 query rows x 2 heads = the 32 columns of its
// tiles (column c = 16 * head + row).  Odd GQA group sizes take one head and 32 query rows per
// wavefront instead (workgroups of 128 or 256 rows); everything below is written for two heads
// and holds for one with "row" = c.  The workgroup walks the context in steps of 32 tokens
// (the 32 rows of a score tile).  With 8 wavefronts the two groups of four run half a turn
// apart, so that the two wavefronts of a SIMD are in opposite halves of their turns.
//
// K and V rows travel from the cache straight into LDS (global_load_lds_dwordx4: lane l of a
// wavefront writes its 16 bytes at M0 + 16 * l, no register staging), requested two turns
// before their first use (K rows four steps ahead, V rows three); which bytes a
// lane fetches is chosen so that the LDS image is
//   K rows: 16-byte chunks XOR-permuted by the row number (A-operand reads of 16 rows x the
//           same dims then touch every bank once);
//   V rows: 64-byte granules rotated by the row number (the 4 rows x 64 bytes that a
//           half-wavefront reads in one transposing access then fall into disjoint banks).
// Four steps of K and four of V are in LDS (64 KiB).
//
// Per step, with lane = 32 * half + c:
//   S^T = K . Q^T      8 x v_mfma_f32_32x32x16_bf16 (depth = the 128 dims).  A: K row c of the
//                      step, dims 16j + 8*half .. +7; B: the same dims of column c's query row.
//                      The lane receives the 16 scores of column c against tokens
//                      8*(v/4) + 4*half + v%4, v < 16.
//   softmax            all 16 scores of a lane belong to one column: in-lane max (raw scores,
//                      the scale is positive), one fused multiply-add and one exponential per
//                      score (weight = exp2(score * scale - m)); the weights are rounded to
//                      bf16 for P.V and added up in fp32 for the normaliser.  The two halves of
//                      a column meet only when the reference point m moves (lazily: when some
//                      score exceeds it by more than 2^8) and once at the end.
//   O^T += V^T . P^T   8 x v_mfma_f32_32x32x16_bf16: 4 blocks of 32 dims x 2 slices of 16
//                      tokens.  B is the weight registers as they stand (slice n = registers
//                      8n .. 8n+7, depth slot 8*half + i = token 16n + 8*(i/4) + 4*half + i%4);
//                      A = V^T comes from LDS in that token order by transposing reads
//                      (ds_read_b64_tr_b16: 4 consecutive tokens of the lane's dim per read).
//
// The causal mask only bites in the last one or two steps of a wavefront: steps entirely below
// the diagonal of all 16 rows run code without mask or range checks.  Token 0 is visible to
// every query row and steps are walked in order, so every column has a finite reference point
// after the first step.  Workgroups with the most steps (the last query rows) are dispatched
// first.
#include <float.h>
#include <math.h>

#include <algorithm>

#include "kvc_internal.h"
#include "pa_mfma_tile.h"

namespace kvc {

namespace {

using namespace mfma;

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kStepTokens = 32;
constexpr int kStageBytes = kStepTokens * D * 2;  // K (or V) rows of a step: 32 rows x 256 bytes
constexpr float kLazyLog2 = 8.0f;
constexpr int kKStages = 4;   // K rows of steps s+1 .. s+4 during turn s
constexpr int kVStages = 4;   // V rows of steps s .. s+3
// Steps from which a split workgroup's second group takes a share (800 tokens whole 19.7, split 19.5 us; 1000 tokens
// 23.1 / 22.4 us; 600 tokens 16.7 / 17.2 us).
constexpr int kMinSplitSteps = 24;

// Online-softmax state of one column (query row x head); lane (half, c) holds
// O[column c][32*b + 8*(v/4) + 4*half + v%4] in acc[b][v].
struct ColumnState {
    floatx16 acc[4];
    float lsum;  // sum of the rounded weights of this lane's tokens (the other half's lane holds the rest)
    float m;     // reference point of the weights (base-2 units): within 2^kLazyLog2 of the column's running max

    __device__ inline void reset(float lowest) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
        lsum = 0.f;
        m = lowest;
    }
};

// The value lane l ^ 32 holds, next to this lane's: one swap of the two 32-lane halves.
__device__ inline float max_over_halves(float x) {
    const unsigned u = __float_as_uint(x);
    const u32x2 b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const float b0 = __uint_as_float(b[0]), b1 = __uint_as_float(b[1]);
    return b0 > b1 ? b0 : b1;  // inputs are never NaN
}
__device__ inline float sum_over_halves(float x) {
    const unsigned u = __float_as_uint(x);
    const u32x2 b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// max of three without the quieting moves the compiler puts in front of a max whose inputs
// come out of the matrix pipe (they are never NaN here: finite scores or -inf)
__device__ inline float max3(float a, float b, float c) {
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// Raw scores of a step into x (if MASKED, -inf where the token is not visible to the lane's
// column: `limit` = tokens of the step it sees, may be <= 0) and their max over the lane.
template <bool MASKED>
__device__ inline float take_scores(float (&x)[16], const floatx16 &s, int limit, int half) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        x[v] = s[v];
        if (MASKED && 8 * (v >> 2) + 4 * half + (v & 3) >= limit) x[v] = -INFINITY;
    }
    const float a = max3(x[0], x[1], x[2]), b = max3(x[3], x[4], x[5]), c = max3(x[6], x[7], x[8]);
    const float d = max3(x[9], x[10], x[11]), e = max3(x[12], x[13], x[14]);
    const float f = max3(a, b, c), g = max3(d, e, x[15]);
    float h;
    asm("v_max_f32 %0, %1, %2" : "=v"(h) : "v"(f), "v"(g));
    return h;
}

// Lazy rebase: the reference point m only moves when some column's scaled max has grown by more
// than 2^kLazyLog2 over it (always in the first step, m = -inf), so weights are at most
// 2^kLazyLog2 and the 65 multiplies of the rebase are rare.  Every column sees token 0 in its
// first step, so m - m_new is never inf - inf.
__device__ inline void rebase(ColumnState &st, float lane_max, float scale_log2e) {
    const float scaled = lane_max * scale_log2e;
    // the test needs no cross-lane max: if no lane holds a score above m + 2^kLazyLog2, none exists
    if (__builtin_amdgcn_ballot_w64(scaled > st.m + kLazyLog2) != 0) {
        const float m_new = fmaxf(st.m, max_over_halves(scaled));
        const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
        st.m = m_new;
#pragma unroll
        for (int b = 0; b < 4; ++b) st.acc[b] *= alpha;
        st.lsum *= alpha;
    }
}

// A operands of O^T += V^T . P^T straight from LDS.  The transposing read hands lane i of a
// 16-lane block the i-th 16-bit element of each of the four 16-element groups that lanes
// 4k .. 4k+3 of the block point at (8 bytes each).  Block (half, w) of this wavefront covers
// dims 32b + 16w .. +15; its lanes 4k .. 4k+3 point at dims +0, 4, 8, 12 of token
// 16n + 8g + 4*half + k, so the lane of dim 32b + c receives that dim of the four tokens
// 16n + 8g + 4*half .. +3: depth slots 8*half + 4g .. +3 of slice n, the order the score layout
// fixed.  Row R of a V stage keeps its 64-byte granule b at granule position (b + R) % 4, and
// R % 4 = k for the row a lane points at, so the byte offset of the lane inside a stage for
// dim block b is v_lane_offset(b) + (16n + 8g) rows.
__device__ inline int v_lane_offset(int b, int half, int c) {
    const int i16 = c & 15, k = i16 >> 2;
    return (4 * half + k) * 256 + ((b + k) & 3) * 64 + 32 * (c >> 4) + 8 * (i16 & 3);
}
template <int N>
__device__ inline void read_v_operand(uint2 (&va)[2], const unsigned char *vlane) {
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef v4i16 __attribute__((address_space(3))) * lds_v4i16_ptr;
#pragma unroll
    for (int g = 0; g < 2; ++g)
        va[g] = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(vlane + (16 * N + 8 * g) * 256)));
}

// V rows at or past `vlim` (tokens of the step visible to any column of this wavefront) are
// zeroed in the operand of slice N: their weights are zero for every column and the rows may
// hold NaN.
template <int N>
__device__ inline void mask_v_operand(uint2 (&va)[2], int vlim, int half) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const int tok = 16 * N + 8 * g + 4 * half;
        va[g].x &= (tok < vlim ? 0xffffu : 0u) | (tok + 1 < vlim ? 0xffff0000u : 0u);
        va[g].y &= (tok + 2 < vlim ? 0xffffu : 0u) | (tok + 3 < vlim ? 0xffff0000u : 0u);
    }
}

__device__ inline bf16x8 v_operand(const uint2 (&va)[2]) {
    const uint4 aw = {va[0].x, va[0].y, va[1].x, va[1].y};
    return __builtin_bit_cast(bf16x8, aw);
}

// K operand j of a step from LDS (a stage is 32 rows of 256 bytes, 16-byte chunks XOR-permuted
// by row % 16); lane (half, c) reads row c, dims 16j + 8*half .. +7.
template <int J>
__device__ inline bf16x8 read_k_operand(const unsigned char *krow, int half, int c) {
    return *reinterpret_cast<const bf16x8 *>(krow + (((2 * J + half) ^ (c & 15)) << 4));
}

// 16 bytes per lane from global memory straight into LDS: lane l's bytes land at lds_addr +
// 16 * l (lds_addr uniform).  The two-instruction forms load a second 1 KiB from 1 KiB further
// on both sides.  The compiler does not see these accesses: the caller orders them against LDS
// reads with barriers and waits for them with wait_loads_but().
__device__ inline void load_rows_to_lds(const void *base, uint32_t off0, uint32_t off1_minus_1k, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\tglobal_load_lds_dwordx4 %2, %3 offset:1024"
                 :: "s"(lds_addr), "v"(off0), "v"(off1_minus_1k), "s"(base) : "memory");
}
__device__ inline void load_row_group_to_lds(const void *base, uint32_t off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds_addr), "v"(off), "s"(base) : "memory");
}
__device__ inline void load_lane_to_lds(const void *addr, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_addr), "v"(addr) : "memory");
}
template <int N>
__device__ inline void wait_loads_but() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// The barrier that ends a turn.  The wavefront first waits for its own LDS reads (operands
// requested for the next turn): the loads of the next turn overwrite the stages they come from.
__device__ inline void turn_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The barrier in the middle of a turn orders no data (see the kernel): it only keeps the two
// groups of wavefronts half a turn apart.
__device__ inline void phase_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Nothing moves across this point when the compiler orders the instructions of a turn.
#define KVC_PIN() __builtin_amdgcn_sched_barrier(0)

// One turn of the software pipeline: the weights and the P.V accumulation of step `cur` (raw
// scores in x) together with the scores and the max of step `next`.  The order of the turn is
// pinned chunk by chunk, one matrix instruction (32 cycles in the matrix pipe, 8 on the issue
// port) per chunk together with the vector work that fits under it and the LDS reads of operands
// that are due half a turn or more later:
//     chunks  0 ..  3   S(next) += K operand j . Q, j < 4       2 weights of cur each (fma, exp2), rounding, sum
//                       reads K operand 4 + j of step next
//     chunks  4 ..  7   O block b += V slice 0 . weights 0..7   2 weights each (scores 8 .. 15), rounding, sum
//                       reads V operand b, slice 1, of step cur
//     chunks  8 .. 11   S(next) += K operand j . Q, j >= 4      block id of the following turn's loads (`lookup`)
//                       reads K operand j - 4 of the step after next and V operand j - 4, slice 0, of step next
//     chunks 12 .. 15   O block b += V slice 1 . weights 8..15  max of S(next)
//                       requests the K and V rows of the step four ahead (`issue_k`, `issue_v`)
// so the turn starts with ka_lo = K operands 0 .. 3 of step next and va0 = the slice-0 V
// operands of step cur in registers and ends with those of the following turn.
// On return x holds the raw scores of step `next` and the reference point is rebased for it.
// MASKED: `vlim_cur` = tokens of step cur visible to any column of this wavefront,
// `limit_next` = tokens of step next visible to this lane's column.
template <bool MASKED, class IssueK, class IssueV, class Mid, class Lookup>
__device__ inline void pipeline_turn(ColumnState &st, float (&x)[16], bf16x8 (&ka_lo)[4], uint2 (&va0)[4][2],
                                     const unsigned char *krow1, const unsigned char *krow2,
                                     const unsigned char *sv_cur, const unsigned char *sv_next, const int (&voff)[4],
                                     const bf16x8 (&qb)[8], float scale_log2e, int vlim_cur, int limit_next, int half,
                                     int c, const IssueK &issue_k, const IssueV &issue_v, const Mid &mid, const Lookup &lookup) {
    const float neg_m = -st.m;
    float arg[16], pf[16], pair[8];
    uint32_t w[8];
    bf16x8 ka_hi[4];
    uint2 va1[4][2];
    floatx16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;

    // The softmax arithmetic of score pair P goes through four stages placed in different chunks,
    // so that no instruction waits for the result of the one in front of it: exponent arguments,
    // exponentials, rounding to bf16 plus the pair's sum, and the addition to the normaliser.
#define KVC_ARG(P)                                                           \
    arg[2 * (P)] = __builtin_fmaf(x[2 * (P)], scale_log2e, neg_m);           \
    arg[2 * (P) + 1] = __builtin_fmaf(x[2 * (P) + 1], scale_log2e, neg_m)
#define KVC_EXP(P)                                        \
    pf[2 * (P)] = __builtin_amdgcn_exp2f(arg[2 * (P)]);   \
    pf[2 * (P) + 1] = __builtin_amdgcn_exp2f(arg[2 * (P) + 1])
#define KVC_ROUND(P)                                \
    w[P] = pack_bf16(pf[2 * (P)], pf[2 * (P) + 1]); \
    pair[P] = pf[2 * (P)] + pf[2 * (P) + 1]
#define KVC_SUM(P) st.lsum += pair[P]
#define KVC_QK_LO(J)                                                          \
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka_lo[J], qb[J], s, 0, 0, 0); \
    ka_hi[J] = read_k_operand<4 + (J)>(krow1, half, c)
#define KVC_QK_HI(J)                                                                \
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka_hi[J], qb[4 + (J)], s, 0, 0, 0); \
    ka_lo[J] = read_k_operand<J>(krow2, half, c);                                   \
    read_v_operand<0>(va0[J], sv_next + voff[J])

    KVC_PIN();
    KVC_QK_LO(0); KVC_ARG(0); KVC_ARG(1); KVC_EXP(0);
    KVC_PIN();
    KVC_QK_LO(1); KVC_ARG(2); KVC_EXP(1); KVC_ROUND(0);
    KVC_PIN();
    KVC_QK_LO(2); KVC_ARG(3); KVC_EXP(2); KVC_ROUND(1); KVC_SUM(0);
    KVC_PIN();
    KVC_QK_LO(3); KVC_EXP(3); KVC_ROUND(2); KVC_SUM(1); KVC_ARG(4);
    KVC_PIN();
    KVC_ROUND(3);
    const uint4 pw0 = {w[0], w[1], w[2], w[3]};
    const bf16x8 pb0 = __builtin_bit_cast(bf16x8, pw0);

#define KVC_PV0(B)                                                                                        \
    if (MASKED) mask_v_operand<0>(va0[B], vlim_cur, half);                                                \
    st.acc[B] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(va0[B]), pb0, st.acc[B], 0, 0, 0);     \
    read_v_operand<1>(va1[B], sv_cur + voff[B])
    KVC_PV0(0); KVC_SUM(2); KVC_ARG(5); KVC_EXP(4); KVC_SUM(3);
    KVC_PIN();
    KVC_PV0(1); KVC_ARG(6); KVC_EXP(5); KVC_ROUND(4);
    KVC_PIN();
    KVC_PV0(2); KVC_ARG(7); KVC_EXP(6); KVC_ROUND(5); KVC_SUM(4);
    KVC_PIN();
    KVC_PV0(3); KVC_EXP(7); KVC_ROUND(6); KVC_SUM(5);
    KVC_PIN();
    mid();  // the workgroup's half-turn barrier: the other group of wavefronts changes phase here too
    KVC_PIN();

    lookup();  // block id for the loads of the next turn: half a turn for the scalar load to return
    KVC_QK_HI(0); KVC_ROUND(7); KVC_SUM(6);
    KVC_PIN();
    const uint4 pw1 = {w[4], w[5], w[6], w[7]};
    const bf16x8 pb1 = __builtin_bit_cast(bf16x8, pw1);
    KVC_QK_HI(1); KVC_SUM(7);
    KVC_PIN();
    KVC_QK_HI(2);
    KVC_PIN();
    KVC_QK_HI(3);
    KVC_PIN();

    // chunks 12 .. 15 also take the raw scores of step next (masked if need be) and their max
#define KVC_PV1(B)                                                                                        \
    if (MASKED) mask_v_operand<1>(va1[B], vlim_cur, half);                                                \
    st.acc[B] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(va1[B]), pb1, st.acc[B], 0, 0, 0)
    KVC_PV1(0);
    issue_k();
    KVC_PIN();
    KVC_PV1(1);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        x[v] = s[v];
        if (MASKED && 8 * (v >> 2) + 4 * half + (v & 3) >= limit_next) x[v] = -INFINITY;
    }
    const float m0 = max3(x[0], x[1], x[2]), m1 = max3(x[3], x[4], x[5]), m2 = max3(x[6], x[7], x[8]);
    KVC_PIN();
    KVC_PV1(2);
    issue_v();
    const float m3 = max3(x[9], x[10], x[11]), m4 = max3(x[12], x[13], x[14]);
    KVC_PIN();
    KVC_PV1(3);
    const float m5 = max3(m0, m1, m2), m6 = max3(m3, m4, x[15]);
    float lane_max;
    asm("v_max_f32 %0, %1, %2" : "=v"(lane_max) : "v"(m5), "v"(m6));
    rebase(st, lane_max, scale_log2e);
#undef KVC_ARG
#undef KVC_EXP
#undef KVC_SUM
#undef KVC_ROUND
#undef KVC_QK_LO
#undef KVC_QK_HI
#undef KVC_PV0
#undef KVC_PV1
}

// HEADS = 2: the 32 columns of a wavefront are 16 query rows x 2 heads of one KV head (even GQA
// groups); HEADS = 1: 32 query rows of one head.  GROUPS = 1: workgroups of four wavefronts, two
// per compute unit.  GROUPS = 2: workgroups of two groups of four wavefronts, one per compute
// unit; the groups run half a turn apart (see below).  Either way a SIMD holds two wavefronts.
// SPLIT (with GROUPS = 2): the two groups hold the same query rows, those of a four-wavefront workgroup, and
// share the steps of long contexts: group 0 walks the first `cut` of them, group 1 the rest, each with a ring
// of stages of its own, and the parts meet in LDS at the end (log-sum-exp rule).  Of short contexts group 1
// ends at once.  For launches with too few workgroups to fill the device, where a four-wavefront workgroup would
// run one wavefront per SIMD: 256 rows at the end of 12000 tokens, 32 / 8 heads, 172 -> 138 us, 64 rows of 4000
// tokens 63.6 -> 53.7 us, 300 rows of 1000 tokens twice 24 -> 22.4 us.  The groups run in
// step: half a turn apart the first case took 131 us, but the barrier in the middle of a turn cost short contexts,
// which only group 0 walks, 25 ns per step, and a branch around it (154 us) or a second copy of the loop
// (spills, 217 us) costs more.
// SMALL: block_size < 8.
template <bool SMALL, int GROUPS, int HEADS, bool SPLIT>
__global__ __launch_bounds__(256 * GROUPS, 3 - GROUPS) void pa_prefill_mfma32_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k_cache,
    const uint16_t *__restrict__ v_cache, const int32_t *__restrict__ block_tables,
    const int32_t *__restrict__ context_lens, const int32_t *__restrict__ q_start,
    uint16_t *__restrict__ out, PrefillParams p, int query_tiles, int fold_at, int fold_ranked, int rank_from) {
    static_assert(!SPLIT || GROUPS == 2, "the context is split between two groups");
    constexpr int kParts = SPLIT ? 2 : 1;
    constexpr int kShared = GROUPS / kParts;        // groups that share a ring of stages
    __shared__ __attribute__((aligned(1024))) unsigned char s_kv[kParts][kKStages + kVStages][kStageBytes];
    constexpr int kWaveRows = 32 / HEADS;           // query rows of a wavefront: column c = kWaveRows * head + row
    constexpr int kTileRows = 4 * kWaveRows * kShared;  // query rows of a workgroup
    constexpr int kLoads = 2 / kShared;             // 1 KiB loads of K (and of V) per wavefront and step
    constexpr int kWavesPerTile = 2 * kShared;      // wavefronts that share a 16-row tile of a step

    // blockIdx.x = head chunk + chunks * (seq + num_seqs * order); the longest query tiles come
    // first, and from `fold_at` on the shortest: when every workgroup is resident at once, the two
    // that share a compute unit are then a long and a short one.  With a context of `rank_from` tokens or more in
    // the batch (0: never) the same order is taken over the tiles of all sequences by the steps they walk,
    // which only the device knows.
    const int chunks = p.num_q_heads / HEADS;
    const int chunk = blockIdx.x % chunks, index = blockIdx.x / chunks;
    const int head0 = chunk * HEADS;
    const int kvh = head0 / p.group;

    int n = index % p.num_seqs;
    const int order = index / p.num_seqs;
    int qtile = order < fold_at ? query_tiles - 1 - order : order - fold_at;
    int S = context_lens[n], qs = q_start[n], Qn = q_start[n + 1] - qs;
    if (rank_from > 0) {
        const int l = threadIdx.x & 63;
        bool rank_all = false;  // what every workgroup asks in the same way
        if (p.num_seqs <= 8) {  // scalar loads that travel with those above
            for (int i = 0; i < p.num_seqs; i += 4)
#pragma unroll
                for (int u = 0; u < 4; ++u) rank_all |= context_lens[min(i + u, p.num_seqs - 1)] >= rank_from;
        } else {
            rank_all = __ballot(context_lens[l % p.num_seqs] >= rank_from) != 0;
        }
        if (rank_all) {  // every (sequence, query tile) sits in a lane
            const int items = p.num_seqs * query_tiles, n_l = l % p.num_seqs, t_l = l / p.num_seqs;
            const int S_l = context_lens[n_l], qs_l = q_start[n_l], Qn_l = q_start[n_l + 1] - qs_l;
            int steps = 0;
            if (l < items && t_l * kTileRows < Qn_l && Qn_l <= S_l)
                steps = (S_l - Qn_l + min(Qn_l, (t_l + 1) * kTileRows) - 1) / kStepTokens + 1;
            int rank = 0;
            for (int j = 0; j < items; ++j) {
                const int o = __builtin_amdgcn_readlane(steps, j);
                rank += o > steps || (o == steps && j < l);
            }
            const uint64_t mine = __ballot(steps > 0 && rank == (index < fold_ranked ? index : items - 1 - (index - fold_ranked)));
            if (mine == 0) return;  // uniform over the workgroup
            const int it = __builtin_ctzll(mine);
            n = it % p.num_seqs;
            qtile = it / p.num_seqs;
            S = __builtin_amdgcn_readlane(S_l, it);
            qs = __builtin_amdgcn_readlane(qs_l, it);
            Qn = __builtin_amdgcn_readlane(Qn_l, it);
        }
    }
    if (qtile * kTileRows >= Qn || Qn > S) return;  // uniform over the workgroup

    const int tid = threadIdx.x;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int group = wave_id >> 2;  // GROUPS = 2: wavefronts w and w + 4 share a SIMD; group 1 runs half a turn behind group 0
    const int wave = SPLIT ? wave_id & 3 : wave_id;  // among the wavefronts that share a ring
    unsigned char *const s_k = &s_kv[SPLIT ? group : 0][0][0], *const s_v = s_k + kKStages * kStageBytes;
    const int half = lane >> 5, c = lane & 31;
    const int r = c % kWaveRows;  // query row of the column inside the wavefront's rows
    const int my_head = head0 + c / kWaveRows;

    // tiles and steps this workgroup walks (up to the position of its last query row)
    const int last_pos = S - Qn + min(Qn, qtile * kTileRows + kTileRows) - 1;
    const int all_steps = last_pos / kStepTokens + 1;
    const int cut = SPLIT && all_steps >= kMinSplitSteps ? (all_steps + 1) / 2 : all_steps;  // group 0's share
    const int s0 = SPLIT && group == 1 ? cut : 0;              // first step of this wavefront's part
    const int wg_steps = SPLIT && group == 1 ? all_steps - cut : cut;  // and its number of steps
    if (SPLIT && wg_steps == 0) return;  // group 1 of a short context; ended wavefronts do not count at barriers
    constexpr bool phased = GROUPS == 2 && !SPLIT;  // the groups run half a turn apart
    const int32_t *table = block_tables + size_t(n) * p.max_blocks_per_seq;

    // wavefronts past the last query row still load and synchronise, they just never compute
    const int i0 = qtile * kTileRows + kWaveRows * wave;  // first query row of this wavefront
    const bool active = i0 < Qn;
    const int nrows = active ? min(kWaveRows, Qn - i0) : 1;
    const int row = min(r, nrows - 1);      // lanes past the last query row shadow it
    const int p0 = S - Qn + (active ? i0 : 0);  // position of row 0
    const int my_pos = p0 + row;
    const int wave_vis = p0 + nrows;        // tokens visible to some column of this wavefront
    const int free_steps = (p0 + 1) / kStepTokens - s0;  // steps of the part whose every token every column sees

    bf16x8 qb[8];
    {
        const uint16_t *qrow = q + (size_t(qs + (active ? i0 : 0) + row) * p.num_q_heads + my_head) * D + 8 * half;
#pragma unroll
        for (int j = 0; j < 8; ++j) qb[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(qrow + 16 * j));
    }

    // Token 0 is in the first step, so every column starts with a finite score there.  Group 1's first step may
    // hide all its tokens from a column: its reference point starts at the lowest finite value, the weights are 0.
    ColumnState st;
    st.reset(SPLIT ? -FLT_MAX : -INFINITY);

    // ---- this wavefront's share of a step's rows: 4 * kLoads consecutive rows of the 32 (inside
    // one 16-row tile of the step), kLoads loads of 4 rows for K and as many for V.  Lane l of
    // load i writes LDS chunk l % 16 of the share's row 4 * i + l / 16; the chunk it fetches for
    // that place follows from the stage layouts.
    const size_t head_bytes = size_t(p.block_size) * D * 2;
    const size_t block_bytes = head_bytes * p.num_kv_heads;
    const unsigned char *k_head = reinterpret_cast<const unsigned char *>(k_cache) + size_t(kvh) * head_bytes;
    const unsigned char *v_head = reinterpret_cast<const unsigned char *>(v_cache) + size_t(kvh) * head_bytes;
    const int sub_mask = (1 << p.tiles_per_block_log2) - 1;
    const int my_tile = wave / kWavesPerTile;       // tile of the step this wavefront loads from
    const int lrow = 4 * kLoads * (wave % kWavesPerTile) + (lane >> 4);  // row inside the tile of load 0 (load 1: + 4)
    const int lchunk = lane & 15;
    const int brow = lrow & (p.block_size - 1);  // in its block, where that holds 8 tokens (16 or more: lrow)
    const uint32_t k_off = brow * 256 + ((lchunk ^ lrow) << 4);
    const uint32_t k_off1 = (brow + 4) * 256 + ((lchunk ^ (lrow + 4)) << 4);
    const uint32_t v_off = brow * 256 + ((4 * (((lchunk >> 2) - lrow) & 3) + (lchunk & 3)) << 4);  // load 1: + 1024
    const uint32_t lds_k0 = uint32_t(reinterpret_cast<uintptr_t>(s_k)) + 1024 * kLoads * wave;
    const uint32_t lds_v0 = uint32_t(reinterpret_cast<uintptr_t>(s_v)) + 1024 * kLoads * wave;

    // Blocks of 8 tokens and more: the block id of the wavefront's rows (8 or 4 consecutive ones, inside one
    // block) is uniform, it comes through the scalar cache one turn before the loads that use it.  Rows past the
    // last visible token repeat its block (never used unmasked).  Smaller blocks: a / b are the blocks of
    // this lane's row in loads 0 / 1.  (Four chunks of 512 rows on 8-token blocks, contexts up to 4000, 32 / 8
    // heads: 112 us; with a table load per lane, which drains the wavefront's loads in flight, 126 us.)
    const int share_row = 4 * kLoads * (wave % kWavesPerTile);
    struct Ids { int a, b; };
    auto ids_of = [&](int step) __attribute__((always_inline)) -> Ids {
        Ids id;
        if (SMALL) {
            const int tok = min((2 * (s0 + step) + my_tile) * kTileTokens + lrow, last_pos);
            id.a = table[tok >> p.block_size_log2];
            id.b = kLoads == 2 ? table[min(tok + 4, last_pos) >> p.block_size_log2] : 0;
        } else {
            const int tok = min((2 * (s0 + step) + my_tile) * kTileTokens + share_row, last_pos);
            id.a = __builtin_amdgcn_readfirstlane(table[tok >> p.block_size_log2]);
            id.b = (tok >> 4) & sub_mask;
        }
        return id;
    };
    // load this wavefront's K (V) rows of step `src` (the one `id` was looked up for) into a stage
    auto issue_rows = [&](const unsigned char *head, uint32_t dst, uint32_t off, uint32_t off1, int src, const Ids &id)
                          __attribute__((always_inline)) {
        if (SMALL) {
            const int tok = min((2 * (s0 + src) + my_tile) * kTileTokens + lrow, last_pos);
            load_lane_to_lds(head + size_t(id.a) * block_bytes + size_t(tok & (p.block_size - 1)) * 256 + (off & 255), dst);
            if (kLoads == 2) {
                const int tok1 = min(tok + 4, last_pos);
                load_lane_to_lds(head + size_t(id.b) * block_bytes + size_t(tok1 & (p.block_size - 1)) * 256 + (off1 & 255),
                                 dst + 1024);
            }
        } else {
            const unsigned char *tile = head + size_t(unsigned(id.a)) * block_bytes + size_t(id.b) * (kTileTokens * 256);
            if (kLoads == 2) load_rows_to_lds(tile, off, off1 - 1024, dst);
            else load_row_group_to_lds(tile, off, dst);
        }
    };
    auto issue_k = [&](int kst, int src, const Ids &id) __attribute__((always_inline)) {
        issue_rows(k_head, __builtin_amdgcn_readfirstlane(lds_k0 + kst * kStageBytes), k_off, k_off1, src, id);
    };
    auto issue_v = [&](int vst, int src, const Ids &id) __attribute__((always_inline)) {
        issue_rows(v_head, __builtin_amdgcn_readfirstlane(lds_v0 + vst * kStageBytes), v_off, v_off + 1024, src, id);
    };

    // Rows of step j live in K stage j % 4 and V stage j % 4.  Turn s requests the K rows of step
    // s+4 (over those of step s) and the V rows of step s+3 (over those of step s-1), multiplies
    // with operands of steps s+1 (K) and s (V) and reads operands of steps s+1, s+2 (K) and s, s+1
    // (V).  Before the barrier that ends it, a wavefront waits for its own loads of turn s-1 and
    // for its LDS reads.  The workgroup meets at a barrier twice per turn, and group 1 of its
    // wavefronts runs half a turn behind group 0: while one wavefront of a SIMD is in the first,
    // vector-heavy half of a turn the other is in the second, matrix-heavy half.  A stage is
    // overwritten, at the earliest, two barriers after the last wavefront has waited for its
    // reads of it, and read, at the earliest, after the barrier that follows the wait of the last
    // wavefront for its loads into it.  Past the last step the last one is loaded again (unused):
    // the loops stay branch free.
    Ids ids_v;
    {
        const Ids i0s = ids_of(0), i1s = ids_of(min(1, wg_steps - 1)), i2s = ids_of(min(2, wg_steps - 1));
        ids_v = ids_of(min(3, wg_steps - 1));
        issue_k(0, 0, i0s);
        issue_v(0, 0, i0s);
        issue_k(1, min(1, wg_steps - 1), i1s);
        issue_v(1, min(1, wg_steps - 1), i1s);
        issue_k(2, min(2, wg_steps - 1), i2s);
        issue_v(2, min(2, wg_steps - 1), i2s);
        issue_k(3, min(3, wg_steps - 1), ids_v);
    }
    Ids ids_k = ids_of(min(4, wg_steps - 1));
    wait_loads_but<kLoads>();  // steps 0 .. 2 have arrived
    // A use of the Q operand on this side of the barrier: without one the compiler sinks its
    // loads into the path of the active wavefronts, behind the barrier, where nothing hides them.
#pragma unroll
    for (int j = 0; j < 8; ++j) asm volatile("" : "+v"(qb[j]));
    __syncthreads();

    int s = 0;
    // PH = s % 4 (a literal in the unrolled loop: every LDS address of the turn is then a per-lane
    // register plus an immediate)
#define KVC_TURN_BEGIN(PH)                                                                        \
    const int ph = (PH);                                                                          \
    const int src_k = min(s + 4, wg_steps - 1), src_v = min(s + 3, wg_steps - 1);                 \
    const Ids idk = ids_k, idv = ids_v;                                                           \
    auto turn_k = [&]() __attribute__((always_inline)) { issue_k(ph, src_k, idk); };              \
    auto turn_v = [&]() __attribute__((always_inline)) {                                          \
        issue_v((ph + 3) & 3, src_v, idv);                                                        \
        ids_v = idk;                                                                              \
    };                                                                                            \
    auto turn_lookup = [&]() __attribute__((always_inline)) { ids_k = ids_of(min(s + 5, wg_steps - 1)); }
#define KVC_TURN_END()     \
    wait_loads_but<2 * kLoads>();   \
    turn_barrier()

    // Group 0's share may be a step longer than group 1's.
    auto even_out = [&]() __attribute__((always_inline)) {
        if (group == 1)
            for (int i = wg_steps; i < cut; ++i) phase_barrier();
    };

    // Every wavefront of the workgroup passes one more barrier here, two per turn, and one to
    // set group 1 back by half a turn (group 0 passes its counterpart after its last turn).  A
    // wavefront without query rows only loads and synchronises.
    if (!active) {
        __syncthreads();
        if (phased && group == 1) phase_barrier();
        for (; s < wg_steps; ++s) {
            KVC_TURN_BEGIN(s & 3);
            if (phased) phase_barrier();
            turn_lookup();
            turn_k();
            turn_v();
            KVC_TURN_END();
        }
        if (phased && group == 0) phase_barrier();
        wait_loads_but<0>();
        if (SPLIT && cut < all_steps) {  // as the others below
            even_out();
            __syncthreads();
            __syncthreads();
        }
        return;
    }

    const unsigned char *k_lane = s_k + c * 256;  // this lane's K row inside a stage
    int voff[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) voff[b] = v_lane_offset(b, half, c);
    float x[16];
    bf16x8 ka_lo[4];
    uint2 va0[4][2];
    {  // scores of step 0, then the operands turn 0 starts from
        floatx16 sc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = 0.f;
        bf16x8 ka[8];
        ka[0] = read_k_operand<0>(k_lane, half, c); ka[1] = read_k_operand<1>(k_lane, half, c);
        ka[2] = read_k_operand<2>(k_lane, half, c); ka[3] = read_k_operand<3>(k_lane, half, c);
        ka[4] = read_k_operand<4>(k_lane, half, c); ka[5] = read_k_operand<5>(k_lane, half, c);
        ka[6] = read_k_operand<6>(k_lane, half, c); ka[7] = read_k_operand<7>(k_lane, half, c);
#pragma unroll
        for (int j = 0; j < 8; ++j) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[j], qb[j], sc, 0, 0, 0);
        rebase(st, take_scores<true>(x, sc, my_pos + 1 - s0 * kStepTokens, half), p.scale_log2e);
        const unsigned char *krow = k_lane + kStageBytes;
        ka_lo[0] = read_k_operand<0>(krow, half, c); ka_lo[1] = read_k_operand<1>(krow, half, c);
        ka_lo[2] = read_k_operand<2>(krow, half, c); ka_lo[3] = read_k_operand<3>(krow, half, c);
#pragma unroll
        for (int b = 0; b < 4; ++b) read_v_operand<0>(va0[b], s_v + voff[b]);
    }
    __syncthreads();  // K stage 0 has been read: turn 0 may load step 4 over it
    if (phased && group == 1) phase_barrier();

    // The turns below the diagonal first (no mask), unrolled by the four phases of the stage
    // rings, then the one to three turns that the causal mask touches.
    const unsigned char *v_base = s_v;
    auto mid = []() __attribute__((always_inline)) {
        if (phased) phase_barrier();
    };
#define KVC_TURN(MASKED, PH, VLIM, LIMIT)                                                                      \
    {                                                                                                          \
        KVC_TURN_BEGIN(PH);                                                                                    \
        pipeline_turn<MASKED>(st, x, ka_lo, va0, k_lane + ((ph + 1) & 3) * kStageBytes,                        \
                              k_lane + ((ph + 2) & 3) * kStageBytes, v_base + ph * kStageBytes,                \
                              v_base + ((ph + 1) & 3) * kStageBytes, voff, qb, p.scale_log2e, VLIM, LIMIT,     \
                              half, c, turn_k, turn_v, mid, turn_lookup);                                      \
        KVC_TURN_END();                                                                                        \
        ++s;                                                                                                   \
    }
    const int plain_turns = min(max(free_steps - 1, 0), wg_steps);
    while (s + 4 <= plain_turns) {
        KVC_TURN(false, 0, kStepTokens, kStepTokens)
        KVC_TURN(false, 1, kStepTokens, kStepTokens)
        KVC_TURN(false, 2, kStepTokens, kStepTokens)
        KVC_TURN(false, 3, kStepTokens, kStepTokens)
    }
    while (s < plain_turns) KVC_TURN(false, s & 3, kStepTokens, kStepTokens)
    // steps past the last token that any row of this wavefront sees carry no weight for it: it
    // only loads and synchronises during the workgroup's remaining turns
    const int live_turns = min(wg_steps, (wave_vis + kStepTokens - 1) / kStepTokens - s0);
    while (s < live_turns)
        KVC_TURN(true, s & 3, wave_vis - (s0 + s) * kStepTokens, my_pos + 1 - (s0 + s + 1) * kStepTokens)
    for (; s < wg_steps; ++s) {
        KVC_TURN_BEGIN(s & 3);
        mid();
        turn_lookup();
        turn_k();
        turn_v();
        KVC_TURN_END();
    }
#undef KVC_TURN
#undef KVC_TURN_BEGIN
#undef KVC_TURN_END
    if (phased && group == 0) phase_barrier();
    wait_loads_but<0>();  // nothing may still be landing in LDS when the workgroup's LDS is handed on

    // lane (half, c) holds O[query row i0 + r][my_head][32*b + 8*a + 4*half .. +3] in acc[b][4a .. 4a+3]
    uint16_t *const dst = out + (size_t(qs + i0 + r) * p.num_q_heads + my_head) * D + 4 * half;
    const float lsum = sum_over_halves(st.lsum);
    if (SPLIT && cut < all_steps) {
        // the parts meet: each group hands over two dim blocks and finishes the other two
        even_out();
        __syncthreads();  // every wavefront is past its last load and LDS read
        float *const hand = reinterpret_cast<float *>(&s_kv[0][0][0]) + wave * (2 * 34 * 64) + lane;  // [wave][group][32 + 2][64]
        float *const mine = hand + group * (34 * 64);
        const float *const theirs = hand + (1 - group) * (34 * 64);
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) mine[(16 * b + v) * 64] = group == 0 ? st.acc[2 + b][v] : st.acc[b][v];
        mine[32 * 64] = st.m;
        mine[33 * 64] = lsum;
        __syncthreads();
        const float m_o = theirs[32 * 64], l_o = theirs[33 * 64];
        const float M = fmaxf(st.m, m_o);
        const float w_m = __builtin_amdgcn_exp2f(st.m - M), w_o = __builtin_amdgcn_exp2f(m_o - M);
        const float inv = 1.0f / (w_m * lsum + w_o * l_o);
        if (r < nrows) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    float o[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int v = 4 * a + i;
                        o[i] = (w_m * (group == 0 ? st.acc[b][v] : st.acc[2 + b][v]) + w_o * theirs[(16 * b + v) * 64]) * inv;
                    }
                    *reinterpret_cast<uint2 *>(dst + 32 * (2 * group + b) + 8 * a) = uint2{pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3])};
                }
        }
        return;
    }
    const float inv = 1.0f / lsum;
    if (r < nrows) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                uint2 w;
                w.x = pack_bf16(st.acc[b][4 * a] * inv, st.acc[b][4 * a + 1] * inv);
                w.y = pack_bf16(st.acc[b][4 * a + 2] * inv, st.acc[b][4 * a + 3] * inv);
                *reinterpret_cast<uint2 *>(dst + 32 * b + 8 * a) = w;
            }
    }
}

// Calls that the kernel of 64-column wavefronts takes (pa_prefill_wide.h), by heads per workgroup; 0: none.  One workgroup
// of it fills a compute unit, so that a launch needs about 360 of them before the longest tiles no longer stand alone.
// 32 columns / 64 columns, us, one request and 32 / 8 heads: 2500 tokens (320 workgroups) 58.7 / 64.3, 3000 (376) 81.7 /
// 78.0, 4096 130 / 119; 64 / 8 heads: 1000 tokens (256) 27.6 / 31.8, 1500 (384) 50.0 / 44.4; 8 / 2 heads: 4096 (128) 56 / 88,
// four of 4096 120 / 117.  Short requests pay for the start and end of a tile, 15000 cycles against 1400 per 32 tokens: four of
// 1500 tokens, 32 / 8 heads, 77.8 / 80.1, of 2048 131 / 129, of 3000 260 / 251; with two workgroups per KV head, which share
// its rows in L2, four of 1000 81.1 / 80.7 and of 1500 156 / 151 (64 / 8 heads).  Two heads per workgroup (16 / 8 heads): four
// of 2500 96.6 / 99.9, 4096 240 / 228; one request of 8000 244 / 219.  One head: one request of 4096 132 / 129 (32 / 32), 125 /
// 118 (28 / 4), but four of 4096 490 / 488 and 415 / 422.  Batches with a few long requests among short ones stay here.
int wide_heads(const PrefillParams &p, int total_q) {
    const int heads = p.group % 4 == 0 ? 4 : p.group % 2 == 0 ? 2 : 1;
    const int64_t tile_rows = 256 / heads;
    if (p.num_q_heads / heads * ((total_q + tile_rows - 1) / tile_rows) < 360) return 0;
    if (total_q < int64_t(p.num_seqs) * p.max_query_tiles * 32) return 0;  // on average half the longest
    const int least = heads == 4 ? (p.group % 8 == 0 ? 16 : 32) : heads == 2 ? 48 : 40;  // 64-row tiles of the longest
    return p.max_query_tiles >= least && (heads > 1 || p.num_seqs == 1) ? heads : 0;
}

}  // namespace

// Needs a positive scale (the max is taken over raw scores).  heads_per_chunk = 2: two heads of a
// KV head per wavefront (even group sizes); 1: one head, twice the query rows.
hipError_t launch_prefill_mfma32(const void *q, const void *k_cache, const void *v_cache,
                                 const int32_t *block_tables, const int32_t *context_lens,
                                 const int32_t *q_start, void *out, const PrefillParams &p, int total_q,
                                 hipStream_t stream) {
    switch (wide_heads(p, total_q)) {
        case 4: return launch_prefill_wide<4>(q, k_cache, v_cache, block_tables, context_lens, q_start, out, p, stream);
        case 2: return launch_prefill_wide<2>(q, k_cache, v_cache, block_tables, context_lens, q_start, out, p, stream);
        case 1: return launch_prefill_wide<1>(q, k_cache, v_cache, block_tables, context_lens, q_start, out, p, stream);
    }
    const auto *qq = static_cast<const uint16_t *>(q);
    const auto *kk = static_cast<const uint16_t *>(k_cache);
    const auto *vv = static_cast<const uint16_t *>(v_cache);
    auto *oo = static_cast<uint16_t *>(out);
    const int heads = p.heads_per_chunk;
    const int rows64 = 2 / heads;  // 64-row units in the query rows of four wavefronts
    // Two groups per workgroup pay off (by a few percent) for long recomputations with workgroups
    // enough to keep every compute unit busy for several rounds; up to about 2048 query rows per
    // sequence the finer grain of four-wavefront workgroups wins, whatever the batch (measured).
    const auto tiles_of = [&](int groups) { return (p.max_query_tiles + rows64 * groups - 1) / (rows64 * groups); };
    const int64_t wide_grid = int64_t(p.num_q_heads / heads) * p.num_seqs * tiles_of(2);
    const bool wide = wide_grid >= 2 * 256 && p.max_query_tiles >= 48;
    const bool small = p.block_size < 8;
    const int query_tiles = tiles_of(wide ? 2 : 1);  // max_query_tiles counts 64-row tiles
    const int64_t grid = int64_t(p.num_q_heads / heads) * p.num_seqs * query_tiles;
    // at most one workgroup per compute unit (up to two the finer grain of plain ones wins: 2048 tokens 45.6 us
    // plain, 46.2 us split; four chunks of 512 rows 112 / 118 us), and only where the block table reaches far enough
    // for a share: the second group's start costs a short request up to 0.3 us (642 tokens, MHA: 17.3 / 17.6 us)
    const bool split = !wide && !small && grid <= kNumCUs &&
                       int64_t(p.max_blocks_per_seq) * p.block_size > (kMinSplitSteps - 1) * kStepTokens;
    // A grid that fits the device at once (two workgroups of four wavefronts per compute unit)
    // gets the second half of its query tiles in rising order (a few percent on one short request).
    // Chunks of several sequences: what a tile walks depends on its sequence's context, which only the device knows.
    // Up to 64 tiles are ranked there; grids that fit at once then put the shortest ranks beside the longest.  32 / 8
    // heads, 16-token blocks, in given order / ranked: four chunks of 512 rows, contexts of 2000 to 4000, 104 to 112 / 92 to
    // 107 us; six of 600 rows, 8000: 393 to 411 / 365 to 391 us; three of 400, 7000: 138 to 154 / 124 to 147 us; five of 200,
    // 6000: 111 to 127 / 102 to 109 us.  Recomputations, whose tiles are in order anyway, lose by it (three of 1000
    // tokens 39.0 / 44.2 us, sixteen of 220 27.2 / 34.1 us), so the workgroups rank only if some context of the batch is
    // four times as long as the longest chunk may be: under a 4096-token table these take 39.5 and 27.8 us.  A table
    // that reaches less far says so before the launch, and launches that fill no compute unit twice do without.
    const int64_t items = int64_t(p.num_seqs) * query_tiles;
    const int chunks = p.num_q_heads / heads;
    const int64_t chunk_reach = 4 * 64 * int64_t(p.max_query_tiles);
    const int rank_from = p.num_seqs > 1 && items <= 64 && grid > kNumCUs &&
                          int64_t(p.max_blocks_per_seq) * p.block_size >= chunk_reach ? int(chunk_reach) : 0;
    const int fold_at = (!wide && grid <= 2 * kNumCUs) ? (query_tiles + 1) / 2 : query_tiles;
    const int fold_ranked = grid <= 2 * kNumCUs ? std::max(1, std::min(int(items), kNumCUs / chunks)) : int(items);
    const dim3 g{unsigned(grid)}, b(wide || split ? 512 : 256);
#define KVC_LAUNCH(SMALL, GROUPS, HEADS, SPLIT)                                                                        \
    pa_prefill_mfma32_kernel<SMALL, GROUPS, HEADS, SPLIT><<<g, b, 0, stream>>>(qq, kk, vv, block_tables, context_lens, \
                                                                                q_start, oo, p, query_tiles, fold_at, fold_ranked, rank_from)
#define KVC_LAUNCH_SHAPE(SMALL, HEADS)                       \
    do {                                                     \
        if (wide) KVC_LAUNCH(SMALL, 2, HEADS, false);        \
        else if (split) KVC_LAUNCH(false, 2, HEADS, true);   \
        else KVC_LAUNCH(SMALL, 1, HEADS, false);             \
    } while (0)
    if (small && heads == 2) KVC_LAUNCH_SHAPE(true, 2);
    else if (small) KVC_LAUNCH_SHAPE(true, 1);
    else if (heads == 2) KVC_LAUNCH_SHAPE(false, 2);
    else KVC_LAUNCH_SHAPE(false, 1);
#undef KVC_LAUNCH_SHAPE
#undef KVC_LAUNCH
    return hipGetLastError();
}

}  // namespace kvc

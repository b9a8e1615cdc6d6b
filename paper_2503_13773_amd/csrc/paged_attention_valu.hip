// Split-K partial kernel of paged decode attention on the vector ALUs (gfx950).
//
// Computes, for one (sequence, chunk of query heads sharing a KV head, partition of the
// context), the un-normalised softmax-weighted sum of V rows together with the running
// max and sum, reading K and V through the block table (block-allocated KV cache:
// paper Section 1 and 3.3.1).  It serves any supported shape: fp32 tensors, blocks of 1 or 2
// tokens, groups above 16, and at head_dim 64 the calls too small for the matrix-core kernels; other bf16
// shapes normally take those.  A context of several partitions is merged by the workgroup that finishes its last one
// (p.merge_here), or by the merge launch.
//
// Mapping: a token row of K or V is D*sizeof(T) bytes = LR lanes x 16 bytes, so one
// wavefront load covers TPL = 64/LR tokens, fully coalesced.  Each group of LR lanes
// keeps its own online-softmax state over the tokens it sees (no cross-lane traffic in
// the loop beyond the LR-lane dot-product reduction); the TPL groups, then the four to sixteen
// wavefronts, are merged with the log-sum-exp rule at the end.  Scores and softmax are in
// natural-log units, accumulation in fp32.
//
// What bounds small launches is the chain of one workgroup, and in it the instructions that are run once: they come from L2,
// so a merge written out for sixteen wavefronts in every thread, or an exponential (fp32: fifteen instructions) where one lane's
// would do, costs more than it computes.  fp32, 8 / 8 heads of 64, us: 4 x 256 tokens 4.9 with the groups merged pair by pair,
// 4.6 by one maximum and one exponential, 4.3 with a lane weighing each wavefront; 1 x 40 3.7 / 3.5 / 3.2.
//
// PREFILL variant (causal attention of several query positions per sequence, the recompute
// path of Section 2.5 / 3.5, for the calls the matrix-core prefill kernels do not take): a
// "sequence" of the grid is one query row; the row finds its sequence n by a search over
// q_start, attends to the first S_n - Qn + i + 1 tokens of n's block list in one partition and
// writes its normalised output directly.
#include <math.h>

#include <type_traits>

#include "kvc_internal.h"
#include "pa_merge_row.h"

namespace kvc {

namespace {

template <typename T>
struct Elem;

template <>
struct Elem<float> {
    static constexpr int kPerLane = 4;  // elements in 16 bytes
    __device__ static void load16(const float *p, float (&x)[4]) {
        const float4 v = *reinterpret_cast<const float4 *>(p);
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    }
    __device__ static float exp_(float x) { return expf(x); }
    __device__ static float to_out(float x) { return x; }
};

template <>
struct Elem<uint16_t> {  // bfloat16 bit patterns
    static constexpr int kPerLane = 8;
    __device__ static void load16(const uint16_t *p, float (&x)[8]) {
        const uint4 v = *reinterpret_cast<const uint4 *>(p);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[2 * i] = __uint_as_float(w[i] << 16);
            x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    __device__ static float exp_(float x) { return __expf(x); }
    __device__ static uint16_t to_out(float x) {  // round to nearest even
        uint32_t u = __float_as_uint(x);
        if ((u & 0x7fffffffu) > 0x7f800000u) return uint16_t((u >> 16) | 0x40u);
        u += 0x7fffu + ((u >> 16) & 1u);
        return uint16_t(u >> 16);
    }
};

// x + (x of lane l ^ OFF), for sums over aligned groups of lanes taken in the order OFF = 1, 2, 4, ...: before step
// OFF all lanes of an aligned group of OFF hold the same value, so any lane of the neighbouring group will do
// and the step is a lane permutation inside the vector ALU: a mirror of 8 or 16 lanes, or a swap of 16-lane rows.
// The sums are the same bits as with shuffles through the LDS pipe, whose latency a decode call of few
// workgroups waits for in every step (one sequence of 256 tokens, fp32, 16 / 4 heads of 128: 14.6 -> 10.4 us).
// Prefill has wavefronts enough to hide it and keeps the shuffles, which leave the vector ALU free (fp32, 1000 rows,
// 32 / 8 heads of 128: 503 us with shuffles, 566 us with permutations).
template <int LR>
__device__ inline float sum_over_row(float x) {  // LR = 8, 16 or 32 lanes of a token row
    x += lanes::permuted<lanes::kXor1>(x);
    x += lanes::permuted<lanes::kXor2>(x);
    x += lanes::permuted<lanes::kMirror8>(x);
    if constexpr (LR > 8) x += lanes::permuted<lanes::kMirror16>(x);
    if constexpr (LR > 16) {
        const lanes::Pair<float> b = lanes::pair_of<16>(x);
        x = b.first + b.second;
    }
    return x;
}

// Partials that another workgroup of the launch may merge travel by device-scope accesses, which go to the point of coherence
// of the XCDs' caches by themselves.
__device__ inline void store_device(float *p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <int N>
__device__ inline void load_device(const float *p, float (&x)[N]) {
    if constexpr (N == 2) {
        const uint64_t u = __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x[0] = __uint_as_float(uint32_t(u));
        x[1] = __uint_as_float(uint32_t(u >> 32));
    } else {
        x[0] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// UNROLL: tokens per lane group and loop trip (twice as many 16-byte loads in flight).  MERGE: the last partition of a row to
// finish merges it (an instance of its own: as a branch the code cost launches of one partition 0.03 us).  AHEAD: table entries
// are requested ahead of their use (see below).
template <typename T, int D, int GC, bool PREFILL, int WAVES, int UNROLL, bool MERGE, bool AHEAD>
__global__ __launch_bounds__(64 * WAVES) void pa_partial_valu_kernel(
    const T *__restrict__ q, const T *__restrict__ k_cache, const T *__restrict__ v_cache,
    const int32_t *__restrict__ block_tables, const int32_t *__restrict__ context_lens,
    const int32_t *__restrict__ q_start, int num_tables, int max_query_len,
    T *__restrict__ out, Workspace ws, AttnParams p) {
    using E = Elem<T>;
    constexpr int EPL = E::kPerLane;
    constexpr int LR = D / EPL;    // lanes per token row
    constexpr int TPL = 64 / LR;   // tokens per wavefront load
    static_assert(LR == 8 || LR == 16 || LR == 32, "a row is 128, 256 or 512 bytes");

    // blockIdx.x = head_chunk + chunks * (seq + num_seqs * partition): the partition index
    // varies slowest, so the (always busy) first partitions are dispatched first.
    const int chunks = p.num_q_heads / GC;
    const int item = blockIdx.x;
    const int hc = item % chunks;
    const int seq = (item / chunks) % p.num_seqs;
    const int part = item / (chunks * p.num_seqs);
    const int head0 = hc * GC;
    const int kvh = head0 / p.group;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int tg = lane / LR, c = lane % LR;
    const int tok0 = part * p.partition_tokens;
    constexpr int CH = TPL * UNROLL;  // tokens per wavefront per trip

    // AHEAD: the table entries of the tokens of a trip are requested before the context length is known, or under the K and V
    // loads of the trip before; entries past the context may be read, inside the table's row, but are never used.
    int blk[UNROLL];
    const int32_t *table = nullptr;
    auto look_up = [&](int base) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            blk[u] = table[min((base + u * TPL + tg) >> p.block_size_log2, p.max_blocks_per_seq - 1)];
    };
    int base = tok0 + wave * CH;
    float qf[GC][EPL];
    auto load_q = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < GC; ++g)
            E::load16(q + (size_t(seq) * p.num_q_heads + head0 + g) * D + c * EPL, qf[g]);
    };

    int ctx;  // context length of this item
    if (PREFILL) {
        // seq is a row of q: largest n with q_start[n] <= row (sequences without rows are skipped)
        int lo = 0, hi = num_tables;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (q_start[mid] <= seq) lo = mid; else hi = mid;
        }
        const int i = seq - q_start[lo], Qn = q_start[lo + 1] - q_start[lo], S = context_lens[lo];
        if (Qn > S || i >= max_query_len) return;
        ctx = S - Qn + i + 1;
        table = block_tables + size_t(lo) * p.max_blocks_per_seq;
    } else {
        table = block_tables + size_t(seq) * p.max_blocks_per_seq;
        if (AHEAD) {
            look_up(base);
            load_q();
        }
        ctx = min(context_lens[seq], p.max_context_len);
    }

    if (ctx <= 0) {  // empty context: a row of zeros, written by partition 0
        if (part == 0)
            for (int i = tid; i < GC * D; i += 64 * WAVES)
                out[(size_t(seq) * p.num_q_heads + head0) * D + i] = E::to_out(0.f);
        return;
    }
    if (tok0 >= ctx) return;
    const int tok1 = min(ctx, tok0 + p.partition_tokens);
    if (PREFILL || !AHEAD) {
        if (AHEAD) look_up(base);
        load_q();
    }

    float m[GC], l[GC], acc[GC][EPL];
#pragma unroll
    for (int g = 0; g < GC; ++g) {
        m[g] = -INFINITY;
        l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = 0.f;
    }

    const size_t head_stride = size_t(p.block_size) * D;               // elements per (block, kv head)
    const size_t block_stride = head_stride * p.num_kv_heads;

    // A trip of a wavefront.  MAY_END: it may reach past the end; the lanes of tokens there load the trip's first token again (or
    // the last one), whose V must not meet the weight 0, where it is an infinity or NaN.  One head per workgroup: every trip asks, which is
    // the least code in the shortest calls (fp32 of 64, 8 / 8 heads, 1 x 40 tokens 3.3 us, with the last trip apart 3.6; 4 x 256 4.49 and
    // 4.40); several: the last trip is code of its own (fp32 of 128, four heads, 40 x 256 25.2 us, asked in every trip 26.9).
    auto trip = [&](auto may_end, int base) __attribute__((always_inline)) {
        constexpr bool MAY_END = decltype(may_end)::value;
        float kf[UNROLL][EPL], vf[UNROLL][EPL];
        bool valid[UNROLL];
        const int first_block = AHEAD ? __builtin_amdgcn_readfirstlane(blk[0]) : 0;  // of token `base`, which is inside the context
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int t = base + u * TPL + tg;
            valid[u] = !MAY_END || t < tok1;
            const int tc = valid[u] ? t : AHEAD ? base : tok1 - 1;
            const int block = !AHEAD ? table[tc >> p.block_size_log2] : valid[u] ? blk[u] : first_block;
            const int slot = tc & (p.block_size - 1);
            const size_t off = size_t(block) * block_stride + kvh * head_stride + size_t(slot) * D + c * EPL;
            E::load16(k_cache + off, kf[u]);
            E::load16(v_cache + off, vf[u]);
        }
        if (AHEAD && base + WAVES * CH < tok1) look_up(base + WAVES * CH);  // wavefront-uniform
        if (MAY_END && base + CH > tok1) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
#pragma unroll
                for (int e = 0; e < EPL; ++e) vf[u][e] = valid[u] ? vf[u][e] : 0.f;
        }
#pragma unroll
        for (int g = 0; g < GC; ++g) {
            float s[UNROLL];
            float mx = -INFINITY;
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                float d = 0.f;
#pragma unroll
                for (int e = 0; e < EPL; ++e) d = fmaf(qf[g][e], kf[u][e], d);
                if constexpr (PREFILL) {
#pragma unroll
                    for (int off = 1; off < LR; off <<= 1) d += __shfl_xor(d, off);
                } else {
                    d = sum_over_row<LR>(d);
                }
                s[u] = valid[u] ? d * p.scale : -INFINITY;
                mx = fmaxf(mx, s[u]);
            }
            const float m_new = fmaxf(m[g], mx);
            const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // group has seen no token yet
            const float alpha = E::exp_(m[g] - m_ref);
            float psum = 0.f, pv[EPL];
#pragma unroll
            for (int e = 0; e < EPL; ++e) pv[e] = 0.f;
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const float pu = E::exp_(s[u] - m_ref);
                psum += pu;
#pragma unroll
                for (int e = 0; e < EPL; ++e) pv[e] = fmaf(pu, vf[u][e], pv[e]);
            }
            l[g] = fmaf(l[g], alpha, psum);
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[g][e] = fmaf(acc[g][e], alpha, pv[e]);
            m[g] = m_new;
        }
    };
    if constexpr (GC == 1) {
        for (; base < tok1; base += WAVES * CH) trip(std::true_type{}, base);
    } else {
        for (; base + CH <= tok1; base += WAVES * CH) trip(std::false_type{}, base);
        if (base < tok1) trip(std::true_type{}, base);
    }

    // merge the TPL lane groups of this wavefront (log-sum-exp rule): the maximum of all, one exponential, sums
    auto over_groups = [](float x, auto op) __attribute__((always_inline)) {
        if constexpr (LR <= 8) x = op(x, lanes::permuted<lanes::kRor8>(x));
        if constexpr (LR <= 16) {
            const lanes::Pair<float> a = lanes::pair_of<16>(x);
            x = op(a.first, a.second);
        }
        const lanes::Pair<float> b = lanes::pair_of<32>(x);
        return op(b.first, b.second);
    };
    auto add = [](float a, float b) { return a + b; };
#pragma unroll
    for (int g = 0; g < GC; ++g) {
        const float M = over_groups(m[g], [](float a, float b) { return fmaxf(a, b); });
        const float a = E::exp_(m[g] - (M == -INFINITY ? 0.f : M));
        l[g] = over_groups(l[g] * a, add);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = over_groups(acc[g][e] * a, add);
        m[g] = M;
    }

    // merge the wavefronts through LDS
    __shared__ float sm_m[WAVES][GC], sm_l[WAVES][GC];
    __shared__ float sm_acc[WAVES][GC][D];
    if (tg == 0) {
#pragma unroll
        for (int g = 0; g < GC; ++g) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) sm_acc[wave][g][c * EPL + e] = acc[g][e];
        }
        if (c == 0) {
#pragma unroll
            for (int g = 0; g < GC; ++g) {
                sm_m[wave][g] = m[g];
                sm_l[wave][g] = l[g];
            }
        }
    }
    __syncthreads();

    const bool single = ctx <= p.partition_tokens;  // the whole context sat in this partition
    // m, sum and dim d of the accumulator of head g, over all wavefronts
    auto put = [&](int g, int d, float M, float L, float A) __attribute__((always_inline)) {
        const size_t row = size_t(seq) * p.num_q_heads + head0 + g;
        if (single) {
            out[row * D + d] = E::to_out(A / L);
        } else {
            const size_t slot = row * p.max_partitions + part;
            if (MERGE) store_device(ws.acc + slot * D + d, A); else ws.acc[slot * D + d] = A;
            if (d == 0) {
                if (MERGE) {
                    store_device(ws.ml + slot * 2, M);
                    store_device(ws.ml + slot * 2 + 1, L);
                } else {
                    ws.ml[slot * 2] = M;
                    ws.ml[slot * 2 + 1] = L;
                }
            }
        }
    };
    // Weights of the wavefronts: by a lane each, for all 64 dims of a wavefront's share, where the exponential is the long one and a
    // few workgroups' chain is what counts (fp32 of 64, 8 / 8 heads, 4 x 256 tokens 4.6 -> 4.3 us); else every thread its own, which has no
    // chain over the lanes (bf16 of 64, 61 x 91 tokens, 16 / 16 heads, 5.06 with a lane each, 4.88 so; decode up to 512 workgroups 0.97;
    // eight heads 0.98; prefill 0.98).
    if constexpr (sizeof(T) == 4 && GC < 8 && !PREFILL) {
        for (int i = wave; i < GC * (D / 64); i += WAVES) {
            const int g = i / (D / 64), d = i % (D / 64) * 64 + lane;
            const float m_w = lane < WAVES ? sm_m[lane % WAVES][g] : -INFINITY;
            const float M = lanes::wave_max(m_w);
            const float w_w = E::exp_(m_w - (M == -INFINITY ? 0.f : M));  // M = -inf: every score of the partition is
            const float L = lanes::wave_sum(lane < WAVES ? w_w * sm_l[lane % WAVES][g] : 0.f);
            float A = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w)
                A = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_w), w)), sm_acc[w][g][d], A);
            put(g, d, M, L, A);
        }
    } else {
        for (int i = tid; i < GC * D; i += 64 * WAVES) {
            const int g = i / D, d = i % D;
            float M = sm_m[0][g];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) M = fmaxf(M, sm_m[w][g]);
            float L = 0.f, A = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const float wgt = E::exp_(sm_m[w][g] - (M == -INFINITY ? 0.f : M));
                L = fmaf(wgt, sm_l[w][g], L);
                A = fmaf(wgt, sm_acc[w][g][d], A);
            }
            put(g, d, M, L, A);
        }
    }
    if constexpr (MERGE) {
        if (single) return;
        // The workgroup that counts the last partition of its heads merges all of them.  The count may become visible only
        // after the partial: every wavefront waits for its own stores, then all meet.  Nobody waits for anybody.
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        __shared__ int s_last;
        const int nparts = (ctx + p.partition_tokens - 1) / p.partition_tokens;
        int32_t *const counter = ws.cnt + seq * chunks + hc;
        if (tid == 0) s_last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nparts - 1;
        __syncthreads();
        if (!s_last) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");  // the fetches stay behind the count
        if (tid == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        constexpr int DPL = D / 64;
        for (int g = wave; g < GC; g += WAVES) {
            const size_t row = size_t(seq) * p.num_q_heads + head0 + g, slot0 = row * p.max_partitions;
            auto ml_of = [&](int i) {
                float v[2];
                load_device<2>(ws.ml + (slot0 + i) * 2, v);
                return float2{v[0], v[1]};
            };
            float a[DPL];
            const float L = merge_row<DPL, false, 16, true>(
                lane < nparts ? ml_of(lane) : float2{-INFINITY, 0.f}, nparts, lane, ml_of,
                [&](int i, float (&x)[DPL]) { load_device<DPL>(ws.acc + (slot0 + i) * D + lane * DPL, x); }, a);
#pragma unroll
            for (int j = 0; j < DPL; ++j) out[row * D + lane * DPL + j] = E::to_out(a[j] / L);
        }
    }
}

// Whether table entries are requested ahead of their use.  That takes a round trip out of the chain of a workgroup; the registers
// that hold them cost loads in flight or, with four heads in bf16, a wavefront per SIMD.  Both sides, us, at their use / ahead:
//   eight heads: decode, bf16 of 64, 64 / 8 heads, eight of up to 13689 tokens 113.2 / 92.0, fp32 of 128, 8 / 1, eight of up to 2920
//     37.6 / 30.7; prefill, bf16 of 64, 64 / 8, 9 x 1 row of up to 1151 50.6 / 33.1;
//   four: decode, bf16 of 128, 32 / 8, blocks of one, 175 of up to 49 16.5 / 19.0, fp32 of 64, 32 / 8, 42 of up to 1174 26.2 / 31.0;
//     prefill, bf16 of 128, 40 / 2, 9 x 8 rows of up to 695 35.0 / 51.7;
//   two: decode, bf16 99 : 98, fp32 of 128 above two workgroups a compute unit 100 : 105; prefill, bf16 100 : 101;
//   one: fp32 100 : 99; bf16 the same in calls of few workgroups, 34 / 2 heads of 64, blocks of two, 68 of up to 6009 165 / 183.
// Prefill of two or four heads in fp32 goes by the launch: up to two workgroups a compute unit long contexts win (16 / 4 heads of 64, 352
// workgroups at 1671 tokens 100.5 / 81.6, 32 / 16 of 128, 480 at 1835 177 / 142; from about 400 tokens on), short ones and larger launches
// lose (16 / 8 of 128, 448 at 82 8.6 / 9.3, 1376 at 274 37.8 / 44.6).
constexpr bool ahead_of_use(size_t bytes, int heads, bool prefill) {
    return heads == 8 || (bytes == 4 ? heads == 1 : heads == 2 && !prefill);
}

template <typename T, int D, bool PREFILL>
hipError_t launch_for_chunk(int gc, const void *q, const void *k, const void *v, const int32_t *bt,
                            const int32_t *cl, const int32_t *qs, int num_tables, int max_query_len,
                            void *out, Workspace ws, const AttnParams &p, int grid, hipStream_t stream) {
#define KVC_LAUNCH_AS(GC, WAVES, UNROLL, MERGE, AHEAD)                                                                \
    pa_partial_valu_kernel<T, D, GC, PREFILL, WAVES, UNROLL, MERGE, AHEAD><<<dim3(grid), dim3(64 * WAVES), 0, stream>>>( \
        static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v), bt, cl, qs, num_tables,     \
        max_query_len, static_cast<T *>(out), ws, p)
#define KVC_LAUNCH_WAVES(GC, WAVES, UNROLL)                                                                          \
    do {                                                                                                             \
        constexpr bool kAhead = UNROLL == 4 && ahead_of_use(sizeof(T), GC, PREFILL);                                 \
        constexpr bool kEither = PREFILL && sizeof(T) == 4 && (GC == 2 || GC == 4);                                  \
        constexpr bool kMerge = !PREFILL && GC < 8;                                                                  \
        if (kMerge && p.merge_here) KVC_LAUNCH_AS(GC, WAVES, UNROLL, kMerge, kAhead);                                \
        else if (kEither && few_long) KVC_LAUNCH_AS(GC, WAVES, UNROLL, false, kEither || kAhead);                    \
        else KVC_LAUNCH_AS(GC, WAVES, UNROLL, false, kAhead);                                                        \
    } while (0)
    // prefill: up to two workgroups a compute unit, and tables that can hold several trips
    [[maybe_unused]] const bool few_long = grid <= 2 * kNumCUs && int64_t(p.max_blocks_per_seq) * p.block_size >= 512;
    if constexpr (!PREFILL) {
        // A head per workgroup: the fewer trips a partition takes the better, as long as the workgroups of the launch fit the
        // device at once.  Up to one workgroup a compute unit, fp32 takes sixteen wavefronts, with twice the tokens in a trip
        // where four do not cover the partition (rows of 512 bytes: 5 x 1000 tokens, 16 / 4 heads, 15.0 -> 13.8 us, 4 x 256, 8 / 8,
        // 6.0 -> 5.8).  Up to two, and bf16 throughout, eight, where four would make two trips (fp32 of 128, 16 / 4
        // heads, 24 x 200 12.0 -> 11.4; bf16 of 64, 14 / 2 heads, 4 x 1500 7.6 -> 7.4; one trip, fp32 of 64, 12 / 12
        // heads, 24 x 100 4.22 with four, 4.29 with eight).
        if (gc == 1 && grid <= 2 * kNumCUs) {
            constexpr int kTrip = 4 * (64 / (D * int(sizeof(T)) / 16));  // tokens of a wavefront
            if constexpr (sizeof(T) == 4) {
                if (grid <= kNumCUs) {
                    if (p.partition_tokens > 16 * kTrip) KVC_LAUNCH_WAVES(1, 16, 8); else KVC_LAUNCH_WAVES(1, 16, 4);
                    return hipGetLastError();
                }
            }
            if (p.partition_tokens >= 2 * kWaves * kTrip) KVC_LAUNCH_WAVES(1, 8, 4); else KVC_LAUNCH_WAVES(1, kWaves, 4);
            return hipGetLastError();
        }
    }
    // Several heads, up to one workgroup per compute unit: sixteen wavefronts instead of four where the registers allow it and
    // the merge in LDS is small (fp32, 24 x 256 tokens, four heads of 64 per workgroup 9.3 us with four, 9.7 with sixteen, so
    // those stay at four).
    constexpr bool kWide = !PREFILL && sizeof(T) == 4;
#define KVC_LAUNCH_VALU(GC)                                                                       \
    do {                                                                                          \
        constexpr int kMany = kWide && D == 128 && GC < 8 ? 16 : kWaves;                          \
        if (grid <= kNumCUs) KVC_LAUNCH_WAVES(GC, kMany, 4); else KVC_LAUNCH_WAVES(GC, kWaves, 4); \
    } while (0)
    switch (gc) {
        case 8: KVC_LAUNCH_VALU(8); break;
        case 4: KVC_LAUNCH_VALU(4); break;
        case 2: KVC_LAUNCH_VALU(2); break;
        default: KVC_LAUNCH_WAVES(1, kWaves, 4); break;  // prefill, and more than two workgroups a compute unit
    }
#undef KVC_LAUNCH_VALU
#undef KVC_LAUNCH_AS
#undef KVC_LAUNCH_WAVES
    return hipGetLastError();
}

template <bool PREFILL>
hipError_t launch_for_type(const void *q, const void *k_cache, const void *v_cache,
                           const int32_t *block_tables, const int32_t *context_lens,
                           const int32_t *q_start, int num_tables, int max_query_len, void *out,
                           Workspace ws, const AttnParams &p, int dtype, int head_dim, int grid,
                           hipStream_t stream) {
    const int gc = p.head_chunk;
    if (dtype == KVC_F32) {
        if (head_dim == 64)
            return launch_for_chunk<float, 64, PREFILL>(gc, q, k_cache, v_cache, block_tables, context_lens, q_start,
                                                        num_tables, max_query_len, out, ws, p, grid, stream);
        return launch_for_chunk<float, 128, PREFILL>(gc, q, k_cache, v_cache, block_tables, context_lens, q_start,
                                                     num_tables, max_query_len, out, ws, p, grid, stream);
    }
    if (head_dim == 64)
        return launch_for_chunk<uint16_t, 64, PREFILL>(gc, q, k_cache, v_cache, block_tables, context_lens, q_start,
                                                       num_tables, max_query_len, out, ws, p, grid, stream);
    return launch_for_chunk<uint16_t, 128, PREFILL>(gc, q, k_cache, v_cache, block_tables, context_lens, q_start,
                                                    num_tables, max_query_len, out, ws, p, grid, stream);
}

}  // namespace

hipError_t launch_partial_valu(const void *q, const void *k_cache, const void *v_cache,
                               const int32_t *block_tables, const int32_t *context_lens, void *out,
                               Workspace ws, const AttnParams &p, int dtype, int head_dim,
                               int grid, hipStream_t stream) {
    return launch_for_type<false>(q, k_cache, v_cache, block_tables, context_lens, nullptr, 0, 0, out, ws, p,
                                  dtype, head_dim, grid, stream);
}

// p.num_seqs = rows of q, p.partition_tokens covers any context (one partition, no workspace).
hipError_t launch_prefill_valu(const void *q, const void *k_cache, const void *v_cache,
                               const int32_t *block_tables, const int32_t *context_lens,
                               const int32_t *q_start, int num_tables, int max_query_len, void *out,
                               const AttnParams &p, int dtype, int head_dim, int grid,
                               hipStream_t stream) {
    return launch_for_type<true>(q, k_cache, v_cache, block_tables, context_lens, q_start, num_tables,
                                 max_query_len, out, Workspace{nullptr, nullptr, nullptr}, p, dtype, head_dim,
                                 grid, stream);
}

}  // namespace kvc

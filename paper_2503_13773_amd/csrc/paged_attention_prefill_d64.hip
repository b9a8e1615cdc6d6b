// Causal attention of many query positions per sequence over the block-allocated KV cache for
// head_dim 64 (gfx950, bf16) on 32x32x16 matrix-core tiles, with softmax weights kept to 16 bits.
//
// Bound: the vector issue port, in long launches at the power limit (6000 tokens run at 1.92 GHz).  Per 32 tokens x 32
// score columns a wavefront needs 12 matrix instructions (4 for K.Q, 8 for V.P), about 80 plain vector instructions and 16
// exponentials; they take 4 cycles of the port each, an exponential and a matrix instruction 8 (in a mix of them other
// wavefronts of the SIMD don't issue beside: one to four waves, 12 + 96 + 16 of them, 595 to 617 cycles a wave), 550 cycles
// for 384 of the matrix pipe.
// The weights stay in fp32 up to the product with V, where a weight goes into the matrix core as the sum
// of two bf16 values (its upper bits and the rounded rest, 2^-16 relative), the normaliser
// sums the fp32 weights.  Output errors against 64 bits are those of the rounding to bf16.
//
// A turn of a step that every column sees whole computes the scores of the next step beside the weights of this one.  32 / 8
// heads, us, steps one after the other with a scalar load of a block id in each / now: 100 tokens 6.2 / 5.9, 400 10.0 / 9.3,
// 1000 17.5 / 16.4, 1999 35.7 / 32.8 = 500 TFLOP/s, 6000 232 / 222; 12 / 12 heads, 1999 30.1 / 28.0.  Registers decide what
// fits: products with V left over to the next turn, to fill its start, spill a Q operand, whose reload drains the loads in
// flight (1999 tokens 36.5 us); and a kernel that uses scratch memory anywhere starts 0.3 us later (100 tokens 6.1 us with
// 24 bytes of it), so that the masked steps take V by slices and scores are not carried into them.
//
// One workgroup = (sequence, 2 query heads of one KV head, 64 query rows), or one head and 128 rows
// for odd group sizes; 8 wavefronts.  It walks the context in steps of 64 tokens.  Wavefronts 2w and
// 2w + 1 own the same 32 score columns (16 query rows x 2 heads, or 32 rows of one head) and take
// 32 tokens of a step each, so the longest chain of a workgroup is half as long as with one
// wavefront per column set and the causal triangle's last workgroups end sooner; their
// partial results meet in LDS at the end (log-sum-exp rule).  Two workgroups fit a compute unit: four
// wavefronts per SIMD hide each other's matrix and LDS latencies (with two and twice the registers 48 us).
//
// K and V rows (128 bytes) travel straight into LDS (global_load_lds_dwordx4: lane l writes 16
// bytes at M0 + 16 l), one 1 KiB load of K and one of V per wavefront and step, three steps
// ahead, four stages (64 KiB).  Which 16 bytes a lane fetches is chosen so that the LDS image is
//   K rows: chunk ch of row R at chunk position ch ^ (R / 2 % 8): 16 rows x the same dims touch every bank once;
//   V rows: 64-byte granule b of row R at position (b + R / 2) % 2: the 4 rows x 64 bytes of a transposing
//           read fall into disjoint banks.
//
// Operand layouts (lane = 32 * half + c): see the comments at the reads below; every score of a lane
// belongs to one column, so max, weights and sum are lane-local and the halves of a column meet only
// when the reference point moves and at the end.
#include <float.h>
#include <math.h>

#include <type_traits>

#include "kvc_internal.h"
#include "pa_mfma_tile.h"

namespace kvc {

namespace {

using mfma::bf16x8;
using mfma::pack_bf16;

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kDim = 64;
constexpr int kRowBytes = kDim * 2;
constexpr int kStep = 64;                         // tokens of a step: 32 for each of the two wavefronts of a column set
constexpr int kStageBytes = kStep * kRowBytes;    // K (or V) rows of a step
constexpr int kStages = 4;
constexpr int kBlockThreads = kPrefill64Threads;
constexpr float kLazyLog2 = 8.0f;
constexpr float kHugeScore = 1048576.f;  // 2^20: up to here the rounding of m is at most 2^-5

template <int I, int N, class F>
__device__ inline void static_for(const F &f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}
// Nothing moves across this point when the compiler orders the instructions of a turn.
#define KVC_PIN() __builtin_amdgcn_sched_barrier(0)

using lanes::max_over_halves;
using lanes::sum_over_halves;
__device__ inline float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// 16 bytes per lane from global memory to LDS at lds_addr + 16 * lane (lds_addr uniform).  Not seen by the
// compiler: the kernel orders it with barriers and waits for it with wait_loads_but().
__device__ inline void load_lane_to_lds(const void *addr, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_addr), "v"(addr) : "memory");
}
// The same from base + off, base uniform.
__device__ inline void load_row_to_lds(const void *base, uint32_t off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds_addr), "v"(off), "s"(base) : "memory");
}
template <int N>
__device__ inline void wait_loads_but() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
// A wavefront waits for its own LDS reads before the barrier: what they come from may be overwritten after it.
__device__ inline void step_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A operand of O^T += V^T . P^T: slice n (16 tokens) of dim block b, by two transposing reads (the lane of
// dim 32b + c receives that dim of tokens 16n + 8g + 4*half .. +3, the order in which the weights lie).
__device__ inline int v_lane_offset(int b, int half, int c) {
    const int i16 = c & 15, k = i16 >> 2;
    return (4 * half + k) * kRowBytes + ((b + (k >> 1)) & 1) * 64 + 32 * (c >> 4) + 8 * (i16 & 3);
}
__device__ inline uint4 read_v_operand(const unsigned char *vlane, int n) {
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef v4i16 __attribute__((address_space(3))) * lds_v4i16_ptr;
    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(vlane + (16 * n) * kRowBytes)));
    const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(vlane + (16 * n + 8) * kRowBytes)));
    return uint4{lo.x, lo.y, hi.x, hi.y};
}
// tokens at or past `vlim` of the wavefront's 32 are invisible to all its columns; their V may hold anything
__device__ inline uint32_t keep_below(uint32_t w, int tok, int vlim) {
    return w & ((tok < vlim ? 0xffffu : 0u) | (tok + 1 < vlim ? 0xffff0000u : 0u));
}
__device__ inline bool has_non_finite(uint32_t w) {
    return (w & 0x7f80u) == 0x7f80u || (w & 0x7f800000u) == 0x7f800000u;
}
__device__ inline uint32_t finite_only(uint32_t w) {
    return ((w & 0x7f80u) == 0x7f80u ? 0u : w & 0xffffu) | ((w & 0x7f800000u) == 0x7f800000u ? 0u : w & 0xffff0000u);
}

// a * b rounded, also where a subtraction follows: the compiler makes one fused operation of __fmul_rn(a, b) - c.
__device__ inline float rounded_product(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}

__device__ inline float top_of(const floatx16 &x) {
    const float a = max3(max3(x[0], x[1], x[2]), max3(x[3], x[4], x[5]), max3(x[6], x[7], x[8]));
    return fmaxf(a, max3(max3(x[9], x[10], x[11]), max3(x[12], x[13], x[14]), x[15]));
}
// The weights of a pair of tokens as two packed words.  The upper part is cut off, the rest is made positive by 2^-23 of the
// weight (a factor all weights share): an infinity in V keeps its sign, which a rest of 0 or of the other sign would turn
// into NaN.
__device__ inline uint32_t upper_parts(float w0, float w1) {
    return __builtin_amdgcn_perm(__float_as_uint(w1), __float_as_uint(w0), 0x07060302u);
}
__device__ inline float rest_of(float w) {
    return __builtin_fmaf(w, 1.f + FLT_EPSILON, -__uint_as_float(__float_as_uint(w) & 0xffff0000u));
}

// One product, in the order it is written in.
__device__ inline void multiply(floatx16 &acc, const uint4 &a, uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, uint4{b0, b1, b2, b3}), acc, 0, 0, 0);
}

// One turn of a wavefront that sees all tokens of its step and the next, with the raw scores of step s in x:
//     chunks  0 ..  3   S of step s + 1
//     chunks  6 ..  9   O += V . weights of tokens 0 .. 15 of step s, upper parts, then rests
//     chunks 10 .. 13   of tokens 16 .. 31
// and the softmax arithmetic of step s spread over chunks 0 .. 10: that of pair i starts in chunk i, and its arguments, exponentials,
// upper parts and sum, rests take a chunk each.
__device__ inline void pipeline_turn(floatx16 (&acc)[2], floatx16 &x, float &lsum, float &m, uint64_t &huge, const bf16x8 (&qb)[4],
                                     const unsigned char *k_next, const int (&koff)[2], const unsigned char *const (&v_cur)[2], float scale) {
    bf16x8 ka[4];
    uint4 va[2][2];  // [slice of 16 tokens][dim block]
    auto read_k = [&](int j) __attribute__((always_inline)) {
        int at = koff[j >> 1];
        if (j & 1) asm volatile("v_xor_b32 %0, 32, %1" : "=v"(at) : "v"(koff[j >> 1]));  // kept out of the registers of the loop
        ka[j] = *reinterpret_cast<const bf16x8 *>(k_next + at);
    };
    read_k(0);
    read_k(1);
    read_k(2);
    const float top = scale * top_of(x);
    const uint64_t moved = __builtin_amdgcn_ballot_w64(top > m + kLazyLog2);
    float factor = scale;
    if (__builtin_expect((moved | huge) != 0, 0)) {
        if (moved != 0) {
            const float m_new = fmaxf(m, max_over_halves(top));
            const float alpha = __builtin_amdgcn_exp2f(m - m_new);
            m = m_new;
            lsum *= alpha;
            acc[0] *= alpha;
            acc[1] *= alpha;
            huge = __builtin_amdgcn_ballot_w64(fabsf(m) > kHugeScore);
        }
        if (huge != 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = rounded_product(x[v], scale);
            factor = 1.f;
        }
    }
    floatx16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
    uint32_t hi[8], lo[8];
    float rest[16], sum;
    static_for<0, 14>([&](auto chunk) __attribute__((always_inline)) {
        constexpr int T = decltype(chunk)::value;
        KVC_PIN();
        if constexpr (T < 4) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[T], qb[T], s, 0, 0, 0);
        if constexpr (T >= 6) {
            constexpr int N = (T - 6) >> 2, B = T & 1, F = 4 * N;
            if constexpr (((T - 6) & 2) == 0) multiply(acc[B], va[N][B], hi[F], hi[F + 1], hi[F + 2], hi[F + 3]);
            else multiply(acc[B], va[N][B], lo[F], lo[F + 1], lo[F + 2], lo[F + 3]);
        }
        if constexpr (T == 0) read_k(3);
        if constexpr (T == 2 || T == 3) va[0][T - 2] = read_v_operand(v_cur[T - 2], 0);
        if constexpr (T == 6 || T == 7) va[1][T - 6] = read_v_operand(v_cur[T - 6], 1);
        static_for<0, 8>([&](auto pair) __attribute__((always_inline)) {
            constexpr int I = decltype(pair)::value, A = 2 * I, B = A + 1;
            if constexpr (I == T) {
                x[A] = __builtin_fmaf(x[A], factor, -m);
                x[B] = __builtin_fmaf(x[B], factor, -m);
            }
            if constexpr (I + 1 == T) {
                x[A] = __builtin_amdgcn_exp2f(x[A]);
                x[B] = __builtin_amdgcn_exp2f(x[B]);
            }
            if constexpr (I + 2 == T) {
                hi[I] = upper_parts(x[A], x[B]);
                const float both = x[A] + x[B];
                sum = I == 0 ? both : sum + both;
                asm volatile("" : "+v"(hi[I]), "+v"(sum));
                rest[A] = rest_of(x[A]);
            }
            if constexpr (I + 3 == T) {
                rest[B] = rest_of(x[B]);
                lo[I] = pack_bf16(rest[A], rest[B]);
                asm volatile("" : "+v"(lo[I]));
            }
        });
    });
    KVC_PIN();
    lsum += sum;  // once a step, as a step by itself does: weights far below the sum so far add up before they meet it
    x = s;
}

// HEADS = 2: columns are 16 query rows x 2 heads of one KV head; HEADS = 1: 32 query rows of one head.
// SMALL: block_size < 8, the 8 rows a wavefront loads per instruction may lie in several blocks.
template <bool SMALL, int HEADS>
__global__ __launch_bounds__(kBlockThreads, 4) void pa_prefill_d64_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k_cache,
    const uint16_t *__restrict__ v_cache, const int32_t *__restrict__ block_tables,
    const int32_t *__restrict__ context_lens, const int32_t *__restrict__ q_start,
    uint16_t *__restrict__ out, PrefillParams p, int max_query_len, int query_tiles, int fold_at, int spread) {
    __shared__ __attribute__((aligned(1024))) unsigned char s_kv[2 * kStages * kStageBytes];
    unsigned char *const s_k = s_kv, *const s_v = s_kv + kStages * kStageBytes;
    constexpr int kWaveRows = 32 / HEADS;
    constexpr int kTileRows = 4 * kWaveRows;

    // What the start reads is loaded at once: where a part of it is put off to its first use, a workgroup waits for the scalar
    // cache twice (32 / 8 heads, 18 rows, 4.82 us, so 4.55).
    asm volatile("" :: "s"(context_lens), "s"(q_start), "s"(block_tables), "s"(p.num_seqs), "s"(p.num_q_heads), "s"(p.group), "s"(p.max_blocks_per_seq),
                 "s"(max_query_len), "s"(query_tiles), "s"(fold_at), "s"(spread));

    // blockIdx.x = head chunk + chunks * (seq + num_seqs * order), the longest query tiles first; from
    // `fold_at` on the shortest first (grids that are resident at once: a long and a short one share a compute unit)
    const int chunks = p.num_q_heads / HEADS;
    const int item = blockIdx.x;
    const int chunk = chunk_at(item % chunks, spread);
    const int n = (item / chunks) % p.num_seqs;
    const int order = item / (chunks * p.num_seqs);
    const int qtile = order < fold_at ? query_tiles - 1 - order : order - fold_at;
    const int head0 = chunk * HEADS;
    const int kvh = head0 / p.group;

    const int S = context_lens[n];
    const int qs = q_start[n];
    const int Qn = q_start[n + 1] - qs;
    const int rows = min(Qn, max_query_len);  // rows past the caller's bound are not computed
    if (qtile * kTileRows >= rows || Qn > S) return;  // uniform over the workgroup

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int part = wave & 1, set = wave >> 1;  // half of each step's tokens, column set (few rows: on different SIMDs)
    const int half = lane >> 5, c = lane & 31;
    const int r = c % kWaveRows;
    const int my_head = head0 + c / kWaveRows;

    const int last_pos = S - Qn + min(rows, qtile * kTileRows + kTileRows) - 1;
    const int steps = last_pos / kStep + 1;
    const int32_t *table = block_tables + size_t(n) * p.max_blocks_per_seq;

    const int i0 = qtile * kTileRows + kWaveRows * set;  // first query row of this wavefront
    const bool active = i0 < rows;                       // others still load and synchronise
    const int nrows = active ? min(kWaveRows, rows - i0) : 1;
    const int row = min(r, nrows - 1);                   // lanes past the last query row shadow it
    const int p0 = S - Qn + (active ? i0 : 0);
    const int my_pos = p0 + row;
    const int wave_vis = active ? p0 + nrows : 0;        // tokens visible to some column

    // Where the rows of a step lie in a pool, counted in rows (a pool of 2^32 rows would be 512 GiB); past the last visible
    // token its block is repeated (loaded, never used).  The 8 rows of a wavefront are inside one block of 8 tokens and
    // more: lane l holds the place of those of step `window` + l, so that a turn takes a lane read instead of a
    // scalar load, whose wait the LDS reads would share.  SMALL: a load per lane and step.
    const int bs_mask = p.block_size - 1, lrow = lane >> 3;  // the row of the wavefront's 8 that this lane loads from
    const uint32_t block_rows = uint32_t(p.block_size) * p.num_kv_heads;
    auto row_at = [&](int tok) __attribute__((always_inline)) {
        return uint32_t(table[tok >> p.block_size_log2]) * block_rows + (tok & bs_mask);
    };
    auto rows_of_window = [&](int window) __attribute__((always_inline)) {
        return SMALL ? 0 : row_at(min((window + lane) * kStep + 8 * wave, last_pos & ~7));
    };
    int window = 0;
    uint32_t lane_row = rows_of_window(0);  // requested before Q: its wait does not include that

    // Q as the B operand: lane (half, c) holds dims 16j + 8*half .. +7 of column c's row.  The sign of the
    // scale goes into Q (exact), a scale of zero becomes Q = 0.
    bf16x8 qb[4];
    {
        const uint16_t *qrow = q + (size_t(qs + (active ? i0 : 0) + row) * p.num_q_heads + my_head) * kDim + 8 * half;
        const uint32_t flip = p.scale_log2e < 0.f ? 0x80008000u : 0u, keep = p.scale_log2e == 0.f ? 0u : ~0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint4 w = *reinterpret_cast<const uint4 *>(qrow + 16 * j);
            w = uint4{(w.x ^ flip) & keep, (w.y ^ flip) & keep, (w.z ^ flip) & keep, (w.w ^ flip) & keep};
            qb[j] = __builtin_bit_cast(bf16x8, w);
        }
    }
    const float scale = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(p.scale_log2e == 0.f ? 1.f : fabsf(p.scale_log2e))));

    // ---- loads: wavefront w brings rows 8w .. 8w+7 of a step, lane l chunk position l % 8 of row 8w + l / 8
    const size_t head_bytes = size_t(p.block_size) * kRowBytes;
    const unsigned char *k_head = reinterpret_cast<const unsigned char *>(k_cache) + size_t(kvh) * head_bytes;
    const unsigned char *v_head = reinterpret_cast<const unsigned char *>(v_cache) + size_t(kvh) * head_bytes;
    const int lpos = lane & 7;                            // 8 * wave is a multiple of 8: row / 2 % 8 = 4 * (wave % 2) + lrow / 2
    const int k_chunk = (lpos ^ ((4 * wave + (lrow >> 1)) & 7)) * 16;
    const int v_chunk = (4 * (((lpos >> 2) + (lrow >> 1)) & 1) + (lpos & 3)) * 16;
    const uint32_t lds_k = uint32_t(reinterpret_cast<uintptr_t>(s_k)) + 1024 * wave;
    const uint32_t lds_v = uint32_t(reinterpret_cast<uintptr_t>(s_v)) + 1024 * wave;
    auto lookup = [&](int step) __attribute__((always_inline)) -> uint32_t {
        if constexpr (SMALL) return row_at(min(step * kStep + 8 * wave + lrow, last_pos));
        if (__builtin_expect(step - window == 64, 0)) {
            window = step;
            lane_row = rows_of_window(window);
        }
        return __builtin_amdgcn_readlane(lane_row, step - window);
    };
    auto issue = [&](int step, uint32_t at) __attribute__((always_inline)) {
        const uint32_t stage = (step & (kStages - 1)) * kStageBytes;
        const uint32_t to_k = __builtin_amdgcn_readfirstlane(lds_k + stage), to_v = __builtin_amdgcn_readfirstlane(lds_v + stage);
        const size_t off = size_t(at) * kRowBytes;
        if constexpr (SMALL) {
            load_lane_to_lds(k_head + off + k_chunk, to_k);
            load_lane_to_lds(v_head + off + v_chunk, to_v);
        } else {
            load_row_to_lds(k_head + off, lrow * kRowBytes + k_chunk, to_k);
            load_row_to_lds(v_head + off, lrow * kRowBytes + v_chunk, to_v);
        }
    };

    uint32_t at_next;  // three steps ahead
    {
        const uint32_t a0 = lookup(0), a1 = lookup(1), a2 = lookup(2);
        at_next = lookup(3);
        issue(0, a0);
        issue(1, a1);
        issue(2, a2);
    }
    // a use of Q on this side of the loop: its loads are waited for once, not in front of the first product
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(qb[j]));

    floatx16 acc[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
    // Reference point of the weights (base-2 units), within 2^kLazyLog2 of the running max.  It starts at the
    // lowest finite value: scores of -inf then weigh 0 and never meet another infinity.
    float m = -FLT_MAX, lsum = 0.f;
    uint64_t huge = ~uint64_t(0);  // columns whose |m| is above kHugeScore

    // K as the A operand: lane (half, c) holds dims 16j + 8*half .. +7 of token c; this is where those of j = 0 and 2 are in a
    // stage, those of j + 1 are at that ^ 32
    int koff[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) koff[j] = (32 * part + c) * kRowBytes + (((4 * j + half) ^ ((c >> 1) & 7)) << 4);
    const unsigned char *v_lane[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) v_lane[b] = s_v + 32 * part * kRowBytes + v_lane_offset(b, half, c);

    auto scores = [&](int st) __attribute__((always_inline)) {
        floatx16 s;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(s_k + st * kStageBytes + (koff[j >> 1] ^ (j & 1) << 5)), qb[j], s, 0, 0, 0);
        return s;
    };
    // a step by itself, such as those that the causal mask touches: 32 tokens from token t0 on, stage `st`
    auto single_step = [&](auto masked, int st, int t0) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked)::value;
        // tokens of the step that the column (any column) sees, counted from 4 * half; opaque to the compiler,
        // which would otherwise keep sixteen comparisons of them in registers across the whole loop
        int limit = my_pos + 1 - t0 - 4 * half, vlim = wave_vis - t0 - 4 * half;
        if (MASKED) asm volatile("" : "+v"(limit), "+v"(vlim));
        const floatx16 s = scores(st);
        uint4 early[2][2];  // a step that every column sees whole reads V ahead of the softmax; the other checks it
        if constexpr (!MASKED)
#pragma unroll
            for (int nn = 0; nn < 2; ++nn)
#pragma unroll
                for (int b = 0; b < 2; ++b) early[nn][b] = read_v_operand(v_lane[b] + st * kStageBytes, nn);
        // raw scores of column c: token 8*(v/4) + 4*half + v%4 in x[v]
        floatx16 x;
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v] = MASKED && 8 * (v >> 2) + (v & 3) >= limit ? -INFINITY : s[v];
        const float top = scale * top_of(x);
        // the reference point only moves when some score exceeds it by more than 2^kLazyLog2
        if (__builtin_amdgcn_ballot_w64(top > m + kLazyLog2) != 0) {
            const float m_new = fmaxf(m, max_over_halves(top));
            const float alpha = __builtin_amdgcn_exp2f(m - m_new);
            m = m_new;
            lsum *= alpha;
            acc[0] *= alpha;
            acc[1] *= alpha;
            huge = __builtin_amdgcn_ballot_w64(fabsf(m) > kHugeScore);
        }
        // One fused multiply-add per exponent: the product is exact, m is the rounded product of the largest
        // score, so all weights of a column share the factor 2^(rounding of m), which cancels.  Where m is
        // so large that the factor itself would overflow the product is rounded first.
        if (huge != 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = rounded_product(x[v], scale) - m;
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = __builtin_fmaf(x[v], scale, -m);
        }
        float sum = 0.f;
        uint32_t hi[8], lo[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            x[2 * i] = __builtin_amdgcn_exp2f(x[2 * i]);
            x[2 * i + 1] = __builtin_amdgcn_exp2f(x[2 * i + 1]);
            sum += x[2 * i] + x[2 * i + 1];
            hi[i] = upper_parts(x[2 * i], x[2 * i + 1]);
            lo[i] = pack_bf16(rest_of(x[2 * i]), rest_of(x[2 * i + 1]));
        }
        lsum += sum;
#pragma unroll
        for (int nn = 0; nn < 2; ++nn) {  // tokens 16 nn .. 16 nn + 15
            uint4 va[2];
            bool odd = false;  // a V value that is not finite, in a step that not every column sees whole
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                if constexpr (!MASKED) {
                    va[b] = early[nn][b];
                    continue;
                }
                const uint4 w = read_v_operand(v_lane[b] + st * kStageBytes, nn);
                const int tok = 16 * nn;
                va[b] = uint4{keep_below(w.x, tok, vlim), keep_below(w.y, tok + 2, vlim),
                              keep_below(w.z, tok + 8, vlim), keep_below(w.w, tok + 10, vlim)};
                odd |= has_non_finite(va[b].x) | has_non_finite(va[b].y) | has_non_finite(va[b].z) | has_non_finite(va[b].w);
            }
            if (MASKED && __builtin_expect(__builtin_amdgcn_ballot_w64(odd) != 0, 0)) {
                // such a value times the weight 0 of a column that may not see its token would be NaN:
                // the matrix core gets the finite values, the others are added column by column
                for (int t = 16 * nn; t < min(wave_vis - t0, 16 * nn + 16); ++t) {
                    uint32_t upper = 0, rest = 0;  // of the weights of the pair that t is in
#pragma unroll
                    for (int i = 4 * nn; i < 4 * nn + 4; ++i) {
                        const bool here = 2 * (t >> 3) + ((t & 3) >> 1) == i;
                        upper = here ? hi[i] : upper;
                        rest = here ? lo[i] : rest;
                    }
                    const int shift = (t & 1) ? 0 : 16;
                    const float mine = __uint_as_float(upper << shift & 0xffff0000u) + __uint_as_float(rest << shift & 0xffff0000u);
                    const float wt = __shfl(mine, 32 * ((t >> 2) & 1) + c);
                    const int trow = 32 * part + t;
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int dim = 8 * (v >> 2) + 4 * half + (v & 3);  // inside block b
                            const uint16_t u = *reinterpret_cast<const uint16_t *>(
                                s_v + st * kStageBytes + trow * kRowBytes + ((b + (trow >> 1)) & 1) * 64 + 2 * dim);
                            if ((u & 0x7f80u) == 0x7f80u && t - 4 * half < limit)
                                acc[b][v] = fmaf(wt, __uint_as_float(uint32_t(u) << 16), acc[b][v]);
                        }
                }
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    va[b] = uint4{finite_only(va[b].x), finite_only(va[b].y), finite_only(va[b].z), finite_only(va[b].w)};
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) multiply(acc[b], va[b], hi[4 * nn], hi[4 * nn + 1], hi[4 * nn + 2], hi[4 * nn + 3]);
#pragma unroll
            for (int b = 0; b < 2; ++b) multiply(acc[b], va[b], lo[4 * nn], lo[4 * nn + 1], lo[4 * nn + 2], lo[4 * nn + 3]);
        }
    };

    // Step s reads K rows of steps s and s + 1 and V rows of step s.  They have arrived once every wavefront has waited for its
    // own loads of them (the newest three may be outstanding) and met the others.  It requests the rows of step s + 3, over
    // those of step s - 1, which were last read before that barrier.
    int s = 0;
    auto next_stage = [&](int ph) __attribute__((always_inline)) {  // ph = s % 4
        wait_loads_but<SMALL ? 4 : 3>();  // steps by themselves read K rows of step s only
        step_barrier();
        issue(ph + 3, at_next);
        at_next = lookup(s + 4);
    };
    // steps whose 32 tokens every column sees, then the one or two that the causal mask touches, then those past
    // the wavefront's last position, in which it only loads and synchronises
    const int plain = active ? min(steps, (p0 + 1 + 32 - 32 * part) / kStep) : 0;
    const int live = min(steps, (wave_vis + kStep - 1 - 32 * part) / kStep);
    if constexpr (SMALL) {  // the addresses of a turn's loads leave no registers for two steps at once
        for (; s < plain; ++s) {
            next_stage(s & 3);
            single_step(std::false_type{}, s & 3, s * kStep + 32 * part);
        }
    } else if (plain > 0) {
        floatx16 x;
        // PH = s % 4, a literal in the unrolled loop: the LDS addresses of a turn are then per-lane registers plus immediates
#define KVC_TURN(PH)                                                                                           \
    {                                                                                                          \
        const int ph = (PH);                                                                                   \
        const unsigned char *const v_cur[2] = {v_lane[0] + ph * kStageBytes, v_lane[1] + ph * kStageBytes};    \
        pipeline_turn(acc, x, lsum, m, huge, qb, s_k + ((ph + 1) & 3) * kStageBytes, koff, v_cur, scale);      \
        ++s;                                                                                                   \
    }
        next_stage(0);
        x = scores(0);
        while (s + 4 < plain) {
            KVC_TURN(0)
            next_stage(1);
            KVC_TURN(1)
            next_stage(2);
            KVC_TURN(2)
            next_stage(3);
            KVC_TURN(3)
            next_stage(0);
        }
        while (true) {
            KVC_TURN(s & 3)
            if (s == plain) break;
            next_stage(s & 3);
        }
#undef KVC_TURN
    }
    for (; s < live; ++s) {
        next_stage(s & 3);
        single_step(std::true_type{}, s & 3, s * kStep + 32 * part);
    }
    for (; s < steps; ++s) next_stage(s & 3);

    // ---- the two parts of a column set meet: each wavefront hands over one dim block and finishes the other
    lsum = sum_over_halves(lsum);
    wait_loads_but<0>();  // nothing may still be landing in LDS
    step_barrier();
    float *const hand = reinterpret_cast<float *>(s_kv) + set * (2 * 18 * 64) + lane;  // [set][part][16 + 2][64]
    {
        float *mine = hand + part * (18 * 64);
#pragma unroll
        for (int v = 0; v < 16; ++v) mine[v * 64] = part == 0 ? acc[1][v] : acc[0][v];
        mine[16 * 64] = m;
        mine[17 * 64] = lsum;
    }
    step_barrier();
    const float *theirs = hand + (1 - part) * (18 * 64);
    const float m_o = theirs[16 * 64], l_o = theirs[17 * 64];
    const float M = fmaxf(m, m_o);
    const float w_m = __builtin_amdgcn_exp2f(m - M), w_o = __builtin_amdgcn_exp2f(m_o - M);
    const float inv = 1.0f / (w_m * lsum + w_o * l_o);
    if (active && r < nrows) {
        uint16_t *dst = out + (size_t(qs + i0 + r) * p.num_q_heads + my_head) * kDim + 32 * part + 4 * half;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            float o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int v = 4 * a + i;
                o[i] = (w_m * (part == 0 ? acc[0][v] : acc[1][v]) + w_o * theirs[v * 64]) * inv;
            }
            const uint2 w = {pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3])};
            *reinterpret_cast<uint2 *>(dst + 8 * a) = w;
        }
    }
}

}  // namespace

hipError_t launch_prefill_d64(const void *q, const void *k_cache, const void *v_cache,
                              const int32_t *block_tables, const int32_t *context_lens,
                              const int32_t *q_start, void *out, const PrefillParams &p, int max_query_len,
                              hipStream_t stream) {
    const int heads = p.heads_per_chunk;
    const int tile_rows = 128 / heads;
    const int query_tiles = (max_query_len + tile_rows - 1) / tile_rows;
    const int64_t grid = int64_t(p.num_q_heads / heads) * p.num_seqs * query_tiles;
    const int fold_at = grid <= 2 * kNumCUs ? (query_tiles + 1) / 2 : query_tiles;  // two workgroups per compute unit
    const bool small = p.block_size < 8;
    const int spread = chunk_spread(p.num_q_heads / heads, p.group / heads);
#define KVC_LAUNCH(SMALL, HEADS)                                                                     \
    pa_prefill_d64_kernel<SMALL, HEADS><<<dim3(unsigned(grid)), dim3(kBlockThreads), 0, stream>>>(   \
        static_cast<const uint16_t *>(q), static_cast<const uint16_t *>(k_cache),                    \
        static_cast<const uint16_t *>(v_cache), block_tables, context_lens, q_start,                 \
        static_cast<uint16_t *>(out), p, max_query_len, query_tiles, fold_at, spread)
    if (small && heads == 2) KVC_LAUNCH(true, 2);
    else if (small) KVC_LAUNCH(true, 1);
    else if (heads == 2) KVC_LAUNCH(false, 2);
    else KVC_LAUNCH(false, 1);
#undef KVC_LAUNCH
    return hipGetLastError();
}

}  // namespace kvc

// Causal attention of many query positions over the block-allocated KV cache, long requests (gfx950, bf16, head_dim
// 128, positive scale, groups of 4, 8, 12 or 16): wavefronts of 64 score columns on 32x32x16 matrix-core tiles.
//
// What bounds it.  Wavefronts of 32 columns, two per SIMD (paged_attention_prefill32.hip), read 16 KiB of K and V
// operands from LDS per 32 x 32 scores: 128 KiB per step of a compute unit, 1024 cycles of LDS bandwidth against 1024
// matrix cycles; a step takes about 1450 cycles.  Here a wavefront owns two groups of 32 columns that share every
// operand read, which halves the LDS reads, the address arithmetic and the scalar work per score.  128 accumulator and
// 64 Q registers (AGPRs, which only matrix instructions touch) leave room for one wavefront per SIMD, so everything
// that hides latency is in the order of the instructions: a step of 64 columns takes 1390 cycles for 1024 matrix cycles.
// The issue of one wavefront is what is left: about 220 instructions per step of 4 to 5 cycles each, 8 for an
// exponential (without loads, LDS reads and barriers a step still takes 1160 cycles).  Long launches run at the power
// limit (1.75 to 1.9 of 2.4 GHz), where the LDS reads saved count as well.  32 / 8 heads, one request, kernel of 32
// columns / this one, us: 3500 tokens 98.9 / 93.6, 4096 126.1 / 121.2, 8000 442 / 434, 16384 1803 / 1768 (1244 TFLOP/s);
// six of 3600 437 / 417.  Which calls it takes: prefill_wide() in prefill_route.h.
//
// Workgroup = (sequence, 4 query heads of one KV head, 64 consecutive query rows), four wavefronts of 16 rows, one
// workgroup per compute unit.  Column C = kWaveRows * head + row of a wavefront is column c = C % 32 of group C / 32.
// Layouts of the tiles, of the weights and of the LDS stages are those of paged_attention_prefill32.hip: lane = 32 *
// half + c holds the 16 scores of column c against tokens 8 (v / 4) + 4 half + v % 4; K rows with 16-byte chunks
// XOR-permuted by the row, V rows with 64-byte granules rotated by the row, both written by direct loads.
//
// Turn s of the pipeline: S(s + 1) = K . Q (matrix instructions 0 .. 15), the weights of step s, and O += V . P of step
// s - 1 (16 .. 31).  Three steps are in flight, so the softmax arithmetic spreads over the whole turn.
//
// The reference point of a column is set kBias above its largest score, and moves when some weight reaches 2: that
// shows in the exponent bits of the rounded weights, which are collected by OR (10 instructions instead of the 20 of a
// running maximum).  The weights of the step are then made again from its scores, which stay in registers; weights are
// below 2 as they reach O and the sum, and so below 2^(kBias + 1) times what the largest score of the last move weighs.
//
// The score products are inline asm: the compiler would put their results into AGPRs and copy each score.  It inserts
// no wait states for them, so nothing near them needs any: scores are read two and more matrix instructions after the
// last one that writes them, operands come from LDS and from Q (checked in the compiled form by a test).
#include <float.h>
#include <math.h>

#include <type_traits>

#include "kvc_internal.h"
#include "pa_prefill32_tile.h"

namespace kvc {

namespace {

using namespace prefill32;

// Chunk of the turn (one matrix instruction each) in which the arithmetic of score e starts: argument, exponential,
// rounding and pair sum, sum, one chunk after the other.  Score e: register 2 (e / 4) + e % 2 of group (e / 2) % 2.
constexpr int arg_chunk(int e) { return e * 3 / 4; }
// Chunks of the loads: behind the LDS reads.  Between them a turn takes 1426 to 1470 cycles instead of 1391.
constexpr int kLoadK = 27, kLoadV = 29;

// One turn: S of step `next`, the weights of step cur (raw scores in x), O += V . P of the step before (weights in w).
//     chunks  0 .. 15   S += K operand j . Q, both groups; reads K operands 4 .. 7, then the V operands
//     chunks 16 .. 31   O block += V operand . weights, both groups; reads K operands 0 .. 3 of the step after next,
//                       requests the K rows of the step four ahead of cur and the V rows of the step two ahead
// The turn starts with ka[0 .. 3] = K operands of step next.  On return x holds the raw scores of step next, w the
// weights of step cur.  MASKED: `vlim_prev` = tokens of the step before that some column sees, `limit_next` = tokens of
// step next that this lane's columns see.
template <bool MASKED, class IssueK, class IssueV, class Lookup, class Math>
__device__ inline void pipeline_turn(floatx16 (&acc)[2][4], float (&x)[2][16], uint32_t (&w)[2][8], float (&lsum)[2], float (&m)[2],
                                     bf16x8 (&ka)[8], const unsigned char *krow1, const unsigned char *krow2, const unsigned char *sv_prev,
                                     const int (&voff)[4], const bf16x8 (&qb)[2][8], float scale_log2e, int vlim_prev,
                                     const int (&limit_next)[2], int half, int c, const IssueK &issue_k, const IssueV &issue_v,
                                     const Lookup &lookup, const Math &math) {
    float arg[32], pf[32], pair[16];
    uint2 va[8][2];
    uint32_t wn[2][8], any[4];
    floatx16 s[2];
    const float neg_m[2] = {-m[0], -m[1]}, lsum_before[2] = {lsum[0], lsum[1]};
    static_for<0, 32>([&](auto chunk) __attribute__((always_inline)) {
        constexpr int T = decltype(chunk)::value;
        KVC_PIN();
        if constexpr (T < 16) {
            constexpr int J = T >> 1, G = T & 1;
            if constexpr (J == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s[G]) : "v"(ka[J]), "a"(qb[G][J]));
            else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s[G]) : "v"(ka[J]), "a"(qb[G][J]));
        } else {
            constexpr int U = (T - 16) >> 1, G = T & 1, N = U >> 2, B = U & 3;
            if constexpr (G == 0 && MASKED) mask_v_operand<N>(va[U], vlim_prev, half);
            acc[G][B] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(va[U]), four_words(w[G], N), acc[G][B], 0, 0, 0);
        }
        if constexpr (T < 4) ka[4 + T] = read_k_operand<4 + T>(krow1, half, c);
        if constexpr (T >= 4 && T < 20) {
            constexpr int U = (T - 4) >> 1, H = T & 1;
            va[U][H] = read_v_half<(U >> 2), H>(sv_prev + voff[U & 3]);
        }
        if constexpr (T >= 20 && T < 24) ka[T - 20] = read_k_operand<T - 20>(krow2, half, c);
        static_for<0, 32>([&](auto score) __attribute__((always_inline)) {
            constexpr int E = decltype(score)::value, P = E >> 1;
            constexpr int G = P & 1, V = 2 * (P >> 1) + (E & 1);
            if constexpr (arg_chunk(E) == T) arg[E] = __builtin_fmaf(x[G][V], scale_log2e, neg_m[G]);
            if constexpr (arg_chunk(E) + 1 == T) pf[E] = __builtin_amdgcn_exp2f(arg[E]);
            if constexpr ((E & 1) && arg_chunk(E) + 2 == T) {
                wn[G][P >> 1] = pack_bf16(pf[E - 1], pf[E]);
                asm volatile("" : "+v"(wn[G][P >> 1]));
                pair[P] = pf[E - 1] + pf[E];
            }
            if constexpr ((E & 1) && arg_chunk(E) + 3 == T) {
                lsum[G] += pair[P];
                asm volatile("" : "+v"(lsum[G]));
            }
            if constexpr ((E & 7) == 7 && arg_chunk(E) + 3 == T) {   // words of pairs P - 3 .. P
                constexpr int I = P >> 1;
                uint32_t o = wn[0][I - 1] | wn[1][I - 1] | wn[0][I];
                if constexpr (P >= 4) o = o | wn[1][I] | any[(P >> 2) - 1];
                else o = o | wn[1][I];
                asm volatile("" : "+v"(o));
                any[P >> 2] = o;
            }
        });
        if constexpr (T == 0) lookup();
        if constexpr (T == 31) math();
        if constexpr (T == kLoadK) issue_k();
        if constexpr (T == kLoadV) issue_v();
        if constexpr (MASKED && T == 18) {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int v = 0; v < 16; ++v) s[g][v] = 8 * (v >> 2) + 4 * half + (v & 3) >= limit_next[g] ? -INFINITY : s[g][v];
        }
    });
    KVC_PIN();
    // Both ways to the join below have the accumulators in AGPRs: otherwise they are copied there and back in each turn.
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int b = 0; b < 4; ++b) asm volatile("" : "+a"(acc[g][b]));
    if (__builtin_expect(__builtin_amdgcn_ballot_w64((any[3] & 0x40004000u) != 0) != 0, 0)) {
        // some weight is 2 or more (or NaN): a new reference point, and the weights by it
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            float top = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) top = fmaxf(top, x[g][v]);
            const float m_new = fmaxf(m[g], max_over_halves(top) * scale_log2e + kBias);
            const float alpha = __builtin_amdgcn_exp2f(m[g] - m_new);
            m[g] = m_new;
            lsum[g] = lsum_before[g] * alpha;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                acc[g][b] *= alpha;
                asm volatile("" : "+a"(acc[g][b]));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float a = __builtin_amdgcn_exp2f(__builtin_fmaf(x[g][2 * i], scale_log2e, -m_new));
                const float b = __builtin_amdgcn_exp2f(__builtin_fmaf(x[g][2 * i + 1], scale_log2e, -m_new));
                wn[g][i] = pack_bf16(a, b);
                lsum[g] += a + b;
            }
        }
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
#pragma unroll
        for (int v = 0; v < 16; ++v) x[g][v] = s[g][v];
#pragma unroll
        for (int i = 0; i < 8; ++i) w[g][i] = wn[g][i];
    }
}

// SMALL: block_size < 8, rows gathered by a table look-up per lane.
template <bool SMALL>
__global__ __launch_bounds__(256, 1) __attribute__((amdgpu_waves_per_eu(1, 1))) void pa_prefill_wide_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k_cache, const uint16_t *__restrict__ v_cache,
    const int32_t *__restrict__ block_tables, const int32_t *__restrict__ context_lens, const int32_t *__restrict__ q_start,
    uint16_t *__restrict__ out, PrefillParams p, int spread) {
    constexpr int kHeads = 4;
    constexpr int kWaveRows = 64 / kHeads;         // query rows of a wavefront
    constexpr int kTileRows = 4 * kWaveRows;       // and of the workgroup
    constexpr int kQBytes = 64 * D * 2;            // Q rows of a wavefront's columns
    __shared__ __attribute__((aligned(1024))) unsigned char s_k[kRing * kStageBytes], s_v[kRing * kStageBytes], s_q4[4 * kQBytes];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int half = lane >> 5, c = lane & 31;
    unsigned char *const s_q = s_q4 + wave * kQBytes;

    const int chunks = p.num_q_heads / kHeads;
    // blockIdx.x = head chunk + chunks * (seq + num_seqs * order), the longest query tiles first
    const int chunk = chunk_at(blockIdx.x % chunks, spread), index = blockIdx.x / chunks;
    const int head0 = chunk * kHeads;
    const int kvh = head0 / p.group;
    const int n = index % p.num_seqs, qtile = p.max_query_tiles - 1 - index / p.num_seqs;
    const int S = context_lens[n], qs = q_start[n], Qn = q_start[n + 1] - qs;
    if (qtile * kTileRows >= Qn || Qn > S) return;  // uniform over the workgroup
    const int last_pos = S - Qn + min(Qn, (qtile + 1) * kTileRows) - 1;  // position of the workgroup's last query row
    const int steps = last_pos / kStepTokens + 1;
    const int32_t *const table = block_tables + size_t(n) * p.max_blocks_per_seq;
    // a wavefront past the last query row shadows that row
    const int first_row = qtile * kTileRows + kWaveRows * wave;
    const bool active = first_row < Qn;
    const int i0 = min(first_row, Qn - 1);
    const int nrows = min(kWaveRows, Qn - i0);
    const int p0 = S - Qn + i0;         // position of row 0
    const int wave_vis = p0 + nrows;    // tokens visible to some column

    // This wavefront's share of a step's rows: 8 consecutive ones, inside one 16-row tile and one block (SMALL apart).
    const size_t head_bytes = size_t(p.block_size) * D * 2;
    const size_t block_bytes = head_bytes * p.num_kv_heads;
    const unsigned char *const k_head = reinterpret_cast<const unsigned char *>(k_cache) + size_t(kvh) * head_bytes;
    const unsigned char *const v_head = reinterpret_cast<const unsigned char *>(v_cache) + size_t(kvh) * head_bytes;
    const unsigned tile_mask = (p.block_size - 1) & ~15;  // of a token: its 16-row tile inside its block
    const int share_row = 8 * wave;
    const int lchunk = lane & 15;
    const int lrow = (share_row & 15) + (lane >> 4);  // row of load 0 in its tile; load 1: + 4
    const int brow = lrow & (p.block_size - 1);       // in its block, where that holds 8 tokens (16 or more: lrow)
    // offsets of load 1 are 1024 bytes on through its immediate, on both sides
    const uint32_t k_off[2] = {uint32_t(brow * 256 + ((lchunk ^ lrow) << 4)), uint32_t(brow * 256 + ((lchunk ^ (lrow + 4)) << 4))};
    const uint32_t v_off = brow * 256 + ((4 * (((lchunk >> 2) - lrow) & 3) + (lchunk & 3)) << 4);
    const uint32_t lds_k0 = uint32_t(reinterpret_cast<uintptr_t>(s_k)) + 256 * share_row;
    const uint32_t lds_v0 = uint32_t(reinterpret_cast<uintptr_t>(s_v)) + 256 * share_row;
    const uint32_t lds_q0 = uint32_t(reinterpret_cast<uintptr_t>(s_q));
    const unsigned char *const k_lane = s_k + c * 256;
    int voff[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) voff[b] = v_lane_offset(b, half, c);

    // Block ids of the wavefront's rows, through the scalar cache a turn before the loads (SMALL: of this lane's rows in
    // loads 0 and 1), then their byte offsets.  Rows past the last visible token repeat it (never used unmasked).
    struct Ids { uint32_t a, b; };
    int tok_next = share_row;
    auto next_ids = [&]() __attribute__((always_inline)) -> Ids {
        Ids id;
        if constexpr (SMALL) {
            const int tok = tok_next - (share_row & 15) + lrow;
            id.a = table[min(tok, last_pos) >> p.block_size_log2];
            id.b = table[min(tok + 4, last_pos) >> p.block_size_log2];
        } else {
            const unsigned tok = unsigned(min(tok_next, last_pos));
            // the byte offset fits 32 bits (blocks of 8 tokens and more), which the scalar load adds by itself
            id.a = *reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(table) + (tok >> p.block_size_log2) * 4u);
            id.b = (tok & tile_mask) * 256;
        }
        tok_next += kStepTokens;
        return id;
    };
    using At = std::conditional_t<SMALL, Ids, uint64_t>;
    auto offset_of = [&](const Ids &id) __attribute__((always_inline)) -> At {
        if constexpr (SMALL) return id;
        else return uint64_t(id.a) * uint32_t(block_bytes) + id.b;
    };
    auto issue_rows = [&](const unsigned char *head, uint32_t off0, uint32_t off1_minus_1k, uint32_t lds, const At &at) __attribute__((always_inline)) {
        lds = __builtin_amdgcn_readfirstlane(lds);
        if constexpr (SMALL) {
            load_lane_to_lds(head + size_t(at.a) * block_bytes + (lrow & (p.block_size - 1)) * 256 + (off0 & 255), lds);
            load_lane_to_lds(head + size_t(at.b) * block_bytes + ((lrow + 4) & (p.block_size - 1)) * 256 + (off1_minus_1k & 255), lds + 1024);
        } else {
            load_rows(head + at, off0, off1_minus_1k, lds);
        }
    };
    auto issue_k = [&](int stage, const At &at) __attribute__((always_inline)) {
        issue_rows(k_head, k_off[0], k_off[1], lds_k0 + stage * kStageBytes, at);
    };
    auto issue_v = [&](int stage, const At &at) __attribute__((always_inline)) {
        issue_rows(v_head, v_off, v_off, lds_v0 + stage * kStageBytes, at);
    };
    // Q rows go through LDS as well: their loads are then waited for together with those of the first K and V rows.
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int C = 4 * i + (lane >> 4), row = min(C % kWaveRows, nrows - 1);
        load_lane_to_lds(reinterpret_cast<const unsigned char *>(q) +
                             (size_t(qs + i0 + row) * p.num_q_heads + head0 + C / kWaveRows) * (D * 2) + ((lchunk ^ (C & 15)) << 4),
                         __builtin_amdgcn_readfirstlane(lds_q0 + 1024 * i));
    }
    // Rows of step j live in stages j % 4.  Turn s requests the K rows of step s + 4 (over those of step s) and the V rows
    // of step s + 2 (over those of step s - 2), and reads K rows of steps s + 1 and s + 2 and V rows of step s - 1.  Before
    // the barrier that ends it a wavefront waits for its LDS reads and for its loads of turn s - 1 (the V rows of step s + 1
    // are read in turn s + 2, or by the last step in place of turn s + 1).
    At at_v[2], at_k;
    static_for<0, kRing>([&](auto i) __attribute__((always_inline)) {
        constexpr int I = decltype(i)::value;
        const At at = offset_of(next_ids());
        issue_k(I, at);
        if constexpr (I < kRing - 2) issue_v(I, at);
        if constexpr (I >= kRing - 2) at_v[I - (kRing - 2)] = at;
    });
    at_k = offset_of(next_ids());
    Ids ids;
    // V rows of the step before the first: turn 0, or the last step if it is the first, multiplies them by weights of 0
#pragma unroll
    for (int i = 0; i < kStageBytes / 4096; ++i)
        *reinterpret_cast<uint4 *>(s_v + (kRing - 1) * kStageBytes + (4 * i + wave) * 1024 + lane * 16) = uint4{0, 0, 0, 0};
    wait_for<0, 0>();
    barrier();

    bf16x8 qb[2][8];
    static_for<0, 8>([&](auto j) __attribute__((always_inline)) {
        constexpr int J = decltype(j)::value;
        qb[0][J] = read_k_operand<J>(s_q + c * 256, half, c);
        qb[1][J] = read_k_operand<J>(s_q + (32 + c) * 256, half, c);
    });
    floatx16 acc[2][4];
    float x[2][16], m[2], lsum[2];
    uint32_t w[2][8];
    bf16x8 ka[8];
    int seen[2];  // tokens that a column sees
#pragma unroll
    for (int g = 0; g < 2; ++g) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[g][b][v] = 0.f;
        lsum[g] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) w[g][i] = 0;
        seen[g] = p0 + min((32 * g + c) % kWaveRows, nrows - 1) + 1;
    }
    {  // scores of step 0
        floatx16 sc[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[0][v] = sc[1][v] = 0.f;
        static_for<0, 8>([&](auto j) __attribute__((always_inline)) {
            constexpr int J = decltype(j)::value;
            const bf16x8 a = read_k_operand<J>(k_lane, half, c);
            sc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qb[0][J], sc[0], 0, 0, 0);
            sc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qb[1][J], sc[1], 0, 0, 0);
        });
        static_for<0, 4>([&](auto j) __attribute__((always_inline)) {
            constexpr int J = decltype(j)::value;
            ka[J] = read_k_operand<J>(k_lane + kStageBytes, half, c);
        });
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            float top = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                x[g][v] = 8 * (v >> 2) + 4 * half + (v & 3) >= seen[g] ? -INFINITY : sc[g][v];
                top = fmaxf(top, x[g][v]);
            }
            // not below the lowest finite value: a first step of -inf scores weighs nothing then, instead of -inf - -inf
            m[g] = fmaxf(max_over_halves(top) * p.scale_log2e + kBias, -FLT_MAX);
        }
    }
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int j = 0; j < 8; ++j) asm volatile("" : "+a"(qb[g][j]));
    wait_for<0, 0>();
    barrier();  // the first K stage has been read, and Q: turn 0 may load step 4 over it

    int s = 0;
#define KVC_TURN(MASKED, PHASE, VLIM, LIMIT0, LIMIT1)                                                                 \
    {                                                                                                                 \
        const int ph = (PHASE);                                                                                       \
        auto turn_math = [&]() __attribute__((always_inline)) {                                                       \
            at_v[0] = at_v[1];                                                                                        \
            at_v[1] = at_k;                                                                                           \
            at_k = offset_of(ids);                                                                                    \
        };                                                                                                            \
        auto turn_k = [&]() __attribute__((always_inline)) { issue_k(ph, at_k); };                                    \
        auto turn_v = [&]() __attribute__((always_inline)) { issue_v((ph + kRing - 2) % kRing, at_v[0]); };           \
        auto turn_lookup = [&]() __attribute__((always_inline)) { ids = next_ids(); };                                \
        const int lim[2] = {LIMIT0, LIMIT1};                                                                          \
        pipeline_turn<MASKED>(acc, x, w, lsum, m, ka, k_lane + ((ph + 1) % kRing) * kStageBytes,                      \
                              k_lane + ((ph + 2) % kRing) * kStageBytes, s_v + ((ph + kRing - 1) % kRing) * kStageBytes,\
                              voff, qb, p.scale_log2e, VLIM, lim, half, c, turn_k, turn_v, turn_lookup, turn_math);   \
        wait_for<4, 0>();                                                                                             \
        barrier();                                                                                                    \
        ++s;                                                                                                          \
    }
    const int plain = min((p0 + 1) / kStepTokens - 1, steps - 1);  // turns whose next step every column sees whole
    // One after the other and not as paths of one loop: the compiler would keep a copy of the accumulators for each.
    while (s + kRing <= plain) {
        KVC_TURN(false, 0, 0, 0, 0)
        KVC_TURN(false, 1, 0, 0, 0)
        KVC_TURN(false, 2, 0, 0, 0)
        KVC_TURN(false, 3, 0, 0, 0)
    }
    while (s < plain) KVC_TURN(false, s % kRing, 0, 0, 0)
    while (s < steps - 1)
        KVC_TURN(true, s % kRing, wave_vis - (s - 1) * kStepTokens, seen[0] - (s + 1) * kStepTokens, seen[1] - (s + 1) * kStepTokens)
#undef KVC_TURN
    // the last step, a turn without scores of a next one
    {
        float top[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            top[g] = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) top[g] = fmaxf(top[g], x[g][v]);
            top[g] = fmaxf(m[g], max_over_halves(top[g]) * p.scale_log2e - 1.0f);
        }
        auto pv = [&](const unsigned char *sv, int vlim, const uint32_t (&ww)[2][8]) __attribute__((always_inline)) {
            static_for<0, 8>([&](auto u) __attribute__((always_inline)) {
                constexpr int U = decltype(u)::value, N = U >> 2, B = U & 3;
                uint2 va[2] = {read_v_half<N, 0>(sv + voff[B]), read_v_half<N, 1>(sv + voff[B])};
                mask_v_operand<N>(va, vlim, half);
                acc[0][B] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(va), four_words(ww[0], N), acc[0][B], 0, 0, 0);
                acc[1][B] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(va), four_words(ww[1], N), acc[1][B], 0, 0, 0);
            });
        };
        pv(s_v + ((s + kRing - 1) % kRing) * kStageBytes, wave_vis - (s - 1) * kStepTokens, w);
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int b = 0; b < 4; ++b) asm volatile("" : "+a"(acc[g][b]));
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(top[0] > m[0] || top[1] > m[1]) != 0, 0)) {
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const float alpha = __builtin_amdgcn_exp2f(m[g] - top[g]);
                lsum[g] *= alpha;
                m[g] = top[g];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    acc[g][b] *= alpha;
                    asm volatile("" : "+a"(acc[g][b]));
                }
            }
        }
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float a = __builtin_amdgcn_exp2f(__builtin_fmaf(x[g][2 * i], p.scale_log2e, -m[g]));
                const float b = __builtin_amdgcn_exp2f(__builtin_fmaf(x[g][2 * i + 1], p.scale_log2e, -m[g]));
                w[g][i] = pack_bf16(a, b);
                lsum[g] += a + b;
            }
        pv(s_v + (s % kRing) * kStageBytes, wave_vis - s * kStepTokens, w);
    }
    wait_for<0, 0>();  // nothing may still be landing in LDS when the workgroup's LDS is handed on
    // lane (half, c) holds O[column 32 g + c][32 b + 8 a + 4 half .. +3] in acc[g][b][4 a .. 4 a + 3]
    auto store = [&](int g, int b, const float (&o)[16], float inv) __attribute__((always_inline)) {
        const int C = 32 * g + c, row = C % kWaveRows;
        if (active && row < nrows) {
            uint16_t *const dst = out + (size_t(qs + i0 + row) * p.num_q_heads + head0 + C / kWaveRows) * D + 32 * b + 8 * half;
#pragma unroll
            for (int a = 0; a < 4; a += 2) {
                // halves swap four dims, so that each lane stores eight
                const u32x2 lo = __builtin_amdgcn_permlane32_swap(pack_bf16(o[4 * a] * inv, o[4 * a + 1] * inv),
                                                                  pack_bf16(o[4 * a + 4] * inv, o[4 * a + 5] * inv), false, false);
                const u32x2 hi = __builtin_amdgcn_permlane32_swap(pack_bf16(o[4 * a + 2] * inv, o[4 * a + 3] * inv),
                                                                  pack_bf16(o[4 * a + 6] * inv, o[4 * a + 7] * inv), false, false);
                *reinterpret_cast<uint4 *>(dst + 8 * a) = uint4{lo[0], hi[0], lo[1], hi[1]};
            }
        }
    };
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const float inv = 1.0f / sum_over_halves(lsum[g]);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            float o[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) o[v] = acc[g][b][v];
            store(g, b, o, inv);
        }
    }
}

}  // namespace

hipError_t launch_prefill_wide(const void *q, const void *k_cache, const void *v_cache, const int32_t *block_tables,
                               const int32_t *context_lens, const int32_t *q_start, void *out, const PrefillParams &p,
                               hipStream_t stream) {
    const int64_t grid = int64_t(p.num_q_heads / 4) * p.num_seqs * p.max_query_tiles;
    const auto kernel = p.block_size < 8 ? pa_prefill_wide_kernel<true> : pa_prefill_wide_kernel<false>;
    kernel<<<dim3(unsigned(grid)), dim3(256), 0, stream>>>(static_cast<const uint16_t *>(q), static_cast<const uint16_t *>(k_cache),
                                                           static_cast<const uint16_t *>(v_cache), block_tables, context_lens,
                                                           q_start, static_cast<uint16_t *>(out), p, chunk_spread(p.num_q_heads / 4, p.group / 4));
    return hipGetLastError();
}

}  // namespace kvc

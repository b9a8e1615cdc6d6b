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
// One workgroup = (sequence, 2 query heads sharing one KV head, 64 consecutive query rows); each of
// its 4 wavefronts owns 16 query rows x 2 heads = the 32 columns of its tiles (column c = 16 * head
// + row).  Odd GQA group sizes take one head and 32 query rows per wavefront instead (workgroups of
// 128 rows); everything below is written for two heads and holds for one with "row" = c.  The
// workgroup walks the context in steps of 32 tokens (the 32 rows of a score tile).
//
// What bounds it.  Two wavefronts of a SIMD read 128 KiB of operands from LDS per step of a compute
// unit, 1024 cycles of its bandwidth against 1024 matrix cycles; a step of both takes about 1450 cycles
// in long launches, 1600 in four chunks of 512 rows and 1850 at 2048 tokens.  Rows that are not in L2 are
// not what the chunks wait for: with the heads of a KV head on one XCD their launch misses 0.81 M times
// instead of 1.52 M, and takes the same time (matrix pipes busy 55 % of the cycles, 1.80 GHz).
// One alone is bound by its own issue, about 130 instructions of 4 to 5 cycles (8 for an
// exponential), and takes about 950 cycles for 512 matrix cycles.  A turn holds three steps: the
// scores of the next, the weights of this one, V . P of the one before, so that the softmax
// arithmetic spreads over the whole turn and neither product waits for it.  32 / 8 heads, one
// request, turns of two steps (scores of the next beside weights and V . P of this one) / of three:
// 100 tokens 8.6 / 7.5 us, 1000 22.6 / 21.5, 2048 44.3 / 39.6; four chunks of 512 rows of up to 4000
// tokens 109.9 / 103.8; 256 rows of 12000 tokens 137 / 118.5.
//
// K and V rows travel from the cache straight into LDS (global_load_lds_dwordx4: lane l of a
// wavefront writes its 16 bytes at M0 + 16 * l, no register staging), requested a turn
// or more before their first use (K rows four steps ahead, V rows two); which bytes a
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
//   softmax            all 16 scores of a lane belong to one column: one fused multiply-add and one
//                      exponential per score (weight = exp2(score * scale - m)); the weights are
//                      rounded to bf16 for P.V and added up in fp32 for the normaliser.  The
//                      reference point m is set 2^kBias above the largest score and moves when some
//                      weight reaches 2, which shows in the exponent bits of the rounded weights;
//                      they are collected by OR (4 instructions, a running maximum takes 9), and the
//                      step's weights are then made again from its scores.  The two halves of a
//                      column meet only there and once at the end.
//   O^T += V^T . P^T   8 x v_mfma_f32_32x32x16_bf16: 4 blocks of 32 dims x 2 slices of 16
//                      tokens.  B is the weight registers as they stand (slice n = registers
//                      8n .. 8n+7, depth slot 8*half + i = token 16n + 8*(i/4) + 4*half + i%4);
//                      A = V^T comes from LDS in that token order by transposing reads
//                      (ds_read_b64_tr_b16: 4 consecutive tokens of the lane's dim per read).
//
// The causal mask only bites in the last one or two steps of a wavefront: steps entirely below
// the diagonal of all 16 rows run code without mask or range checks.  Workgroups with the most
// steps (the last query rows) are dispatched first.
#include <float.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "kvc_internal.h"
#include "pa_prefill32_tile.h"

namespace kvc {

namespace {

using namespace prefill32;

// Chunk of the turn (one matrix instruction each) in which the arithmetic of score e starts: argument, exponential,
// rounding and pair sum, sum, one chunk after the other.
constexpr int arg_chunk(int e) { return e * 10 / 16; }

// One turn: S of step `next`, the weights of step cur (raw scores in x), O += V . P of the step before (weights in w).
// Products with K and with V alternate, so that no matrix instruction waits for the one in front of it.
//     even chunks   S += K operand j . Q
//     odd chunks    O block += V operand u . weights
// LDS reads: K operands 4 .. 7 of step next and V operands 3 .. 7 of the step before, then K operands 0 .. 3 of the step
// after next and V operands 0 .. 2 of step cur, which the following turn starts with.  `issue` requests the K rows of the
// step four ahead of cur and the V rows of the step two ahead.  On return x holds the raw scores of step next, w the
// weights of step cur.  MASKED: `vlim_prev`, `vlim_cur` = tokens of those steps that some column sees, `limit_next` =
// tokens of step next that this lane's column sees.
template <bool MASKED, class IssueK, class IssueV, class Lookup, class Math>
__device__ inline void pipeline_turn(floatx16 (&acc)[4], float (&x)[16], uint32_t (&w)[8], float &lsum, float &m, bf16x8 (&ka)[8],
                                     uint2 (&va)[8][2], const unsigned char *krow1, const unsigned char *krow2,
                                     const unsigned char *sv_prev, const unsigned char *sv_cur, const int (&voff)[4],
                                     const bf16x8 (&qb)[8], float scale_log2e, int vlim_prev, int limit_next, int half, int c,
                                     const IssueK &issue_k, const IssueV &issue_v, const Lookup &lookup, const Math &math) {
    float arg[16], pf[16], pair[8];
    uint32_t wn[8], any[3];
    uint64_t moved = 0;
    floatx16 s;
    const float neg_m = -m, lsum_before = lsum;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
    static_for<0, 16>([&](auto chunk) __attribute__((always_inline)) {
        constexpr int T = decltype(chunk)::value, U = T >> 1;
        KVC_PIN();
        if constexpr ((T & 1) == 0) {
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[U], qb[U], s, 0, 0, 0);
        } else {
            if constexpr (MASKED) mask_v_operand<(U >> 2)>(va[U], vlim_prev, half);
            acc[U & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(va[U]), four_words(w, U >> 2), acc[U & 3], 0, 0, 0);
        }
        if constexpr (T < 4) ka[4 + T] = read_k_operand<4 + T>(krow1, half, c);
        if constexpr (T < 10) {
            constexpr int R = 3 + (T >> 1), H = T & 1;
            va[R][H] = read_v_half<(R >> 2), H>(sv_prev + voff[R & 3]);
        }
        if constexpr (T >= 8 && T < 12) ka[T - 8] = read_k_operand<T - 8>(krow2, half, c);
        if constexpr (T >= 8 && T < 14) {
            constexpr int R = (T - 8) >> 1, H = T & 1;
            va[R][H] = read_v_half<0, H>(sv_cur + voff[R]);
        }
        static_for<0, 16>([&](auto score) __attribute__((always_inline)) {
            constexpr int E = decltype(score)::value, P = E >> 1;
            if constexpr (arg_chunk(E) == T) arg[E] = __builtin_fmaf(x[E], scale_log2e, neg_m);
            if constexpr (arg_chunk(E) + 1 == T) pf[E] = __builtin_amdgcn_exp2f(arg[E]);
            if constexpr ((E & 1) && arg_chunk(E) + 2 == T) {
                wn[P] = pack_bf16(pf[E - 1], pf[E]);
                asm volatile("" : "+v"(wn[P]));
                pair[P] = pf[E - 1] + pf[E];
            }
            if constexpr ((E & 1) && arg_chunk(E) + 3 == T) {
                lsum += pair[P];
                asm volatile("" : "+v"(lsum));
                if constexpr (P == 2) { any[0] = wn[0] | wn[1] | wn[2]; asm volatile("" : "+v"(any[0])); }
                if constexpr (P == 4) { any[1] = any[0] | wn[3] | wn[4]; asm volatile("" : "+v"(any[1])); }
                if constexpr (P == 6) { any[2] = any[1] | wn[5] | wn[6]; asm volatile("" : "+v"(any[2])); }
            }
        });
        if constexpr (T == 0) lookup();
        if constexpr (T == 12) issue_k();
        if constexpr (T == 14) issue_v();
        if constexpr (T == 14) moved = __builtin_amdgcn_ballot_w64(((any[2] | wn[7]) & 0x40004000u) != 0);
        if constexpr (T == 15) math();
    });
    KVC_PIN();
    if (MASKED)
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 8 * (v >> 2) + 4 * half + (v & 3) >= limit_next ? -INFINITY : s[v];
    if (__builtin_expect(moved != 0, 0)) {
        // some weight is 2 or more (or NaN): a new reference point, and the weights by it
        float top = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) top = fmaxf(top, x[v]);
        const float m_new = fmaxf(m, max_over_halves(top) * scale_log2e + kBias);
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        lsum = lsum_before * alpha;
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[b] *= alpha;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float a = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * i], scale_log2e, -m_new));
            const float b = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * i + 1], scale_log2e, -m_new));
            wn[i] = pack_bf16(a, b);
            lsum += a + b;
        }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = s[v];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = wn[i];
}

// HEADS = 2: the 32 columns of a wavefront are 16 query rows x 2 heads of one KV head (even GQA
// groups); HEADS = 1: 32 query rows of one head.  Two workgroups of four wavefronts share a compute unit, two
// wavefronts a SIMD.
// SPLIT: a workgroup has two groups of four wavefronts that hold the same query rows and
// share the steps of long contexts: group 0 walks the first `cut` of them, group 1 the rest, each with a ring
// of stages of its own, and the parts meet in LDS at the end (log-sum-exp rule).  Of short contexts group 1
// ends at once.  For launches with too few workgroups to fill the device, where a four-wavefront workgroup would
// run one wavefront per SIMD (256 rows at the end of 12000 tokens, 32 / 8 heads, 118 us).
// SMALL: block_size < 8 (spills 4 registers with two heads, 2 with one; 2048 tokens, 32 / 8 heads: blocks of 4 43.0 us, of 16 40.0).
template <bool SMALL, int HEADS, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? 512 : 256, SPLIT ? 1 : 2) void pa_prefill_mfma32_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k_cache,
    const uint16_t *__restrict__ v_cache, const int32_t *__restrict__ block_tables,
    const int32_t *__restrict__ context_lens, const int32_t *__restrict__ q_start,
    uint16_t *__restrict__ out, PrefillParams p, int query_tiles, int fold_at, int fold_ranked, int rank_from, int by_units, int spread) {
    constexpr int kParts = SPLIT ? 2 : 1;
    __shared__ __attribute__((aligned(1024))) unsigned char s_kv[kParts][2 * kRing][kStageBytes];
    constexpr int kWaveRows = 32 / HEADS;           // query rows of a wavefront: column c = kWaveRows * head + row
    constexpr int kTileRows = 4 * kWaveRows;        // query rows of a workgroup

    // blockIdx.x = head chunk + chunks * (seq + num_seqs * order); the longest query tiles come
    // first, and from `fold_at` on the shortest: when every workgroup is resident at once, the two
    // that share a compute unit are then a long and a short one.  With a context of `rank_from` tokens or more in
    // the batch (0: never) the same order is taken over the tiles of all sequences by the steps they walk,
    // which only the device knows.
    // by_units (all workgroups, or 0): blockIdx.x places the head by head_place() instead.  spread: chunk_spread() of the chunks.
    int head0, kvh, index;
    if (HEADS == 1 && by_units > 0) {
        const HeadPlace at = head_place(blockIdx.x, by_units, p.group, p.num_kv_heads);
        head0 = at.head, kvh = at.kv_head, index = at.index;
    } else {
        const int chunks = p.num_q_heads / HEADS;
        head0 = chunk_at(blockIdx.x % chunks, spread) * HEADS, index = blockIdx.x / chunks;
        kvh = head0 / p.group;
    }

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
    const int group = wave_id >> 2;  // SPLIT: wavefronts w and w + 4 share a SIMD
    const int wave = SPLIT ? wave_id & 3 : wave_id;  // among the wavefronts that share a ring
    unsigned char *const s_k = &s_kv[SPLIT ? group : 0][0][0], *const s_v = s_k + kRing * kStageBytes;
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

    // ---- this wavefront's share of a step's rows: 8 consecutive rows of the 32 (inside one 16-row tile of the step), two
    // loads of 4 rows for K and as many for V.  Lane l of load i writes LDS chunk l % 16 of the share's row 4 * i + l / 16;
    // the chunk it fetches for that place follows from the stage layouts.
    const size_t head_bytes = size_t(p.block_size) * D * 2;
    const size_t block_bytes = head_bytes * p.num_kv_heads;
    const unsigned char *k_head = reinterpret_cast<const unsigned char *>(k_cache) + size_t(kvh) * head_bytes;
    const unsigned char *v_head = reinterpret_cast<const unsigned char *>(v_cache) + size_t(kvh) * head_bytes;
    const unsigned tile_mask = (p.block_size - 1) & ~15;  // of a token: its 16-row tile inside its block
    const int my_tile = wave / 2;       // tile of the step this wavefront loads from
    const int lrow = 8 * (wave % 2) + (lane >> 4);  // row inside the tile of load 0 (load 1: + 4)
    const int lchunk = lane & 15;
    const int brow = lrow & (p.block_size - 1);  // in its block, where that holds 8 tokens (16 or more: lrow)
    const uint32_t k_off = brow * 256 + ((lchunk ^ lrow) << 4);
    const uint32_t k_off1 = (brow + 4) * 256 + ((lchunk ^ (lrow + 4)) << 4);
    const uint32_t v_off = brow * 256 + ((4 * (((lchunk >> 2) - lrow) & 3) + (lchunk & 3)) << 4);  // load 1: + 1024
    const uint32_t lds_k0 = uint32_t(reinterpret_cast<uintptr_t>(s_k)) + 2048 * wave;
    const uint32_t lds_v0 = uint32_t(reinterpret_cast<uintptr_t>(s_v)) + 2048 * wave;

    // Blocks of 8 tokens and more: the block id of the wavefront's 8 rows, which lie inside one block, is uniform; it comes
    // through the scalar cache one turn before the loads that use it.  Rows past the last visible token repeat it (never
    // used unmasked).  Smaller blocks: a / b are the blocks of this lane's row in loads 0 / 1.  (Four chunks of 512 rows on
    // 8-token blocks, contexts up to 4000, 32 / 8 heads: 112 us; with a table load per lane, which drains the wavefront's
    // loads in flight, 126 us.)
    const int share_row = 8 * (wave % 2);
    struct Ids { uint32_t a, b; };
    int tok_next = s0 * kStepTokens + 8 * wave;
    auto next_ids = [&]() __attribute__((always_inline)) -> Ids {
        Ids id;
        if constexpr (SMALL) {
            const int tok = tok_next - share_row + lrow;
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
        issue_rows(k_head, k_off, k_off1 - 1024, lds_k0 + stage * kStageBytes, at);
    };
    auto issue_v = [&](int stage, const At &at) __attribute__((always_inline)) {
        issue_rows(v_head, v_off, v_off, lds_v0 + stage * kStageBytes, at);
    };

    // Rows of step j live in stages j % 4.  Turn s requests the K rows of step s + 4 (over those of step s) and the V rows
    // of step s + 2 (over those of step s - 2), and reads K rows of steps s + 1 and s + 2 and V rows of steps s - 1 and s.
    // Before the barrier that ends it a wavefront waits for its LDS reads and for its loads of turn s - 1.  Past the last step
    // the last one is loaded again (unused): the loops stay branch free.
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
    auto turn_math = [&]() __attribute__((always_inline)) {                                       \
        at_v[0] = at_v[1];                                                                        \
        at_v[1] = at_k;                                                                           \
        at_k = offset_of(ids);                                                                    \
    };                                                                                            \
    auto turn_k = [&]() __attribute__((always_inline)) { issue_k(ph, at_k); };                    \
    auto turn_v = [&]() __attribute__((always_inline)) { issue_v((ph + 2) & 3, at_v[0]); };       \
    auto turn_lookup = [&]() __attribute__((always_inline)) { ids = next_ids(); }
#define KVC_TURN_END()                \
    wait_for<4, 0>();                 \
    barrier()
    // a turn of a wavefront that has nothing to compute: it only loads and synchronises
#define KVC_IDLE_TURN()                                                                           \
    {                                                                                             \
        KVC_TURN_BEGIN(s & 3);                                                                    \
        turn_lookup();                                                                            \
        turn_k();                                                                                 \
        turn_v();                                                                                 \
        turn_math();                                                                              \
        KVC_TURN_END();                                                                           \
    }

    // Group 0's share may be a step longer than group 1's.
    auto even_out = [&]() __attribute__((always_inline)) {
        if (group == 1)
            for (int i = wg_steps; i < cut; ++i) barrier();
    };

    // Every wavefront of a part passes the same barriers: one behind the scores of step 0, one per turn, wg_steps - 1 of
    // them; where two groups share a context, even_out() and two more around the exchange of the parts.  A wavefront
    // without query rows only loads and synchronises.
    if (!active) {
        __syncthreads();
        for (; s < wg_steps - 1; ++s) KVC_IDLE_TURN();
        wait_for<0, 0>();
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
    floatx16 acc[4];  // lane (half, c) holds O[column c][32*b + 8*(v/4) + 4*half + v%4] in acc[b][v]
    float x[16], m, lsum = 0.f;
    uint32_t w[8];
    bf16x8 ka[8];
    uint2 va[8][2];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = 0;
    const int seen = my_pos + 1 - s0 * kStepTokens;  // tokens of the part that this lane's column sees
    const int vis = wave_vis - s0 * kStepTokens;     // and some column
    {  // scores of step 0, then the operands turn 0 starts from
        floatx16 sc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = 0.f;
        static_for<0, 8>([&](auto j) __attribute__((always_inline)) {
            constexpr int J = decltype(j)::value;
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k_operand<J>(k_lane, half, c), qb[J], sc, 0, 0, 0);
        });
        static_for<0, 4>([&](auto j) __attribute__((always_inline)) {
            constexpr int J = decltype(j)::value;
            ka[J] = read_k_operand<J>(k_lane + kStageBytes, half, c);
        });
        static_for<0, 3>([&](auto u) __attribute__((always_inline)) {
            constexpr int U = decltype(u)::value;
            va[U][0] = va[U][1] = uint2{0, 0};
        });
        float top = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            x[v] = 8 * (v >> 2) + 4 * half + (v & 3) >= seen ? -INFINITY : sc[v];
            top = fmaxf(top, x[v]);
        }
        // not below the lowest finite value: a first step that hides all its tokens from a column, or whose scores are
        // -inf, weighs nothing then, instead of -inf - -inf
        m = fmaxf(max_over_halves(top) * p.scale_log2e + kBias, -FLT_MAX);
    }
    wait_for<0, 0>();
    __syncthreads();  // K stage 0 has been read: turn 0 may load step 4 over it

    // The turns whose next step is below the diagonal first (no mask), unrolled by the four phases of the stage rings, then
    // the ones that the causal mask touches, each loop for itself (as paths of one loop they cost a copy of the accumulators).
#define KVC_TURN(MASKED, PH, VLIM, LIMIT)                                                                      \
    {                                                                                                          \
        KVC_TURN_BEGIN(PH);                                                                                    \
        pipeline_turn<MASKED>(acc, x, w, lsum, m, ka, va, k_lane + ((ph + 1) & 3) * kStageBytes,       \
                                      k_lane + ((ph + 2) & 3) * kStageBytes, s_v + ((ph + 3) & 3) * kStageBytes, \
                                      s_v + ph * kStageBytes, voff, qb, p.scale_log2e, VLIM, LIMIT, half, c,   \
                                      turn_k, turn_v, turn_lookup, turn_math);                                 \
        KVC_TURN_END();                                                                                        \
        ++s;                                                                                                   \
    }
    // steps past the last token that any row of this wavefront sees carry no weight for it: it
    // only loads and synchronises during the workgroup's remaining turns
    const int live_steps = max(1, min(wg_steps, (wave_vis + kStepTokens - 1) / kStepTokens - s0));
    const int plain_turns = min(free_steps - 1, live_steps - 1);
    while (s + 4 <= plain_turns) {
        KVC_TURN(false, 0, 0, 0)
        KVC_TURN(false, 1, 0, 0)
        KVC_TURN(false, 2, 0, 0)
        KVC_TURN(false, 3, 0, 0)
    }
    while (s < plain_turns) KVC_TURN(false, s & 3, 0, 0)
    while (s < live_steps - 1) KVC_TURN(true, s & 3, vis - (s - 1) * kStepTokens, seen - (s + 1) * kStepTokens)
    // this wavefront's last step, a turn without scores of a next one
    {
        float top = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) top = fmaxf(top, x[v]);
        top = fmaxf(m, max_over_halves(top) * p.scale_log2e - 1.0f);
        static_for<0, 8>([&](auto u) __attribute__((always_inline)) {
            constexpr int U = decltype(u)::value;
            if constexpr (U >= 3) {
                const unsigned char *const sv = s_v + ((s + 3) & 3) * kStageBytes + voff[U & 3];
                va[U][0] = read_v_half<(U >> 2), 0>(sv);
                va[U][1] = read_v_half<(U >> 2), 1>(sv);
            }
            mask_v_operand<(U >> 2)>(va[U], vis - (s - 1) * kStepTokens, half);
            acc[U & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(va[U]), four_words(w, U >> 2), acc[U & 3], 0, 0, 0);
        });
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(top > m) != 0, 0)) {
            const float alpha = __builtin_amdgcn_exp2f(m - top);
            lsum *= alpha;
            m = top;
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[b] *= alpha;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float a = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * i], p.scale_log2e, -m));
            const float b = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * i + 1], p.scale_log2e, -m));
            w[i] = pack_bf16(a, b);
            lsum += a + b;
        }
        static_for<0, 8>([&](auto u) __attribute__((always_inline)) {
            constexpr int U = decltype(u)::value;
            const unsigned char *const sv = s_v + (s & 3) * kStageBytes + voff[U & 3];
            uint2 vl[2] = {read_v_half<(U >> 2), 0>(sv), read_v_half<(U >> 2), 1>(sv)};
            mask_v_operand<(U >> 2)>(vl, vis - s * kStepTokens, half);
            acc[U & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(vl), four_words(w, U >> 2), acc[U & 3], 0, 0, 0);
        });
    }
    for (; s < wg_steps - 1; ++s) KVC_IDLE_TURN();
#undef KVC_TURN
#undef KVC_IDLE_TURN
#undef KVC_TURN_BEGIN
#undef KVC_TURN_END
    wait_for<0, 0>();  // nothing may still be landing in LDS when the workgroup's LDS is handed on

    // lane (half, c) holds O[query row i0 + r][my_head][32*b + 8*a + 4*half .. +3] in acc[b][4a .. 4a+3]
    uint16_t *const dst = out + (size_t(qs + i0 + r) * p.num_q_heads + my_head) * D + 4 * half;
    lsum = sum_over_halves(lsum);
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
            for (int v = 0; v < 16; ++v) mine[(16 * b + v) * 64] = group == 0 ? acc[2 + b][v] : acc[b][v];
        mine[32 * 64] = m;
        mine[33 * 64] = lsum;
        __syncthreads();
        const float m_o = theirs[32 * 64], l_o = theirs[33 * 64];
        const float M = fmaxf(m, m_o);
        const float w_m = __builtin_amdgcn_exp2f(m - M), w_o = __builtin_amdgcn_exp2f(m_o - M);
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
                        o[i] = (w_m * (group == 0 ? acc[b][v] : acc[2 + b][v]) + w_o * theirs[(16 * b + v) * 64]) * inv;
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
                w.x = pack_bf16(acc[b][4 * a] * inv, acc[b][4 * a + 1] * inv);
                w.y = pack_bf16(acc[b][4 * a + 2] * inv, acc[b][4 * a + 3] * inv);
                *reinterpret_cast<uint2 *>(dst + 32 * b + 8 * a) = w;
            }
    }
}

}  // namespace

// Needs a positive scale (the max is taken over raw scores).  heads_per_chunk = 2: two heads of a
// KV head per wavefront (even group sizes); 1: one head, twice the query rows.
hipError_t launch_prefill_mfma32(const void *q, const void *k_cache, const void *v_cache,
                                 const int32_t *block_tables, const int32_t *context_lens,
                                 const int32_t *q_start, void *out, const PrefillParams &p, int total_q,
                                 hipStream_t stream) {
    if (prefill_wide(p, total_q)) return launch_prefill_wide(q, k_cache, v_cache, block_tables, context_lens, q_start, out, p, stream);
    const auto *qq = static_cast<const uint16_t *>(q);
    const auto *kk = static_cast<const uint16_t *>(k_cache);
    const auto *vv = static_cast<const uint16_t *>(v_cache);
    auto *oo = static_cast<uint16_t *>(out);
    const int heads = p.heads_per_chunk;
    const bool small = p.block_size < 8;
    const int query_tiles = prefill32_tiles(p);
    const int64_t grid = prefill32_grid(p);
    const bool split = prefill_split(p);
    // A grid that fits the device at once (two workgroups of four wavefronts per compute unit)
    // gets the second half of its query tiles in rising order (a few percent on one short request).
    // Chunks of several sequences: what a tile walks depends on its sequence's context, which only the device knows.
    // Up to 64 tiles are ranked there; grids that fit at once then put the shortest ranks beside the longest.  32 / 8
    // heads, 16-token blocks, us, in given order / ranked: four chunks of 512 rows, contexts of 2000 to 4000, 103.7 / 103.0
    // and 106.4 / 106.6; six of 600 rows, 8000: 372 / 328; three of 400, 7000: 137.6 / 129.8; five of 200, 6000: 110.3 / 94.9;
    // 64 / 8, four of 512, 4000: 234 / 205.  Recomputations, whose tiles are in order anyway, lose by it (three of 1000
    // tokens 31.0 / 36.4, sixteen of 220 22.6 / 29.3), so the workgroups rank only if some context of the batch is
    // four times as long as the longest chunk may be: under a 4096-token table these take 31.3 and 23.1.  A table
    // that reaches less far says so before the launch, and launches that fill no compute unit twice do without.
    const int64_t items = int64_t(p.num_seqs) * query_tiles;
    const int chunks = p.num_q_heads / heads;
    const int64_t chunk_reach = 4 * 64 * int64_t(p.max_query_tiles);
    const int rank_from = p.num_seqs > 1 && items <= 64 && grid > kNumCUs &&
                          int64_t(p.max_blocks_per_seq) * p.block_size >= chunk_reach ? int(chunk_reach) : 0;
    const int fold_at = grid <= 2 * kNumCUs ? (query_tiles + 1) / 2 : query_tiles;
    const int fold_ranked = grid <= 2 * kNumCUs ? std::max(1, std::min(int(items), kNumCUs / chunks)) : int(items);
    const int by_units = prefill_by_units(p) ? int(grid) : 0;
    const dim3 g{unsigned(grid)}, b(split ? 512 : 256);
    const int spread = chunk_spread(chunks, p.group / heads);
#define KVC_LAUNCH(SMALL, HEADS, SPLIT)                                                                        \
    pa_prefill_mfma32_kernel<SMALL, HEADS, SPLIT><<<g, b, 0, stream>>>(qq, kk, vv, block_tables, context_lens, \
                                                                       q_start, oo, p, query_tiles, fold_at, fold_ranked, rank_from, by_units, spread)
    if (small && heads == 2) KVC_LAUNCH(true, 2, false);
    else if (small) KVC_LAUNCH(true, 1, false);
    else if (heads == 2 && split) KVC_LAUNCH(false, 2, true);
    else if (heads == 2) KVC_LAUNCH(false, 2, false);
    else if (split) KVC_LAUNCH(false, 1, true);
    else KVC_LAUNCH(false, 1, false);
#undef KVC_LAUNCH
    return hipGetLastError();
}

}  // namespace kvc

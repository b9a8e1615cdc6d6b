// Paged decode attention of few rows on the matrix cores, one launch (gfx950, bf16, head_dim 128 or 64,
// block_size >= 4, group <= 16, at most 64 sequences and 128 (sequence, KV head) rows).
//
// Bound: latency.  A handful of sequences is a few MB of K and V, a few microseconds of streaming; what
// counts is the chain of dependent steps around it.  The balanced kernel, which deals the flattened tiles of
// the batch to single wavefronts, cuts such rows into many pieces (one sequence of 32000 tokens: 32 to 128 per
// row) and lets one wavefront merge them.  Here a workgroup of eight wavefronts takes one piece of one row:
//
//   P = smallest piece (tiles) for which all pieces of all rows fit the grid, at least the caller's
//       minimum and at most 64 pieces per row; row n has ceil(t_n / P) pieces, workgroup b takes piece
//       b / num_kv_heads of the flattened list for KV head b % num_kv_heads;
//   the wavefronts take the tiles of the piece in turn (first loads of all of them in flight at once) and
//       merge their softmax states through LDS;
//   a row of one piece is written at once.  Otherwise the workgroup stores its partial (device-scope
//       accesses), waits for the stores and adds 1 to the row's counter word; the one that counts the
//       last piece merges all of them, 512 threads wide, in slot order (so the bits of the result do not
//       depend on who came last), writes the row and resets the counter.  Nobody waits for anybody.
//
// Measured against the balanced kernel, launches back to back, 32 / 8 heads of 128: one sequence of 3217 tokens 15.0 ->
// 10.3 us (13 MB: 2.1 us of streaming; the exchange of pieces takes about 2.5 us), 8000 tokens 24.8 -> 12.7 us, 32000
// tokens 68 -> 25.9 us.
//
// Every wavefront works out the placement by itself: lane n holds the length of sequence n, sums and
// prefixes are a few steps inside the vector ALU, no LDS and no barrier before the first loads (by shuffles, stamps of one sequence
// of 3217 tokens, us from entry: placed 1.8, first loads 2.7, tiles consumed 4.0, wavefronts merged 5.4, stored 5.9,
// counted 6.9, pieces fetched and weighed 9.4, written 10.6).
#include <math.h>

#include <algorithm>

#include "kvc_internal.h"
#include "pa_mfma_tile.h"
#include "pa_partials.h"
#include "pa_quotient.h"

namespace kvc {

namespace {

using namespace mfma;

constexpr int kRowThreads = 512;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kStage = 64;        // tiles whose addresses are staged in LDS per wavefront at a time
constexpr int kMaxPieces = kMaxRowPieces;
// One sequence, 32 / 8 heads of 128, launches back to back: 19 tiles whole 7.3 us, in three pieces 8.4 us; 24 tiles
// 8.0 us against 8.4 us; 32 tiles 9.1 us against 8.5 us (head_dim 64: 16 tiles 7.0 / 8.1, 24 tiles 8.3 / 8.2).
constexpr int kWholeTiles = kRowWholeTiles;

using lanes::wave_max;
using lanes::wave_sum;

// Divisions by numbers the host knows, as multiplications: an integer division is some forty instructions, and here it would stand
// between two round trips to memory (32 / 8 heads of 128, us: 1 x 700 tokens 7.9 / 7.5, 1 x 3217 10.65 / 9.95, 4 x 2000 9.5 / 9.1).
struct Divisors {
    uint32_t room, slack;       // 2^32 / room and 2^32 / (room - num_seqs), rounded up
    int rooms;                  // room: pieces per KV head that the grid holds
    uint32_t kv_heads16;        // 2^16 / num_kv_heads, rounded up: exact below 2^16 / num_kv_heads
    uint32_t group16;           // 2^16 / group, rounded up: exact below 2^16 / group
    uint32_t vectors20;         // 2^20 / (group * HD / 4), rounded up: exact below 2^20 / that
};
// x / d, recip = 2^32 / d rounded up: the product is never too small and at most one too large (d = 1 does not fit)
__device__ inline int divided(int x, int d, uint32_t recip) {
    if (d == 1) return x;
    const int q = int(__umulhi(uint32_t(x), recip));
    return q - (q * d > x);
}

// Loads of one tile: entry(u) = pool index of its unit u (a tile is 1 << (kTokensLog2 - unit_log2) of them).  k_off / v_off:
// this lane's place inside a unit, in elements.  UNIFORM: units of 16 tokens and more, so that all lanes of a
// wavefront ask for the same unit and entry() returns a scalar: base addresses stay in scalar registers.
template <int HD, bool UNIFORM, class Entry>
__device__ inline void load_tile(typename Shape<HD>::Tile &t, Entry entry, const uint16_t *k_cache, const uint16_t *v_cache, int k_off,
                                 int v_off, size_t unit_elems, int unit_log2, int quad, int r) {
    constexpr int kSubs = Shape<HD>::kTokens / 16;
#pragma unroll
    for (int h = 0; h < kSubs; ++h) {
        const int in_unit = kSubs == 2 && unit_log2 == 5 ? 16 * h * HD : 0;  // second half of a 32-token unit
        const uint16_t *kp, *vp;
        if constexpr (UNIFORM) {
            const size_t base = size_t(entry((16 * h) >> unit_log2)) * unit_elems + in_unit;
            kp = k_cache + base + k_off;
            vp = v_cache + base + v_off;
        } else {
            kp = k_cache + size_t(entry((16 * h + r) >> unit_log2)) * unit_elems + in_unit + k_off;
            vp = v_cache + size_t(entry((16 * h + 4 * quad) >> unit_log2)) * unit_elems + in_unit + v_off;
        }
        if constexpr (HD == 128) {
#pragma unroll
            for (int j = 0; j < 4; ++j) t.k[j] = load16_stream(kp + 32 * j);
#pragma unroll
            for (int i = 0; i < 4; ++i) t.v[i] = load16_stream(vp + i * HD);
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) t.k[2 * h + j] = load16_stream(kp + 32 * j);
#pragma unroll
            for (int i = 0; i < 4; ++i) t.v[4 * h + i] = load8_stream(vp + i * HD);
        }
    }
}

template <int HD>
__device__ inline void consume_tile(typename Shape<HD>::State &st, typename Shape<HD>::Tile &t, const bf16x8 (&qb)[Shape<HD>::kQ],
                                    float scale_log2e, int left, int quad) {
    if constexpr (HD == 128) {
        bf16x8 ka[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) ka[j] = __builtin_bit_cast(bf16x8, t.k[j]);
        compute_tile(st, ka, t.v, qb, scale_log2e, left, quad);
    } else {
        compute_tile(st, t.k, t.v, qb, scale_log2e, left, quad);
    }
}

// `count` tiles in two register sets, no branch around the loads of the steady loop (see the balanced kernel)
template <class Tile, class Issue, class Compute>
__device__ inline void stream_tiles(int count, Issue issue, Compute compute) {
    Tile tA, tB;
    issue(tA);
    int it = 0;
    for (; it + 3 < count; it += 2) {
        issue(tB);
        compute(tA);
        issue(tA);
        compute(tB);
    }
    if (it + 3 == count) {
        issue(tB);
        compute(tA);
        issue(tA);
        compute(tB);
        compute(tA);
    } else if (it + 2 == count) {
        issue(tB);
        compute(tA);
        compute(tB);
    } else {
        compute(tA);
    }
}

// One workgroup's share: a piece of a row.
struct Piece {
    int n, kvh;         // sequence, KV head
    int ctx;            // context length of the sequence
    int tile0, tiles;   // first tile, number of tiles (0: nothing to do)
    int pieces;         // of the row
    int slot0;          // workgroup (partial slot) of the row's piece 0; the others follow num_kv_heads apart
};

template <int HD, int MODE>
__global__ __launch_bounds__(kRowThreads, 2) void pa_rows_mfma_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k_cache,
    const uint16_t *__restrict__ v_cache, const int32_t *__restrict__ block_tables,
    const int32_t *__restrict__ context_lens, uint16_t *__restrict__ out, Workspace ws,
    AttnParams p, Divisors by, int unit_log2, int units_per_block_log2, Schedule sched) {
    using TS = Shape<HD>;
    constexpr int kTokens = TS::kTokens, NV = TS::kVecs;
    constexpr int kMaxUnits = kTokens / 4;
    constexpr int kTileInts = kRowWaves * kStage * kMaxUnits;
    constexpr int kAccFloats = kRowWaves * 16 * HD;
    // tile addresses while streaming, softmax states of the wavefronts and what the merge exchanges afterwards
    __shared__ __attribute__((aligned(16))) float s_mem[kAccFloats > kTileInts ? kAccFloats : kTileInts];
    __shared__ float2 s_ml[kRowWaves][16];
    __shared__ int s_last;

    const int tid = threadIdx.x;
    const int wave = uniform(tid >> 6), lane = tid & 63;
    const int quad = lane >> 4, r = lane & 15;
    const int b = blockIdx.x;
    const int nseq = p.num_seqs, Hkv = p.num_kv_heads, G = p.group;
    const int U_log2 = TS::kTokensLog2 - unit_log2;
    int *const s_tile = reinterpret_cast<int *>(s_mem) + wave * kStage * kMaxUnits;

    // ---- placement
    Piece pc;
    bool empty_seq;  // sequence b has no context: its output row is zero
    if constexpr (MODE == kScheduled) {
        const int word = lane < kPlanInts ? sched.plans[size_t(b) * kPlanInts + lane] : 0;
        // as many tile addresses as the window or this workgroup's share of the schedule holds; entries past
        // the piece are never used
        const int *mine = sched.tiles + size_t(b) * sched.stride;
        for (int e = lane; e < (kStage << U_log2); e += 64) {
            const int at = ((wave + kRowWaves * (e >> U_log2)) << U_log2) + (e & ((1 << U_log2) - 1));
            if (at < sched.stride) s_tile[e] = mine[at];
        }
        auto w = [&](int i) { return __builtin_amdgcn_readlane(word, i); };
        pc = Piece{w(0), w(1), w(2), w(3), w(4), w(5), w(6)};
        empty_seq = w(7) != 0;
    } else {
        const int ctx = lane < nseq ? min(max(context_lens[lane], 0), p.max_context_len) : 0;
        const int t = (ctx + kTokens - 1) >> TS::kTokensLog2;
        const int total = wave_sum(t), longest = wave_max(t);
        empty_seq = b < nseq && __builtin_amdgcn_readlane(ctx, b < nseq ? b : 0) == 0;
        const int room = by.rooms;  // pieces per KV head the grid holds: at least 2 * num_seqs
        // rows of up to kWholeTiles tiles are not cut if the grid allows: the exchange costs more than it saves
        const int least = longest <= kWholeTiles ? longest : p.min_chunk_tiles;
        int lo = max(max(max(least, 1), divided(total + room - 1, room, by.room)), (longest + kMaxPieces - 1) / kMaxPieces);
        // sum ceil(t / P) <= total / P + num_seqs
        int hi = max(lo, divided(total + room - nseq - 1, room - nseq, by.slack));
        auto pieces_of = [&](int len) __attribute__((always_inline)) {  // no row has more than kMaxPieces
            return quotient(t + len - 1, len, __builtin_amdgcn_rcpf(float(len)));
        };
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (wave_sum(pieces_of(mid)) <= room) hi = mid; else lo = mid + 1;
        }
        const int P = lo;
        const int pieces = pieces_of(P);
        const int incl = lanes::prefix_sum(pieces);
        const int excl = incl - pieces;
        const int idx = int((uint32_t(b) * by.kv_heads16) >> 16);
        pc = Piece{0, b - idx * Hkv, 0, 0, 0, 0, 0};
        const uint64_t at = __ballot(pieces > 0 && excl <= idx && idx < incl);
        if (at) {
            pc.n = __builtin_ctzll(at);
            pc.ctx = __builtin_amdgcn_readlane(ctx, pc.n);
            pc.pieces = __builtin_amdgcn_readlane(pieces, pc.n);
            const int first = __builtin_amdgcn_readlane(excl, pc.n);
            pc.slot0 = first * Hkv + pc.kvh;
            pc.tile0 = (idx - first) * P;
            pc.tiles = min(P, __builtin_amdgcn_readlane(t, pc.n) - pc.tile0);
        }
    }
    if constexpr (MODE == kBuild) {
        const int words[kPlanInts] = {pc.n, pc.kvh, pc.ctx, pc.tile0, pc.tiles, pc.pieces, pc.slot0, empty_seq, 0, 0, 0, 0, 0, 0, 0, 0};
        int mine = 0;
#pragma unroll
        for (int i = 0; i < kPlanInts; ++i) mine = lane == i ? words[i] : mine;
        if (wave == 0 && lane < kPlanInts) sched.plans[size_t(b) * kPlanInts + lane] = mine;
    } else if (empty_seq) {
        uint4 *row = reinterpret_cast<uint4 *>(out + size_t(b) * p.num_q_heads * HD);
        for (int i = tid; i < p.num_q_heads * (HD / 8); i += kRowThreads) row[i] = uint4{0u, 0u, 0u, 0u};
    }
    if (pc.tiles == 0) return;  // uniform over the workgroup

    // Pool index of unit u of the piece (see the balanced kernel: a unit is the part of a tile inside one
    // block); units past the end of the context repeat the last valid one, loaded and masked.
    const int unit_tokens = 1 << unit_log2;
    const int last_unit = ((pc.ctx + unit_tokens - 1) >> unit_log2) - 1;
    auto unit_index = [&](int u) __attribute__((always_inline)) {
        const int unit = min((pc.tile0 << U_log2) + u, last_unit);
        const int blk = block_tables[size_t(pc.n) * p.max_blocks_per_seq + (unit >> units_per_block_log2)];
        return ((blk * Hkv + pc.kvh) << units_per_block_log2) + (unit & ((1 << units_per_block_log2) - 1));
    };
    if constexpr (MODE == kBuild) {
        int *mine = sched.tiles + size_t(b) * sched.stride;
        for (int u = tid; u < (pc.tiles << U_log2); u += kRowThreads) mine[u] = unit_index(u);
        return;
    }

    // ---- this wavefront's tiles: wave, wave + 8, ... of the piece
    const int count = pc.tiles > wave ? (pc.tiles - wave + kRowWaves - 1) / kRowWaves : 0;
    auto stage = [&](int from, int first) __attribute__((always_inline)) {
        const int entries = min(kStage, count - from) << U_log2;
        for (int e = first; e < entries; e += 64) {
            const int u = ((wave + kRowWaves * (from + (e >> U_log2))) << U_log2) + (e & ((1 << U_log2) - 1));
            if constexpr (MODE == kScheduled) s_tile[e] = sched.tiles[size_t(b) * sched.stride + u];
            else s_tile[e] = unit_index(u);
        }
    };
    typename TS::State st;
    st.reset();
    if (count > 0) {
        bf16x8 qb[TS::kQ];
        // the first table entries are requested before Q and the rest of the window after it: the wait for the
        // entries then does not include Q
        int entry = 0;
        if constexpr (MODE == kDirect) entry = unit_index(((wave + kRowWaves * (lane >> U_log2)) << U_log2) + (lane & ((1 << U_log2) - 1)));
        load_q_operand(qb, q + (size_t(pc.n) * p.num_q_heads + pc.kvh * G + (r < G ? r : 0)) * HD, quad, r < G);
        if constexpr (MODE == kDirect) {
            s_tile[lane] = entry;
            stage(0, lane + 64);
        }

        const size_t unit_elems = size_t(unit_tokens) * HD;
        const int k_off = (r & (unit_tokens - 1)) * HD + 8 * quad, v_off = ((4 * quad) & (unit_tokens - 1)) * HD + HD / 16 * r;
        int ki = 0, staged = 0;
        auto issue = [&](typename TS::Tile &t) __attribute__((always_inline)) {
            if (ki - staged == kStage) {  // long pieces only
                stage(ki, lane);
                staged = ki;
            }
            const int *e = s_tile + ((ki - staged) << U_log2);
            load_tile<HD, false>(t, [&](int u) { return e[u]; }, k_cache, v_cache, k_off, v_off, unit_elems, unit_log2, quad, r);
            ++ki;
        };
        int left = pc.ctx - (pc.tile0 + wave) * kTokens;  // tokens of the context from the next tile on
        auto compute = [&](typename TS::Tile &t) __attribute__((always_inline)) {
            consume_tile<HD>(st, t, qb, p.scale_log2e, left, quad);
            left -= kRowWaves * kTokens;
        };
        stream_tiles<typename TS::Tile>(count, issue, compute);
        st.finish();
    }

    // ---- the wavefronts' states meet in LDS.  A state is nv4 = G * HD / 4 vectors in slot layout; thread f
    // (< nv4 <= 512) owns vector f: head f % G, dims HD/4 * quad + 4 v with 4 v + quad = f / G.
    __syncthreads();  // the tile addresses are no longer needed
    if (r < G) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
            *reinterpret_cast<float4 *>(s_mem + wave * G * HD + slot_vec<HD>(0, G, v, quad, r) / 4) = acc_vec(st, v);
        if (quad == 0) s_ml[wave][r] = float2{st.m, st.l};
    }
    __syncthreads();
    const int nv4 = G * HD / 4;
    const int share = int((uint32_t(tid) * by.vectors20) >> 20), f = tid - share * nv4;  // share: which pieces a thread merges in the second step
    const int vq = int((uint32_t(f) * by.group16) >> 16), head = f - vq * G;
    uint16_t *dst = out + (size_t(pc.n) * p.num_q_heads + pc.kvh * G + head) * HD + HD / 4 * (vq & 3) + 4 * (vq >> 2);
    auto write_out = [&](const float4 &a, float L) __attribute__((always_inline)) {
        const float inv = 1.0f / L;
        *reinterpret_cast<uint2 *>(dst) = uint2{pack_bf16(a.x * inv, a.y * inv), pack_bf16(a.z * inv, a.w * inv)};
    };
    auto add = [](float4 &a, float w, const float4 &x) __attribute__((always_inline)) {
        a.x = fmaf(w, x.x, a.x);
        a.y = fmaf(w, x.y, a.y);
        a.z = fmaf(w, x.z, a.z);
        a.w = fmaf(w, x.w, a.w);
    };
    float M = -INFINITY, L = 0.f;
    float4 a = {0.f, 0.f, 0.f, 0.f};
    if (tid < nv4) {
#pragma unroll
        for (int w = 0; w < kRowWaves; ++w) M = fmaxf(M, s_ml[w][head].x);  // finite: wavefront 0 has a tile
#pragma unroll
        for (int w = 0; w < kRowWaves; ++w) {
            if (w >= pc.tiles) break;  // wavefronts without a tile hold nothing
            const float2 ml = s_ml[w][head];
            const float wgt = __builtin_amdgcn_exp2f(ml.x - M);
            L = fmaf(wgt, ml.y, L);
            add(a, wgt, *reinterpret_cast<const float4 *>(s_mem + w * G * HD + 4 * f));
        }
        if (pc.pieces == 1) write_out(a, L);
    }
    if (pc.pieces == 1) return;

    // ---- publish the piece; the last workgroup to arrive at the row merges all of them
    const uint32_t slots = gridDim.x;
    const __amdgpu_buffer_rsrc_t acc_buf = raw_buffer(ws.acc, slots * uint32_t(G * HD) * 4u);
    const __amdgpu_buffer_rsrc_t ml_buf = raw_buffer(ws.ml, slots * uint32_t(G) * 8u);
    if (tid < nv4) {
        store4_device_scope(acc_buf, (uint32_t(b) * nv4 + f) * 16u, a.x, a.y, a.z, a.w);
        if (vq == 0) store2_device_scope(ml_buf, slot_ml(b, G, head), M, L);
    }
    // the count may become visible only after the partial: every wavefront waits for its own stores, then all meet
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int32_t *const counter = ws.cnt + pc.n * Hkv + pc.kvh;
    if (tid == 0) s_last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == pc.pieces - 1;
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");  // the fetches stay behind the count
    if (tid == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // thread (share, f) takes the pieces share, share + shares, ... of vector f; the shares of a vector meet in LDS
    const int shares = int((uint32_t(kRowThreads) * by.vectors20) >> 20);
    const bool active = share < shares;
    float *const s_w = s_mem;                                                   // [64 pieces][G] weights
    float4 *const s_part = reinterpret_cast<float4 *>(s_mem + kMaxPieces * 16);  // [shares][nv4]
    constexpr int kBatch = 8;
    float4 x[kBatch];
    auto fetch = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int i = i0 + u * shares;
            if (active && i < pc.pieces) x[u] = load4_device_scope(acc_buf, (uint32_t(pc.slot0 + i * Hkv) * nv4 + f) * 16u);
        }
    };
    // wavefront w weighs the pieces for heads w and w + 8, lane i holds piece i
    float2 pml[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        pml[j] = float2{-INFINITY, 0.f};
        if (wave + j * kRowWaves < G && lane < pc.pieces)
            pml[j] = load2_device_scope(ml_buf, slot_ml(pc.slot0 + lane * Hkv, G, wave + j * kRowWaves));
    }
    fetch(share);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (wave + j * kRowWaves < G) {  // wavefront-uniform
            const float top = wave_max(pml[j].x);
            const float wgt = lane < pc.pieces ? __builtin_amdgcn_exp2f(pml[j].x - top) : 0.f;
            const float sum = wave_sum(wgt * pml[j].y);
            s_w[lane * G + wave + j * kRowWaves] = wgt;
            if (lane == 0) s_ml[0][wave + j * kRowWaves].y = sum;
        }
    }
    __syncthreads();
    a = float4{0.f, 0.f, 0.f, 0.f};
    for (int i0 = share; i0 < pc.pieces; i0 += kBatch * shares) {
        if (i0 != share) fetch(i0);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int i = i0 + u * shares;
            if (active && i < pc.pieces) add(a, s_w[i * G + head], x[u]);
        }
    }
    if (shares > 1) {
        if (active) s_part[share * nv4 + f] = a;
        __syncthreads();
        if (tid < nv4)
            for (int s = 1; s < shares; ++s) add(a, 1.f, s_part[s * nv4 + f]);
    }
    if (tid < nv4) write_out(a, s_ml[0][head].y);
}

// Short contexts, any number of rows: a workgroup of four wavefronts takes a whole row, no placement, no exchange.
// Block-table entries and Q are requested together with the context length (entries past the context are read
// but never used), so the first K and V bytes are two memory round trips away.  20 sequences of 100 tokens, 32 / 8
// heads of 128: 4.9 us (9.4 us in ranges); 64 of 300: 14.5 us = 5.4 TB/s (19.8 us).  Two wavefronts per SIMD at
// head_dim 128: with three the registers spill (16.3 us), at head_dim 64 three fit.
constexpr int kWholeWaves = 4;

template <int HD, int MODE, bool UNIFORM>
__global__ __launch_bounds__(64 * kWholeWaves, HD == 128 ? 2 : 3) void pa_whole_mfma_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k_cache,
    const uint16_t *__restrict__ v_cache, const int32_t *__restrict__ block_tables,
    const int32_t *__restrict__ context_lens, uint16_t *__restrict__ out, AttnParams p, uint32_t group16, int unit_log2,
    int units_per_block_log2, Schedule sched) {
    using TS = Shape<HD>;
    constexpr int kTokens = TS::kTokens, NV = TS::kVecs;
    __shared__ __attribute__((aligned(16))) float s_acc[kWholeWaves * 16 * HD];
    __shared__ float2 s_ml[kWholeWaves][16];
    __shared__ int s_tiles[kWholeWaves][64];  // pool indices of the units of a wavefront's tiles: at most 64 (checked by the host)

    const int tid = threadIdx.x;
    const int wave = uniform(tid >> 6), lane = tid & 63;
    const int quad = lane >> 4, r = lane & 15;
    const int kvh = blockIdx.x, n = blockIdx.y;
    const int Hkv = p.num_kv_heads, G = p.group;
    const int U_log2 = TS::kTokensLog2 - unit_log2;
    const size_t row = size_t(n) * Hkv + kvh;

    // unit of this lane's entry: the wavefront takes tiles wave, wave + 4, ... of the row
    const int unit = ((wave + kWholeWaves * (lane >> U_log2)) << U_log2) + (lane & ((1 << U_log2) - 1));
    int ctx, entry;
    if constexpr (MODE == kScheduled) {
        ctx = sched.ctx[n];
        entry = sched.tiles[row * sched.stride + min(unit, sched.stride - 1)];
    } else {
        ctx = min(max(context_lens[n], 0), p.max_context_len);
        const int blk = block_tables[size_t(n) * p.max_blocks_per_seq + min(unit >> units_per_block_log2, p.max_blocks_per_seq - 1)];
        entry = int(((unsigned(blk) * unsigned(Hkv) + unsigned(kvh)) << units_per_block_log2) +
                    unsigned(unit & ((1 << units_per_block_log2) - 1)));
    }
    const int tiles = (ctx + kTokens - 1) >> TS::kTokensLog2;
    if constexpr (MODE == kBuild) {
        if (tid == 0 && kvh == 0) sched.ctx[n] = ctx;
        if (unit < sched.stride) sched.tiles[row * sched.stride + unit] = entry;
        return;
    }
    bf16x8 qb[TS::kQ];
    load_q_operand(qb, q + (size_t(n) * p.num_q_heads + kvh * G + (r < G ? r : 0)) * HD, quad, r < G);
    uint16_t *const dst_row = out + (size_t(n) * p.num_q_heads + kvh * G) * HD;
    if (tiles == 0) {
        for (int i = tid; i < G * (HD / 8); i += 64 * kWholeWaves) reinterpret_cast<uint4 *>(dst_row)[i] = uint4{0u, 0u, 0u, 0u};
        return;
    }
    if constexpr (!UNIFORM) s_tiles[wave][lane] = entry;

    typename TS::State st;
    st.reset();
    const int count = tiles > wave ? (tiles - wave + kWholeWaves - 1) / kWholeWaves : 0;
    if (count > 0) {
        const int unit_tokens = 1 << unit_log2;
        const int last_unit = ((ctx + unit_tokens - 1) >> unit_log2) - 1;
        const size_t unit_elems = size_t(unit_tokens) * HD;
        const int k_off = (r & (unit_tokens - 1)) * HD + 8 * quad, v_off = ((4 * quad) & (unit_tokens - 1)) * HD + HD / 16 * r;
        int ki = 0;
        auto issue = [&](typename TS::Tile &t) __attribute__((always_inline)) {
            const int last = last_unit - ((wave + kWholeWaves * ki) << U_log2);  // units of the tile past it repeat it
            const int first = ki << U_log2;
            load_tile<HD, UNIFORM>(t, [&](int u) __attribute__((always_inline)) {
                if constexpr (UNIFORM) return __builtin_amdgcn_readlane(entry, first + min(u, last));
                else return s_tiles[wave][first + min(u, last)];
            }, k_cache, v_cache, k_off, v_off, unit_elems, unit_log2, quad, r);
            ++ki;
        };
        int left = ctx - wave * kTokens;
        auto compute = [&](typename TS::Tile &t) __attribute__((always_inline)) {
            consume_tile<HD>(st, t, qb, p.scale_log2e, left, quad);
            left -= kWholeWaves * kTokens;
        };
        stream_tiles<typename TS::Tile>(count, issue, compute);
        st.finish();
    }
    if (r < G) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
            *reinterpret_cast<float4 *>(s_acc + wave * G * HD + slot_vec<HD>(0, G, v, quad, r) / 4) = acc_vec(st, v);
        if (quad == 0) s_ml[wave][r] = float2{st.m, st.l};
    }
    __syncthreads();
    const int nv4 = G * HD / 4;
    for (int f = tid; f < nv4; f += 64 * kWholeWaves) {
        const int vq = int((uint32_t(f) * group16) >> 16), head = f - vq * G;  // as in the kernel above
        float M = -INFINITY, L = 0.f;
        float4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWholeWaves; ++w) M = fmaxf(M, s_ml[w][head].x);
#pragma unroll
        for (int w = 0; w < kWholeWaves; ++w) {
            if (w >= tiles) break;
            const float2 ml = s_ml[w][head];
            const float wgt = __builtin_amdgcn_exp2f(ml.x - M);
            const float4 x = *reinterpret_cast<const float4 *>(s_acc + w * G * HD + 4 * f);
            L = fmaf(wgt, ml.y, L);
            a.x = fmaf(wgt, x.x, a.x);
            a.y = fmaf(wgt, x.y, a.y);
            a.z = fmaf(wgt, x.z, a.z);
            a.w = fmaf(wgt, x.w, a.w);
        }
        const float inv = 1.0f / L;
        *reinterpret_cast<uint2 *>(dst_row + head * HD + HD / 4 * (vq & 3) + 4 * (vq >> 2)) =
            uint2{pack_bf16(a.x * inv, a.y * inv), pack_bf16(a.z * inv, a.w * inv)};
    }
}

}  // namespace

hipError_t launch_rows_mfma(const void *q, const void *k_cache, const void *v_cache,
                            const int32_t *block_tables, const int32_t *context_lens,
                            void *out, Workspace ws, const AttnParams &p, int head_dim, int grid,
                            int mode, Schedule sched, hipStream_t stream) {
    const int tile_log2 = head_dim == 128 ? Shape<128>::kTokensLog2 : Shape<64>::kTokensLog2;
    const int unit_log2 = p.block_size_log2 < tile_log2 ? p.block_size_log2 : tile_log2;
#define KVC_LAUNCH_ROWS(HD, MODE)                                                                                 \
    pa_rows_mfma_kernel<HD, MODE><<<dim3(grid), dim3(kRowThreads), 0, stream>>>(                                  \
        static_cast<const uint16_t *>(q), static_cast<const uint16_t *>(k_cache), static_cast<const uint16_t *>(v_cache), \
        block_tables, context_lens, static_cast<uint16_t *>(out), ws, p, by, unit_log2, p.block_size_log2 - unit_log2, sched)
    auto recip = [](uint64_t one, int d) { return uint32_t(std::min<uint64_t>((one + d - 1) / d, UINT32_MAX)); };  // d = 1: not used
    const int room = grid / p.num_kv_heads;
    const Divisors by{recip(uint64_t(1) << 32, room), recip(uint64_t(1) << 32, room - p.num_seqs), room, recip(1 << 16, p.num_kv_heads),
                      recip(1 << 16, p.group), recip(1 << 20, p.group * head_dim / 4)};
    if (head_dim == 64) KVC_LAUNCH_ROWS(64, kDirect);  // stateless calls only
    else if (mode == kDirect) KVC_LAUNCH_ROWS(128, kDirect);
    else if (mode == kBuild) KVC_LAUNCH_ROWS(128, kBuild);
    else KVC_LAUNCH_ROWS(128, kScheduled);
#undef KVC_LAUNCH_ROWS
    return hipGetLastError();
}

hipError_t launch_whole_mfma(const void *q, const void *k_cache, const void *v_cache,
                             const int32_t *block_tables, const int32_t *context_lens,
                             void *out, Workspace, const AttnParams &p, int head_dim, int,
                             int mode, Schedule sched, hipStream_t stream) {
    const int tile_log2 = head_dim == 128 ? Shape<128>::kTokensLog2 : Shape<64>::kTokensLog2;
    const int unit_log2 = p.block_size_log2 < tile_log2 ? p.block_size_log2 : tile_log2;
#define KVC_LAUNCH_WHOLE(HD, MODE, UNIFORM)                                                                                \
    pa_whole_mfma_kernel<HD, MODE, UNIFORM><<<dim3(p.num_kv_heads, p.num_seqs), dim3(64 * kWholeWaves), 0, stream>>>( \
        static_cast<const uint16_t *>(q), static_cast<const uint16_t *>(k_cache), static_cast<const uint16_t *>(v_cache), \
        block_tables, context_lens, static_cast<uint16_t *>(out), p, uint32_t(((1 << 16) + p.group - 1) / p.group), unit_log2, \
        p.block_size_log2 - unit_log2, sched)
    const bool uniform_units = p.block_size >= 16;
    if (mode == kBuild) KVC_LAUNCH_WHOLE(128, kBuild, false);
    else if (head_dim == 64 && uniform_units) KVC_LAUNCH_WHOLE(64, kDirect, true);  // stateless calls only
    else if (head_dim == 64) KVC_LAUNCH_WHOLE(64, kDirect, false);
    else if (mode == kDirect && uniform_units) KVC_LAUNCH_WHOLE(128, kDirect, true);
    else if (mode == kDirect) KVC_LAUNCH_WHOLE(128, kDirect, false);
    else if (uniform_units) KVC_LAUNCH_WHOLE(128, kScheduled, true);
    else KVC_LAUNCH_WHOLE(128, kScheduled, false);
#undef KVC_LAUNCH_WHOLE
    return hipGetLastError();
}

}  // namespace kvc

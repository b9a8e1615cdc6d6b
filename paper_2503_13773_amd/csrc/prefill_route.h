// What a prefill call on 32x32 tiles launches: plain C++, so that tests on the host ask the library's own rules.
#pragma once

#include <stdint.h>

namespace kvc {

constexpr int kNumCUs = 256;        // MI355X

// Causal multi-query (prefill / recompute) attention.
struct PrefillParams {
    int num_seqs;
    int num_q_heads;
    int num_kv_heads;
    int group;                 // num_q_heads / num_kv_heads
    int heads_per_chunk;       // query heads one wavefront carries (1 or 2; divides group)
    int block_size;
    int block_size_log2;
    int tiles_per_block_log2;  // log2(block_size / 16); 0 for block sizes below 16
    int max_blocks_per_seq;
    int max_query_tiles;       // ceil(max_query_len / 64)
    float scale_log2e;
};

// Whether 32x32 tiles serve a call at head_dim 128: their max is taken over raw scores, so the scale has to be positive, and
// they hold the bytes of a block in 32 bits.  Others go to the kernel of 16x16 tiles.
inline bool prefill_tiles32(const PrefillParams &p) {
    return p.scale_log2e > 0.0f && int64_t(p.block_size) * p.num_kv_heads * 256 < (int64_t(1) << 32);
}

// Query tiles of the longest sequence and workgroups of a launch on 32-column wavefronts: 64 rows of two heads, or 128 of one.
inline int prefill32_tiles(const PrefillParams &p) {
    const int rows64 = 2 / p.heads_per_chunk;
    return (p.max_query_tiles + rows64 - 1) / rows64;
}
inline int64_t prefill32_grid(const PrefillParams &p) {
    return int64_t(p.num_q_heads / p.heads_per_chunk) * p.num_seqs * prefill32_tiles(p);
}

// Steps (32 tokens) from which the second group of a split workgroup takes a share.  The last 64 rows of one request, 32 / 8
// heads, us, whole / split: 800 tokens 15.2 / 16.7, 1200 20.0 / 20.7, 1500 (47 steps) 23.2 / 23.8, 1600 (50 steps, equal
// shares) 24.1 / 23.8, 1900 28.2 / 27.3, 2100 30.5 / 28.8; 200 rows of two 1500 23.8 / 24.2, 1600 24.7 / 24.4, 1700 25.6 / 25.8, 1800
// 26.3 / 26.0; 4 / 4 heads, 64 rows 1500 20.6 / 21.1, 1600 21.1 / 21.0, 2100 26.3 / 25.7.
constexpr int kMinSplitSteps = 50;

// Whether workgroups are split: at most one per compute unit (up to two the finer grain of plain ones wins: one request of 2048
// tokens 40.0 us plain, 49.2 split; four chunks of 512 rows at 4000 tokens 106.6 / 118.2), where the block table
// reaches far enough for a share (the second group costs a short context nothing measurable then: 642 tokens 13.8 us
// either way) and holds blocks of 8 tokens or more.
inline bool prefill_split(const PrefillParams &p) {
    return p.block_size >= 8 && prefill32_grid(p) <= kNumCUs &&
           int64_t(p.max_blocks_per_seq) * p.block_size > (kMinSplitSteps - 1) * 32;
}

// Workgroups of odd groups, one query head each: where a launch has enough of them, the `group` workgroups of a unit
// (KV head, sequence, query tile) are eight blocks apart, which the device hands to one XCD, so that one L2 fetches the
// unit's K and V rows instead of up to `group` of them.  With fewer than eight KV heads the tiles of a sequence differ too much from
// XCD to XCD (7 / 1 heads, eight of 1500 tokens, 35.6 us in plain order, 42.9 by units), and so do those of short launches
// (50 / 10, one of 1200, 500 workgroups, 29.0 / 30.9; four of 500, 800 workgroups, 28.7 / 29.8).  us, plain order / by units:
// 40 / 8 heads, two chunks of 3600 rows at 12000 tokens 1303 / 1111, four of 4096 620 / 540, one of 4096 165.7 / 165.3; 56 / 8,
// four of 4096 915 / 757; 50 / 10, four of 4096 823 / 702; 48 / 16 775 / 679.  One head per KV head has nothing to share.
inline bool prefill_by_units(const PrefillParams &p) {
    return p.heads_per_chunk == 1 && p.group > 1 && p.num_kv_heads >= 8 && prefill32_grid(p) > 4 * kNumCUs;
}

// The place of workgroup `block` of `blocks` (a multiple of group * kv_heads) by units.  A unit's number rises with the KV
// head first, then with `index` (sequence and order of the tile).  KV heads in multiples of eight stay on their XCDs;
// others would give the first XCD the longest tile of every eight, so that every other run of units goes backwards.
struct HeadPlace {
    int kv_head, head, index;
};
constexpr HeadPlace head_place(int block, int blocks, int group, int kv_heads) {
    const int run = 8 * group, whole = blocks / run * run;
    int unit = 0, member = 0;
    if (block < whole) {
        const int r = block % run, xcd = r & 7, turn = block / run;
        unit = 8 * turn + ((turn & 1) != 0 && (kv_heads & 7) != 0 ? 7 - xcd : xcd);
        member = r >> 3;
    } else {  // fewer than eight units are left
        const int units = (blocks - whole) / group;
        unit = whole / group + (block - whole) % units;
        member = (block - whole) / units;
    }
    const int kv_head = unit % kv_heads;
    return {kv_head, kv_head * group + member, unit / kv_heads};
}

// The head chunk (the heads of one workgroup) of workgroup `b` among the `chunks` of a query tile; `sharing` of them attend
// over one KV head.  The device hands neighbouring workgroups to its 8 XCDs in turn: chunks in multiples of eight are dealt
// out so that those of a KV head are neighbours on one XCD, whose L2 then fetches its rows once, and every XCD
// keeps its share of each tile.  32 / 8 heads, us, in plain order / so: two of 4096 216.7 / 210.2, six of 2000 148.5 / 145.6,
// of 400 19.7 / 19.0, four chunks of 512 rows at 4000 106.6 / 105.8; heads of 64, four of 1999 107.8 / 106.0.  Heads that share
// nothing gain nothing (32 / 32, two of 3000 122.2 / 123.0).
// The host says how many chunks an XCD holds (0: plain order): worked out in the kernel that took 0.05 us of a call at head_dim 128 (15 / 5
// heads, two chunks of 5 rows, 6.89 us without, 6.99 with), also where nothing is dealt out.
constexpr int chunk_spread(int chunks, int sharing) { return sharing > 1 && (chunks & 7) == 0 ? chunks >> 3 : 0; }
constexpr int chunk_at(int b, int spread) { return spread > 0 ? (b & 7) * spread + (b >> 3) : b; }

// Whether the kernel of 64-column wavefronts (paged_attention_prefill_wide.hip) takes a call: groups that 4 divides, four
// query heads and 64 rows per workgroup, one workgroup per compute unit.  It reads half the LDS operands per score, but nothing hides a
// tile's start and end (15000 cycles against 1390 per 32 tokens), and with one workgroup per compute unit the rounds in which
// the tiles go round the device show.  us, 32 columns / 64 columns, in brackets the workgroups per compute unit:
//   One request, or several of nearly equal rows (on average 97 % of the longest).  Up to 1.6 rounds tiles stand alone; between 1.65 and 2 a long and a short one share a compute unit
//     evenly; past 2 they do not; from 3.4 on there are enough of them.  32 / 8 heads: 3000 tokens [1.5] 75.9 / 77.0, 3500
//     [1.7] 98.9 / 93.6, 4096 [2.0] 126.1 / 121.2, 4600 [2.3] 159.2 / 161.2, 5000 [2.5] 186.0 / 190.9, 6500 [3.2] 299.5 / 299.9,
//     7300 [3.6] 374.8 / 367.4, 12000 [5.9] 980 / 960, 16384 [8] 1803 / 1768; 64 / 8: 2048 [2.0] 74.3 / 72.0, 2500 [2.5]
//     108.7 / 112.2, 3000 [2.9] 148.9 / 151.1, 3600 [3.6] 208.2 / 205.6, 8000 [7.8] 882 / 864; 16 / 2: 6500 [1.6] 161.1 / 161.6, 7300
//     [1.8] 199.6 / 188.7, 10500 [2.6] 389.5 / 394.7, 16384 [4] 904 / 876; 48 / 4: 3500 [2.6] 142.2 / 147.9, 4600 [3.4] 233.6 /
//     229.8; 12 / 1: 11000 [2.02] 342 / 326.  Of tiles of fewer than 32 (64 rows each) the starts and ends are too large a
//     share: 128 / 16, 1750 (28 tiles) [3.5] 111.6 / 112.8, 2048 (32) [4] 146.0 / 142.7.  Equal requests, 32 / 8: two of 4096 [4.0]
//     246.8 / 238.3, four of 4096 [8] 489 / 472; 64 / 8, two of 4096 [8] 489 / 470; 16 / 2, two of 3600 [1.8] 103.5 / 99.8, of 5000
//     [2.5] 186.7 / 191.3, three of 3600 [2.6] 150.0 / 153.7, eight of 5000 [9.8] 718 / 696; 8 / 2, six of 5000 [3.7] 273.8 /
//     267.5; with an average of 95 % 16 / 2, three of 5000, and 32 / 8, two of 5000, lose 4 and 2 %.  Below 55
//     tiles only groups of 8 and 16: equal rows can be chunks of unequal contexts, which only the device knows (32 / 8, two
//     chunks of 2048 at 16000 [2] 697 / 715).
//   Several of unequal rows.  They leave an uneven end more often, so that it takes seven rounds, and 55 tiles in the longest, or 32 with 64
//     heads and more, whose workgroups of 32 columns spread a KV head over more XCDs.  32 / 8: six of 3600 [8.3] 437 / 417, of
//     2048 [4.7] 157.6 / 161.5, eight of 2048 [6.6] 229.6 / 252.9, five of 4096 [8.3] 473 / 468; 64 / 8: four of 2048 [7.3] 259.6 /
//     254.5, of 1500 [5.3] 150.8 / 153.9, eight of 2048 [13] 487 / 446; 48 / 4, six of 3600 [12] 665 / 619.  Where heads times
//     requests come to no more than 128 there is nothing in it, or less: 32 / 8, four of 4900 [8.7] 622 / 628, two of 5000 [4.3]
//     325 / 337; 64 / 8, two of 4096 [7] 413 / 434; 16 / 2, two of 6500 [2.8] 262 / 290, each on four XCDs of its own, the longer one
//     last.  With two requests of eight heads it is the workgroups of 32 columns that place them so: 8 / 2, two of 8000 [1.7]
//     231 / 201, of 13000 [2.8] 579 / 537.
//   Blocks of fewer than 8 tokens cost the workgroups of 32 columns more (an address per row and load, registers that spill),
//     and the lines lie lower: three rounds for one request, 2.8 and 45 tiles for several, except those whose requests
//     get XCDs of their own and two of 64 heads and more.  Blocks of 4: 32 / 8, one of 5000 [2.5] 201.2 / 201.7, of 6500 [3.2]
//     323.9 / 313.6, three of 4096 [5.3] 332 / 311, six of 3200 [7.3] 375 / 342, two of 3200 [2.75] 148.1 / 151.2, eight of 2600 (41
//     tiles) [8.4] 378 / 394; 16 / 2, six of 3200 [3.7] 181.7 / 167.7, two of 6500 281 / 308; 64 / 8, two of 3600 [6.2] 361 / 370,
//     three of 2600 [6.7] 299 / 273.
// Batches with a few long requests among short ones (a mean below half the longest) stay on 32 columns.
inline bool prefill_wide(const PrefillParams &p, int64_t total_q) {
    if (p.group % 4 != 0 || total_q < int64_t(p.num_seqs) * p.max_query_tiles * 32) return false;
    const int chunks = p.num_q_heads / 4;
    const int64_t rounds100 = 100 * chunks * ((total_q + 63) / 64) / kNumCUs;
    const bool small = p.block_size < 8, many_heads = chunks >= 16;
    if (p.num_seqs == 1 || 100 * total_q >= 97 * int64_t(p.num_seqs) * p.max_query_tiles * 64)
        return p.max_query_tiles >= (p.num_seqs == 1 || p.group % 8 == 0 ? 32 : 55) &&
               ((rounds100 >= 165 && rounds100 <= 205) || rounds100 >= (small ? 300 : 340));
    if (p.num_seqs == 2 && chunks == 2) return p.max_query_tiles >= 55 && rounds100 >= 165;
    const int64_t tile_row = int64_t(chunks) * p.num_seqs;  // workgroups of one query tile of all requests
    if (small)
        return rounds100 >= (p.num_seqs == 2 && many_heads ? 700 : 280) && tile_row > 8 && p.max_query_tiles >= (many_heads ? 32 : 45);
    return rounds100 >= 700 && tile_row > 32 && p.max_query_tiles >= (many_heads ? 32 : 55);
}

}  // namespace kvc

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

// Workgroups of odd groups, one query head each: where a launch has enough of them, the `group` workgroups of a unit
// (KV head, sequence, query tile) are eight blocks apart, which the device hands to one XCD, so that one L2 fetches the
// unit's K and V rows instead of up to `group` of them.  With fewer than eight KV heads the tiles of a sequence differ too much from
// XCD to XCD (7 / 1 heads, eight of 1500 tokens, 35.6 us in plain order, 42.9 by units), and so do those of short launches
// (50 / 10, one of 1200, 500 workgroups, 29.0 / 30.9; four of 500, 800 workgroups, 28.7 / 29.8).  us, plain order / by units:
// 40 / 8 heads, two chunks of 3600 rows at 12000 tokens 1303 / 1111, four of 4096 620 / 540, one of 4096 165.7 / 165.3; 56 / 8,
// four of 4096 915 / 757; 50 / 10, four of 4096 823 / 702; 48 / 16 775 / 679.  One head per KV head has nothing to share.
inline bool prefill_by_units(const PrefillParams &p, int64_t grid) {
    return p.heads_per_chunk == 1 && p.group > 1 && p.num_kv_heads >= 8 && grid > 4 * kNumCUs;
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

}  // namespace kvc

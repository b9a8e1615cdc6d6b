// kv_cache_append: scatter one new token's K and V per sequence into the block-allocated
// cache (gfx950).  The write that precedes the decode attention of every iteration: each
// running request appends one token to the next free slot of its last block (block-based
// allocation: paper Section 1; iteration structure: Section 3.1).
//
// One 16-byte word per lane for K and one for V; a (sequence, kv head) row is row_bytes / 16
// consecutive lanes, so both the reads of k_new / v_new and the writes into the cache rows
// are coalesced.  Bound: latency, the chain position -> block id -> store; bytes are few
// (num_seqs * Hkv * D * e * 2).  A workgroup serves one sequence: its position and block id are
// scalar loads, the words to be stored are requested before either is known, and
// all indexing is shifts (rows are a power of two of words).  96 sequences, 8 heads of 128, launches back to back:
// 1.93 us; with a flat index over all words and 64-bit divisions 2.12 us; a kernel that fills 64 floats 1.75 us.
#include "kvc_internal.h"

namespace kvc {

namespace {

// PACKED: many sequences of few words, kThreads / words of them per workgroup; each lane looks up its own
// sequence's position and block id (vector loads, one more division).
template <bool PACKED>
__global__ __launch_bounds__(kThreads) void kv_cache_append_kernel(
    const uint4 *__restrict__ k_new, const uint4 *__restrict__ v_new, uint4 *__restrict__ k_cache,
    uint4 *__restrict__ v_cache, const int32_t *__restrict__ block_tables,
    const int32_t *__restrict__ positions, int num_seqs, int chunks, int num_kv_heads, int words_log2,
    int block_size_log2, int max_blocks_per_seq) {
    const int words = num_kv_heads << words_log2;
    int n, i;  // sequence, word of its new token
    if (PACKED) {
        const int per_group = kThreads / words, local = threadIdx.x / words;
        n = blockIdx.x * per_group + local;
        i = threadIdx.x - local * words;
        if (local >= per_group || n >= num_seqs) return;
    } else {  // blockIdx.x = chunk of the sequence's words + chunks * sequence
        n = chunks == 1 ? blockIdx.x : blockIdx.x / chunks;
        i = (blockIdx.x - n * chunks) * kThreads + threadIdx.x;
        if (i >= words) return;
    }
    const size_t src = size_t(n) * words + i;
    const uint4 k = k_new[src], v = v_new[src];
    const int pos = positions[n];
    // negative: skip the sequence; past the block table's reach: nothing to write to (not an error
    // this launch can report, but never an out-of-range table read)
    if (pos < 0 || (pos >> block_size_log2) >= max_blocks_per_seq) return;
    const int blk = block_tables[int64_t(n) * max_blocks_per_seq + (pos >> block_size_log2)];
    const int slot = pos & ((1 << block_size_log2) - 1);
    // cache row index: ((blk * Hkv + h) * Bs + slot), in units of 1 << words_log2
    const int64_t row = ((int64_t(blk) * num_kv_heads + (i >> words_log2)) << block_size_log2) + slot;
    const int64_t dst = (row << words_log2) + (i & ((1 << words_log2) - 1));
    k_cache[dst] = k;
    v_cache[dst] = v;
}

}  // namespace

hipError_t launch_cache_append(const void *k_new, const void *v_new, void *k_cache, void *v_cache,
                               const int32_t *block_tables, const int32_t *positions, int num_seqs,
                               int num_kv_heads, int row_bytes, int block_size_log2,
                               int max_blocks_per_seq, hipStream_t stream) {
    int words_log2 = 0;  // 16-byte words of a row: 8, 16 or 32
    while ((16 << words_log2) < row_bytes) ++words_log2;
    const int64_t words = int64_t(num_kv_heads) << words_log2;
    const int64_t chunks = (words + kThreads - 1) / kThreads;
    // A workgroup per sequence unless most of its lanes would be idle and the workgroups themselves count:
    // 4000 sequences of one head of 64 2.61 us and packed 2.15, of one of 128 2.71 and 2.29; but 700 of two heads
    // of 128 2.01 and 2.06, 1000 of four 2.24 and 2.31, 4000 of eight 6.66 and 6.87.
    const bool packed = words <= 32 && num_seqs > 1024;
    const int64_t per_group = packed ? kThreads / words : 1;
    // a launch holds fewer than 2^32 threads: more sequences than fit go in several
    constexpr int64_t kMostGroups = (int64_t(1) << 32) / kThreads - 1;
    const int64_t most = packed ? kMostGroups * per_group : kMostGroups / chunks;
    if (most == 0) return hipErrorInvalidValue;  // the words of one sequence alone
    for (int64_t n = 0; n < num_seqs; n += most) {
        const int64_t seqs = num_seqs - n < most ? num_seqs - n : most;
        const int64_t grid = packed ? (seqs + per_group - 1) / per_group : seqs * chunks;
        (packed ? kv_cache_append_kernel<true> : kv_cache_append_kernel<false>)<<<dim3(unsigned(grid)), dim3(kThreads), 0, stream>>>(
            static_cast<const uint4 *>(k_new) + n * words, static_cast<const uint4 *>(v_new) + n * words,
            static_cast<uint4 *>(k_cache), static_cast<uint4 *>(v_cache), block_tables + n * max_blocks_per_seq,
            positions + n, int(seqs), int(chunks), num_kv_heads, words_log2, block_size_log2, max_blocks_per_seq);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace kvc

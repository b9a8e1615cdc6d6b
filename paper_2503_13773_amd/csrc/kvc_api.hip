// C ABI of libkvc_hip.so: argument checks, launch planning, kernel launches.
// The contract of every entry point is stated in include/kvc.h.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "kvc_internal.h"

// Workspace of kvc_paged_attention_decode_noalloc: one copy per GPU, placed by the loader with the
// code object and held until the process ends.  In host code the name below is only a handle
// for hipGetSymbolAddress; the address kernels can use is looked up once per device.
constexpr size_t kScratchBytes = size_t(KVC_NOALLOC_WORKSPACE_BYTES);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

thread_local int g_last_hip_error = 0;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call per device).
hipError_t scratch_of_current_device(void **ptr) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

int hip_failed(hipError_t e) {
    g_last_hip_error = int(e);
    return KVC_ERR_LAUNCH;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool is_pow2(int x) { return x > 0 && (x & (x - 1)) == 0; }
int ilog2(int x) { int l = 0; while ((1 << l) < x) ++l; return l; }
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

constexpr int kMaxPartitionTokens = 4096;  // 4 wavefronts x 64 table entries x 16 tokens
constexpr int kMaxBalancedChunkTokens = 1 << 20;  // explicit minimum range of the balanced kernel
constexpr int64_t kMaxGrid = 0x7fffffff;

struct Plan {
    int kernel;
    int partition_tokens;
    int max_partitions;
    int head_chunk;       // vector-ALU kernel
    int64_t partial_grid;
    int64_t merge_grid;
    uint64_t acc_offset;  // offset of the accumulator array inside the workspace (after the counter header)
    uint64_t ml_offset;   // offset of the (max, sum) array
    uint64_t workspace_bytes;  // asked for: does for smaller calls too (below)
    uint64_t workspace_need;   // this call's own
    int min_chunk_tiles;
    int max_context_len;
    int layout;           // balanced: how the rows are dealt out (kRanges, kPieces, kWhole)
};

enum : int {
    kRanges = 0,  // a wavefront per range of the batch's flat tiles
    kPieces = 1,  // few rows: a workgroup per piece of a row
    kWhole = 2    // short contexts: a workgroup per row
};
using BalancedLauncher = decltype(&kvc::launch_partial_mfma_stream);
BalancedLauncher balanced_launcher(const Plan &pl) {
    return pl.layout == kWhole ? kvc::launch_whole_mfma : pl.layout == kPieces ? kvc::launch_rows_mfma : kvc::launch_partial_mfma_stream;
}

bool mfma_ok(const kvc_attn_desc &d) {
    return d.dtype == KVC_BF16 && d.head_dim == 128 && d.block_size >= 16 &&
           d.num_q_heads / d.num_kv_heads <= 16;
}

// The balanced kernel keeps a prefix sum over the batch in LDS and indexes flat tiles in int32.
bool balanced_ok(const kvc_attn_desc &d, int max_ctx) {
    return d.dtype == KVC_BF16 && d.head_dim == 128 && d.block_size >= 4 &&
           d.num_q_heads / d.num_kv_heads <= 16 && d.num_seqs <= kvc::kMaxStreamSeqs &&
           int64_t(d.num_seqs) * d.num_kv_heads * (ceil_div(max_ctx, 16) + 1) < (int64_t(1) << 30) &&
           int64_t(d.num_pool_blocks) * d.num_kv_heads * std::max(1, d.block_size / 16) < (int64_t(1) << 31);
}

// Few rows (sequence, KV head): a workgroup takes a piece of a row and pieces meet once, instead of a wavefront
// taking a range of flat tiles.  The grid holds 256 pieces and the last piece of a row is half empty on average,
// so what many rows of long contexts lose in streaming outgrows what the shorter chain saves.  The line, in
// us with the ranges / with the pieces (head_dim 128, 32 / 8 heads unless said; rows x tokens of the bound):
//   8 x 3217 15.0 / 11.9, 8 x 32000 68 / 28.6, 32 x 32000 76.7 / 68.1, 64 x 8192 38.6 / 37.1, 64 x 16000 63.6 / 64.5,
//   64 x 32000 116 / 121, 128 x 400 11.5 / 10.6, 128 x 3000 25.2 / 25.7, 128 x 8192 60.6 / 69.4;
//   head_dim 64: 8 x 32000 40.2 / 19.1, 64 x 8192 25.0 / 23.1, 128 x 400 11.3 / 7.0, 128 x 1500 12.6 / 13.1.
constexpr int kFewRowSeqs = 64;
constexpr int kFewRowsMinTiles = 8;  // smallest piece of a cut row: a tile for each wavefront
bool few_rows_ok(const kvc_attn_desc &d, int max_ctx) {
    const int64_t rows = int64_t(d.num_seqs) * d.num_kv_heads;
    return d.partition_tokens == 0 && d.num_seqs >= 1 && d.num_seqs <= kFewRowSeqs && rows <= kvc::kMaxFewRows &&
           rows * rows * rows * max_ctx <= (int64_t(1) << 31);
}

// Workspace of the balanced kernel's ranges and pieces: the header and two partial slots per wavefront.
struct BalancedWorkspace {
    uint64_t ml_offset, bytes;
    explicit BalancedWorkspace(const kvc_attn_desc &d) {
        const uint64_t slots = uint64_t(kvc::kNumCUs) * kvc::kWaves * 2, group = d.num_q_heads / d.num_kv_heads;
        ml_offset = (kvc::kWorkspaceHeaderBytes + slots * group * d.head_dim * sizeof(float) + 255) & ~uint64_t(255);
        bytes = ml_offset + slots * group * 2 * sizeof(float);
    }
};

bool balanced64_form(const kvc_attn_desc &d) {
    return d.kernel == KVC_KERNEL_AUTO && d.dtype == KVC_BF16 && d.head_dim == 64 && d.block_size >= 4 &&
           d.partition_tokens == 0 && d.num_q_heads / d.num_kv_heads <= 16;
}

// A workspace sized for a batch has to do for a smaller one or a lower bound that the balanced kernel serves, also where the
// batch itself is the vector ALUs': too many sequences, or few rows.  Up to 640 tokens a smaller batch at head_dim 64 is
// whole rows, which need none; above, it may be pieces or ranges.  (Among calls of the vector-ALU kernel alone sizes can fall
// with the batch, whose partitions get longer then: fp32 of 64, 32 / 8 heads, 1000 tokens, 17305600 bytes for 512
// sequences and 8671744 for 513.)
constexpr int kWhole64Tokens = 640, kWhole128Tokens = 512, kWhole128Rows = 2048;
bool smaller_calls_need_balanced(const kvc_attn_desc &d, int max_ctx) {
    return balanced64_form(d) && d.num_seqs > 0 && max_ctx > kWhole64Tokens;
}

// Short contexts: a workgroup per row, two memory round trips to the first K and V bytes and no exchange.  In us, the
// best of the other layouts / whole rows (32 / 8 heads unless said, lengths at or below the bound):
//   head_dim 128: 1 x 300 7.4 / 5.7, 1 x 500 8.9 / 8.1, 20 x 100 9.4 / 4.9, 64 x 300 19.8 / 14.5, 32 x 600 20.2 / 15.2,
//     128 x 500 45.0 / 41.0; 14 / 2 heads 64 x 700 15.3 / 13.5, 20 x 1000 11.0 / 15.4; 64 x 1000 34.5 / 35.4; with more than
//     about 1000 rows of up to 200 tokens the ranges win: 128 x 100 13.1 / 13.6, 1000 x 80 56 / 70 (128 x 300 31.8 / 26.9).
//     The compute units hold 512 of these workgroups at a time, so a bound far above the lengths costs the more the more rows there
//     are: bounds of 300 to 512, 256 x 250 39.3 / 35.8, 256 x 150 27.3 / 25.5, 256 x 16 7.6 / 11.6; 64 / 8 heads 512 x 150 54.1 / 54.2,
//     512 x 16 13.9 / 23.9; 1024 x 150 97 / 99, 1024 x 16 23 / 42: no more than 2048 rows;
//   head_dim 64: 1 x 500 7.0 / 5.5, 64 x 500 17.9 / 12.4, 20 x 1000 12.8 / 10.7; 14 / 2 heads on the vector ALUs before:
//     128 x 500 36.2 / 8.2; but one head per KV head and many rows of one partition on the vector ALUs: 12 / 12 heads
//     64 x 100 4.3 / 5.1, 83 x 150 7.6 / 8.1 (up to 640 rows they lead by a tenth at most: 42 x 100 3.9 / 4.3, 16 / 16 10 x 256 3.8 / 4.05).
bool whole_ok(const kvc_attn_desc &d, int max_ctx) {
    const int64_t rows = int64_t(d.num_seqs) * d.num_kv_heads;
    if (d.partition_tokens != 0 || d.num_seqs < 1 || d.num_seqs > kvc::kMaxStreamSeqs) return false;
    if (d.head_dim == 128) return max_ctx <= kWhole128Tokens && rows <= kWhole128Rows && !(rows > 1000 && max_ctx <= 200);
    return max_ctx <= (rows > kvc::kMaxFewRows ? 1024 : kWhole64Tokens) &&
           (max_ctx > 256 || rows <= 640 || d.num_q_heads > d.num_kv_heads);
}

// At head_dim 64 the balanced kernel serves calls that KVC_KERNEL_AUTO brings without a split of the caller's
// own: whole rows, few rows, and ranges; the vector ALUs keep what they do as fast.  In us, there / here:
//   few rows, by (query head, partition) pairs.  Groups of four and more to 384: 32 / 8 heads 1 x 1536, 192 pairs, 6.5 / 7.8, 2 x 1536 7.8 / 8.6, 1 x
//     4096, 512 pairs, 9.3 / 8.8; 14 / 2 1 x 1792 6.5 / 7.5, 4 x 2048, 448 pairs, 7.8 / 7.9, 6 x 1792, 588 pairs, 9.9 / 8.2; 16 / 2 1 x 6144
//     8.2 / 8.3, 8 x 1280, 640 pairs, 10.7 / 8.3 (but 16 x 512 in whole rows, 14 / 2 7.3 / 5.4).  Two heads to 512, 16 / 8 2 x 1536 6.5 / 8.6, 8 / 4 16 x
//     1024 8.0 / 9.0, with about a tenth left above: 16 / 8 4 x 4096, 1024 pairs, 9.8 / 10.9, 6 x 2816 11.7 / 11.0.  One head per KV head,
//     where they read nothing twice, to 1024: 12 / 12 2 x 4096 7.9 / 10.5, 8 x 2048, 768 pairs, 11.9 / 15.6, 1 x 21760 19.7 / 17.4, 16 / 16 2 x
//     8192, 1024 pairs, 16.0 / 15.8 (but 128 rows fill the device here: 16 / 16 heads 8 x 1500 15.0 / 13.9);
//   more rows below 2^17 tokens x KV heads: 102 k 9.7 / 11.9, 128 k 14.0 / 11.8, 524 k 39.3 / 25.2, 1 M 33.1 / 20.1 (one head per KV head: 128 rows
//     of 1500 15.5 / 14.2, 12 / 12 heads 16 x 2000 18.8 / 18.6, 64 x 2000 52.6 / 53.1, 64 x 4000 114 / 98).
bool balanced64_ok(const kvc_attn_desc &d, int max_ctx) {
    const int group = d.num_q_heads / d.num_kv_heads;
    const int64_t rows = int64_t(d.num_seqs) * d.num_kv_heads, pairs = rows * group * ceil_div(max_ctx, 256);
    return balanced64_form(d) && d.num_seqs <= kvc::kMaxStreamSeqs &&
           (whole_ok(d, max_ctx) || (few_rows_ok(d, max_ctx) ? pairs > (group == 1 && rows < kvc::kMaxFewRows ? 1024 : group == 2 ? 512 : 384)
                                                              : max_ctx > 256 && rows * max_ctx >= (1 << 17))) &&
           rows * (ceil_div(max_ctx, 32) + 1) < (int64_t(1) << 30) &&
           int64_t(d.num_pool_blocks) * d.num_kv_heads * std::max(1, d.block_size / 32) < (int64_t(1) << 31);
}

// head_dim 64 has a matrix-core prefill kernel of its own, for every group size and scale.  A workgroup of it takes up to 64
// or 128 rows of a sequence, two workgroups a compute unit; one on the vector ALUs takes one row for as many heads as
// it holds (valu_head_chunk: 1 for odd groups, else 2, 4 or 8).  The vector ALUs keep (us there / on the matrix cores)
//   launches of at most two workgroups a compute unit with one head each, or one with two: 14 / 2 heads, one sequence of
//     400 tokens, 2 rows 5.9 / 7.4, 32 rows 6.9 / 7.8, 64 rows 9.2 / 8.2; of 1500, 2 rows 12.1 / 14.9, 32 rows 14.9 / 15.0; 16 / 8 heads
//     of 1500, 2 rows 15.7 / 15.0, four sequences of 16 rows 20.1 / 14.8 (with four heads each, 32 / 8, 1 x 2 rows 24.1 / 15.1);
//   batches that are mostly decode steps, one row each, and a few longer ones, where K and V of a sequence are read
//     once per head chunk by either: 32 / 8 heads, 128 sequences of 800, a fifth of them of two rows and the rest of one 42.8 / 48.5, half of
//     them 48.9 / 48.8, three quarters 57.2 / 48.8; 24 / 8 heads of 200, half of them, 29.3 / 39.5 (of 800 90 / 69).  Two heads per
//     workgroup lose their lead earlier: 16 / 8 heads of 800, 1.2 rows on average 37.5 / 34.4.  Eight heads are too
//     few workgroups: 16 / 1 heads, 64 of 1500 at 1.6 rows 46.2 / 33.0;
//   tiles most of which would be empty: a workgroup without rows still costs 1.2 ns (4096 sequences of 2 rows with a bound of
//     8000 575 / 11000);
//   and what a launch cannot hold: HIP refuses 2^32 threads and more.
bool prefill_d64_ok(const kvc::PrefillParams &p, int total_q, int max_query_len) {
    const int tile_rows = 128 / p.heads_per_chunk, valu_heads = kvc::valu_head_chunk(p.group);
    const int64_t tiles = int64_t(p.num_q_heads / p.heads_per_chunk) * p.num_seqs * ceil_div(std::min(max_query_len, total_q), tile_rows);
    const int64_t valu_grid = int64_t(total_q) * (p.num_q_heads / valu_heads);
    if (max_query_len <= 1 || tiles >= (int64_t(1) << 32) / kvc::kPrefill64Threads || tiles > 8 * valu_grid) return false;
    if (valu_heads <= 2 && valu_grid * valu_heads <= 2 * kvc::kNumCUs) return false;
    const double rows = double(total_q) / p.num_seqs;
    return valu_heads == 8 || rows >= (valu_heads == 2 ? 1.1 : 1.75);
}

// A workgroup of the vector-ALU kernel takes as many heads of a KV head as its registers hold, which reads K and V
// once for all of them; a launch of few workgroups spends its time on the chain of one of them, which is
// shorter with a head each.  The line, in (query head, partition) pairs, and both sides (us with the heads together / one each, or the
// quotient over contexts of 100 to 5000 tokens):
//   four heads, together : one each by pairs: fp32 of 64 1.65 at 256, 1.02 at 384, 0.76 at 448; fp32 of 128 1.50, 0.96, 0.83; bf16 of 64 1.45, 1.31,
//     1.27; bf16 of 128 1.62, 1.01, 1.00, but in several partitions with four heads per KV head, whose reads meet less often in the
//     caches, 32 / 8, 1 x 2560, 320 pairs, 14.9 / 14.5, 1 x 3000, 384 pairs, 15.0 / 16.1 (one partition, 12 x 100, 384 pairs, 8.1 / 5.0);
//   eight heads: 1.6 (fp32 of 64 1.4) at 384, fp32 of 64 1.02 at 672 to 768 and 0.84 above, fp32 of 128 0.98 and 0.90, bf16 of 128
//     1.01 and 0.81, bf16 of 64 1.27 and 1.04;
//   two heads lose less together: rows of 256 bytes and more, fp32 of 64 1.23 at 256, 0.93 at 352 to 384, bf16 of 128 1.24 and 0.89; fp32 of 128
//     crosses before that (1.04 at 200, 0.73 at 256); rows of 128 bytes (bf16 of 64) 1.03 at 384, 1.00 at 512.
int64_t few_row_parts(const kvc_attn_desc &d, int heads, int64_t parts) {
    const bool wide_rows = d.head_dim * (d.dtype == KVC_F32 ? 4 : 2) >= 256;
    if (heads == 8) return 768;
    if (heads == 2 && wide_rows) return 256;
    return d.dtype == KVC_BF16 && wide_rows && d.num_q_heads == 4 * d.num_kv_heads && parts > 1 ? 320 : 384;
}

int make_plan(const kvc_attn_desc *d, Plan *pl) {
    if (!d) return KVC_ERR_NULL;
    if (d->num_seqs < 0 || d->num_q_heads <= 0 || d->num_kv_heads <= 0 || d->head_dim <= 0 ||
        d->block_size <= 0 || d->max_blocks_per_seq <= 0 || d->num_pool_blocks <= 0 ||
        d->max_context_len < 0 || d->partition_tokens < 0 || d->reserved != 0)
        return KVC_ERR_BAD_SHAPE;
    if (d->num_q_heads % d->num_kv_heads != 0) return KVC_ERR_BAD_SHAPE;
    if (d->dtype != KVC_F32 && d->dtype != KVC_BF16) return KVC_ERR_BAD_DTYPE;
    if (d->head_dim != 64 && d->head_dim != 128) return KVC_ERR_UNSUPPORTED;
    if (!is_pow2(d->block_size) || d->block_size > 256) return KVC_ERR_UNSUPPORTED;
    const int64_t table_tokens = int64_t(d->max_blocks_per_seq) * d->block_size;
    if (table_tokens > 0x40000000) return KVC_ERR_BAD_SHAPE;
    if (d->max_context_len > table_tokens) return KVC_ERR_BAD_SHAPE;
    const int max_ctx = d->max_context_len ? d->max_context_len : int(table_tokens);
    if (d->partition_tokens % 16 != 0) return KVC_ERR_BAD_SHAPE;
    if (d->partition_tokens > (d->kernel == KVC_KERNEL_MFMA_BALANCED ? kMaxBalancedChunkTokens : kMaxPartitionTokens))
        return KVC_ERR_BAD_SHAPE;

    int kernel = d->kernel;
    if (kernel < KVC_KERNEL_AUTO || kernel > KVC_KERNEL_MFMA_BALANCED) return KVC_ERR_BAD_SHAPE;
    if (kernel == KVC_KERNEL_AUTO)
        kernel = balanced_ok(*d, max_ctx) || balanced64_ok(*d, max_ctx) ? KVC_KERNEL_MFMA_BALANCED
                 : mfma_ok(*d)            ? KVC_KERNEL_MFMA
                                          : KVC_KERNEL_VALU;
    if ((kernel == KVC_KERNEL_MFMA || kernel == KVC_KERNEL_MFMA_LDS) && !mfma_ok(*d)) return KVC_ERR_UNSUPPORTED;
    if (kernel == KVC_KERNEL_MFMA_BALANCED && !balanced_ok(*d, max_ctx) && !balanced64_ok(*d, max_ctx))
        return KVC_ERR_UNSUPPORTED;

    const int64_t rows = int64_t(d->num_seqs) * d->num_q_heads;
    constexpr uint64_t kHeader = kvc::kWorkspaceHeaderBytes;
    if (kernel == KVC_KERNEL_MFMA_BALANCED) {
        // One launch: cut rows are merged by the last worker to arrive.  A wavefront never takes
        // fewer than min_chunk tiles; the workspace is two partial slots per wavefront.
        const int tile_tokens = d->head_dim == 64 ? 32 : 16;  // 8 KiB of K and V
        const int64_t max_tiles = ceil_div(max_ctx, tile_tokens);
        pl->layout = whole_ok(*d, max_ctx) ? kWhole : few_rows_ok(*d, max_ctx) ? kPieces : kRanges;
        const int min_chunk = pl->layout == kWhole    ? int(max_tiles)
                              : pl->layout == kPieces ? kFewRowsMinTiles
                              : d->partition_tokens ? d->partition_tokens / tile_tokens
                                                    : int(std::max<int64_t>(4, ceil_div(max_tiles, 32)));
        pl->kernel = kernel;
        pl->head_chunk = 0;
        pl->partition_tokens = min_chunk * tile_tokens;
        pl->min_chunk_tiles = min_chunk;
        pl->max_partitions = 2;           // partial slots per worker
        // 4 wavefronts per CU: one worker per SIMD; whole rows: a workgroup each
        pl->partial_grid = pl->layout == kWhole ? int64_t(d->num_seqs) * d->num_kv_heads : kvc::kNumCUs;
        pl->merge_grid = 0;
        pl->max_context_len = max_ctx;
        const BalancedWorkspace need(*d);
        pl->acc_offset = kHeader;
        pl->ml_offset = need.ml_offset;
        pl->workspace_bytes = need.bytes;
        // whole rows need no workspace; head_dim 128 keeps asking for one (its size never depended on the lengths)
        if (d->head_dim == 64 && pl->layout == kWhole && !smaller_calls_need_balanced(*d, max_ctx)) pl->workspace_bytes = 0;
        pl->workspace_need = pl->workspace_bytes;
        return KVC_OK;
    }

    const int group = d->num_q_heads / d->num_kv_heads;
    pl->head_chunk = kvc::valu_head_chunk(group);
    int64_t base_items = kernel == KVC_KERNEL_VALU ? rows / pl->head_chunk : int64_t(d->num_seqs) * d->num_kv_heads;
    int pt = d->partition_tokens;
    if (pt == 0) {
        // Short partitions spread a skewed length mix over the 256 CUs; longer ones keep the
        // grid (mostly idle workgroups when max_context_len is loose) and the workspace small.
        if (max_ctx <= 256) {
            pt = int(ceil_div(max_ctx, 16) * 16);
        } else {
            pt = 256;
            while (pt < kMaxPartitionTokens && base_items * ceil_div(max_ctx, pt) > 16384) pt *= 2;
        }
    }
    const int64_t parts = ceil_div(max_ctx, pt);
    if (kernel == KVC_KERNEL_VALU && rows * parts <= few_row_parts(*d, pl->head_chunk, parts)) {
        pl->head_chunk = 1;
        base_items = rows;
    }
    if (base_items * parts > kMaxGrid || rows * parts > kMaxGrid) return KVC_ERR_BAD_SHAPE;

    pl->kernel = kernel;
    pl->partition_tokens = pt;
    pl->max_partitions = int(parts);
    pl->partial_grid = base_items * parts;
    pl->merge_grid = parts > 1 ? ceil_div(rows, kvc::kWaves) : 0;
    pl->max_context_len = max_ctx;
    pl->min_chunk_tiles = 0;
    pl->layout = kRanges;
    pl->acc_offset = kHeader;
    if (parts > 1) {
        const uint64_t acc = uint64_t(rows) * parts * d->head_dim * sizeof(float);
        pl->ml_offset = (kHeader + acc + 255) & ~uint64_t(255);
        pl->workspace_need = pl->ml_offset + uint64_t(rows) * parts * 2 * sizeof(float);
    } else {
        pl->ml_offset = 0;
        pl->workspace_need = 0;
    }
    pl->workspace_bytes = pl->workspace_need;
    if (kernel == KVC_KERNEL_VALU && smaller_calls_need_balanced(*d, max_ctx))
        pl->workspace_bytes = std::max(pl->workspace_bytes, BalancedWorkspace(*d).bytes);
    return KVC_OK;
}

kvc::AttnParams make_params(const kvc_attn_desc &d, const Plan &pl, float scale) {
    kvc::AttnParams p;
    p.num_seqs = d.num_seqs;
    p.num_q_heads = d.num_q_heads;
    p.num_kv_heads = d.num_kv_heads;
    p.group = d.num_q_heads / d.num_kv_heads;
    p.block_size = d.block_size;
    p.block_size_log2 = ilog2(d.block_size);
    p.max_blocks_per_seq = d.max_blocks_per_seq;
    p.partition_tokens = pl.partition_tokens;
    p.max_partitions = pl.max_partitions;
    p.head_chunk = pl.head_chunk;
    p.merge_here = 0;
    p.k_via_lds = pl.kernel == KVC_KERNEL_MFMA_LDS;
    p.min_chunk_tiles = pl.min_chunk_tiles;
    p.max_context_len = pl.max_context_len;
    p.scale = scale;
    p.scale_log2e = float(double(scale) * 1.4426950408889634);
    return p;
}

int check_workspace(const Plan &pl, void *workspace, size_t workspace_bytes, kvc::Workspace *ws) {
    ws->acc = nullptr;
    ws->ml = nullptr;
    ws->cnt = nullptr;
    if (pl.workspace_need == 0) return KVC_OK;
    if (!workspace || workspace_bytes < pl.workspace_need) return KVC_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return KVC_ERR_ALIGN;
    unsigned char *base = static_cast<unsigned char *>(workspace);
    ws->cnt = reinterpret_cast<int32_t *>(base);
    ws->acc = reinterpret_cast<float *>(base + pl.acc_offset);
    ws->ml = reinterpret_cast<float *>(base + pl.ml_offset);
    return KVC_OK;
}

// Whether the vector-ALU kernel merges the partitions of a context itself: a counter word for each (sequence, heads of a
// workgroup), and no more partials than a wavefront holds weights of at once.  It saves the second launch for a count and a fetch, us in two
// launches / one: fp32, 12 / 12 heads of 64, 7 x 607 tokens 7.4 / 6.8, 16 / 4 of 128, 5 x 1000 18.5 / 17.7; bf16 of 64, 14 / 2, 4 x 1500 7.6 /
// 7.6, 4 of up to 587 under a bound of 1174 6.4 / 5.9.  The last workgroup of a row fetches that row's partials alone, after its own are
// published, while the launch spreads all of them; so few rows of many partitions, which all end at about the same time, do better in two
// launches: bf16 of 64, 16 / 16, 1 x 8192, 32 partitions, 9.1 / 12.4, 14 / 2, 1 x 6144 8.1 / 9.9; fp32, 16 / 4 of 64, 1 x 4096 7.8 / 9.3.  In
// all, one launch : two is 0.96 up to 8 partitions (bf16 6) and from 32 rows on (bf16 64), and 1.02 with less of both, up to 1.27.  Eight
// heads, which four wavefronts merge in two turns: 1.02 (64 / 8 heads of 64, 2 x 4096, bf16 13.1 / 16.1, fp32 17.9 / 20.5).
bool merges_itself(const kvc_attn_desc &d, const Plan &pl) {
    const int64_t rows = int64_t(d.num_seqs) * (d.num_q_heads / std::max(pl.head_chunk, 1));
    const bool wide = d.dtype == KVC_F32;
    return pl.kernel == KVC_KERNEL_VALU && pl.head_chunk < 8 && pl.max_partitions > 1 && pl.max_partitions <= 64 &&
           (pl.max_partitions <= (wide ? 8 : 6) || rows >= (wide ? 32 : 64)) &&
           rows <= int64_t(kvc::kWorkspaceHeaderBytes / sizeof(int32_t));
}

int run_partial(const void *q, const void *k_cache, const void *v_cache, const int32_t *block_tables,
                const int32_t *context_lens, float scale, void *out, const kvc_attn_desc *desc,
                const Plan &pl, kvc::Workspace ws, bool merge_here, hipStream_t stream) {
    kvc::AttnParams p = make_params(*desc, pl, scale);
    p.merge_here = merge_here;
    hipError_t e;
    if (pl.kernel == KVC_KERNEL_VALU)
        e = kvc::launch_partial_valu(q, k_cache, v_cache, block_tables, context_lens, out, ws, p,
                                     desc->dtype, desc->head_dim, int(pl.partial_grid), stream);
    else if (pl.kernel == KVC_KERNEL_MFMA_BALANCED)
        e = balanced_launcher(pl)(q, k_cache, v_cache, block_tables, context_lens, out,
                                            ws, p, desc->head_dim, int(pl.partial_grid), 0, kvc::Schedule{}, stream);
    else
        e = kvc::launch_partial_mfma(q, k_cache, v_cache, block_tables, context_lens, out, ws, p,
                                     int(pl.partial_grid), stream);
    return e == hipSuccess ? KVC_OK : hip_failed(e);
}

int run_merge(const int32_t *context_lens, void *out, const kvc_attn_desc *desc, const Plan &pl,
              kvc::Workspace ws, hipStream_t stream) {
    if (pl.merge_grid == 0) return KVC_OK;
    const kvc::AttnParams p = make_params(*desc, pl, 1.0f);
    const hipError_t e = kvc::launch_merge(context_lens, out, ws, p, desc->dtype, desc->head_dim,
                                           pl.kernel != KVC_KERNEL_VALU, int(pl.merge_grid), stream);
    return e == hipSuccess ? KVC_OK : hip_failed(e);
}

// Layout of a schedule buffer for a descriptor served by the balanced kernel.
struct ScheduleLayout {
    uint64_t pref_off, ctx_off, plans_off, tiles_off, bytes;
    int stride;
};

bool schedule_layout(const kvc_attn_desc &d, const Plan &pl, ScheduleLayout *L) {
    if (pl.kernel != KVC_KERNEL_MFMA_BALANCED || d.head_dim != 128) return false;
    const int64_t units_per_tile = d.block_size >= 16 ? 1 : 16 / d.block_size;
    const int64_t max_tiles = ceil_div(pl.max_context_len, 16);
    const int64_t rows = int64_t(d.num_seqs) * d.num_kv_heads;
    // Ranges: no wavefront takes more flat units than this, whatever the context lengths turn out to be.
    const int64_t range_workers = int64_t(kvc::kNumCUs) * kvc::kWaves;
    const int64_t min_chunk = d.partition_tokens ? d.partition_tokens / 16 : std::max<int64_t>(4, ceil_div(max_tiles, 32));
    const int64_t range_chunk = std::max<int64_t>(min_chunk, ceil_div(rows * (max_tiles + 1), range_workers));
    // Pieces: nor a workgroup more tiles than this with n sequences.
    auto piece_chunk = [&](int64_t n) {
        return std::max({int64_t(kFewRowsMinTiles), std::min<int64_t>(max_tiles, kvc::kRowWholeTiles),
                         ceil_div(max_tiles, kvc::kMaxRowPieces),
                         ceil_div(n * max_tiles, kvc::kNumCUs / d.num_kv_heads - n)});
    };
    const int64_t workers = pl.layout == kRanges ? range_workers : pl.partial_grid;  // wavefronts, or workgroups
    const int64_t stride = units_per_tile * (pl.layout == kWhole ? max_tiles : pl.layout == kPieces ? piece_chunk(d.num_seqs) : range_chunk);
    if (stride > (int64_t(1) << 28)) return false;
    auto up = [](uint64_t x) { return (x + 255) & ~uint64_t(255); };
    L->stride = int(stride);
    L->pref_off = 0;
    L->ctx_off = up(uint64_t(d.num_seqs + 2) * 4);
    L->plans_off = L->ctx_off + up(uint64_t(d.num_seqs) * 4);
    L->tiles_off = L->plans_off + up(uint64_t(workers) * 16 * 4);
    // A buffer sized for a batch has to do for a smaller one or a lower bound, also where those have another
    // layout: room for the largest of the layouts that they can have.
    auto body = [&](int64_t n, int64_t chunk) {
        return up(uint64_t(n) * 16 * 4) + up(uint64_t(n) * uint64_t(chunk * units_per_tile) * 4);
    };
    uint64_t most = body(range_workers, range_chunk);
    if (d.partition_tokens == 0) {
        most = std::max(most, body(std::min<int64_t>(rows, kWhole128Rows), std::min<int64_t>(max_tiles, kWhole128Tokens / 16)));
        const int64_t few = std::min<int64_t>({d.num_seqs, kFewRowSeqs, kvc::kMaxFewRows / d.num_kv_heads});
        if (few > 0) most = std::max(most, body(kvc::kNumCUs, piece_chunk(few)));
    }
    L->bytes = L->plans_off + most;
    return true;
}

kvc::Schedule schedule_view(void *base, const ScheduleLayout &L) {
    auto *b = static_cast<unsigned char *>(base);
    kvc::Schedule s;
    s.pref = reinterpret_cast<int *>(b + L.pref_off);
    s.ctx = reinterpret_cast<int *>(b + L.ctx_off);
    s.plans = reinterpret_cast<int *>(b + L.plans_off);
    s.tiles = reinterpret_cast<int *>(b + L.tiles_off);
    s.stride = L.stride;
    return s;
}

int check_attn_args(const void *q, const void *k_cache, const void *v_cache,
                    const int32_t *block_tables, const int32_t *context_lens, float scale,
                    const void *out) {
    if (!q || !k_cache || !v_cache || !block_tables || !context_lens || !out) return KVC_ERR_NULL;
    if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(out))
        return KVC_ERR_ALIGN;
    if (!isfinite(scale)) return KVC_ERR_BAD_SHAPE;
    return KVC_OK;
}

int check_pools(const kvc_pool *src, const kvc_pool *dst, const int64_t *mapping, int64_t num_pairs) {
    if (!src || !dst) return KVC_ERR_NULL;
    if (num_pairs < 0) return KVC_ERR_BAD_SHAPE;
    for (const kvc_pool *pl : {src, dst}) {
        if (pl->num_blocks <= 0 || pl->block_bytes <= 0 || pl->num_planes <= 0 || pl->reserved != 0)
            return KVC_ERR_BAD_SHAPE;
        if (pl->num_planes > 65535) return KVC_ERR_UNSUPPORTED;
        if (pl->block_bytes % 16 != 0) return KVC_ERR_ALIGN;
        if (pl->num_planes > 1) {
            if (pl->plane_stride_bytes % 16 != 0) return KVC_ERR_ALIGN;
            if (pl->plane_stride_bytes / pl->block_bytes < pl->num_blocks) return KVC_ERR_BAD_SHAPE;
        }
    }
    if (src->block_bytes != dst->block_bytes || src->num_planes != dst->num_planes)
        return KVC_ERR_BAD_SHAPE;
    if (num_pairs == 0) return KVC_OK;
    if (!src->base || !dst->base || !mapping) return KVC_ERR_NULL;
    if (!aligned16(src->base) || !aligned16(dst->base)) return KVC_ERR_ALIGN;
    const int64_t slabs = ceil_div(src->block_bytes, kvc::kCopySlabBytes);
    if (num_pairs > kMaxGrid / slabs) return KVC_ERR_BAD_SHAPE;
    return KVC_OK;
}

}  // namespace

extern "C" {

int kvc_version(void) { return 200; }

const char *kvc_status_string(int status) {
    switch (status) {
        case KVC_OK: return "ok";
        case KVC_ERR_NULL: return "a required pointer is NULL";
        case KVC_ERR_BAD_SHAPE: return "a size is non-positive or inconsistent";
        case KVC_ERR_BAD_DTYPE: return "unknown dtype";
        case KVC_ERR_UNSUPPORTED: return "shape or option not implemented";
        case KVC_ERR_WORKSPACE: return "workspace missing or too small";
        case KVC_ERR_ALIGN: return "pointer or stride not aligned";
        case KVC_ERR_LAUNCH: return "HIP call failed (see kvc_last_hip_error)";
        case KVC_ERR_BAD_INDEX: return "index out of range";
        case KVC_ERR_DUPLICATE: return "destination block listed twice";
        case KVC_ERR_OVERLAP: return "source and destination blocks overlap in one pool";
        default: return "unknown status";
    }
}

int kvc_last_hip_error(void) { return g_last_hip_error; }

int kvc_attn_plan(const kvc_attn_desc *desc, kvc_attn_plan_info *plan) {
    if (!plan) return KVC_ERR_NULL;
    Plan pl;
    const int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    plan->kernel = pl.kernel;
    plan->partition_tokens = pl.partition_tokens;
    plan->max_partitions = pl.max_partitions;
    plan->partial_grid = int32_t(pl.partial_grid);
    plan->merge_grid = int32_t(pl.merge_grid);
    plan->reserved = 0;
    plan->workspace_bytes = pl.workspace_bytes;
    return KVC_OK;
}

size_t kvc_paged_attention_decode_workspace_bytes(const kvc_attn_desc *desc) {
    Plan pl;
    return make_plan(desc, &pl) == KVC_OK ? size_t(pl.workspace_bytes) : 0;
}

int kvc_paged_attention_decode_workspace_init(void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (workspace_bytes == 0) return KVC_OK;
    if (!workspace || workspace_bytes < kvc::kWorkspaceHeaderBytes) return KVC_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return KVC_ERR_ALIGN;
    const hipError_t e = kvc::launch_workspace_init(workspace, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? KVC_OK : hip_failed(e);
}

int kvc_paged_attention_decode_partial(const void *q, const void *k_cache, const void *v_cache,
                                       const int32_t *block_tables, const int32_t *context_lens,
                                       float scale, void *out, const kvc_attn_desc *desc,
                                       void *workspace, size_t workspace_bytes, void *hip_stream) {
    Plan pl;
    int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    if (desc->num_seqs == 0) return KVC_OK;
    rc = check_attn_args(q, k_cache, v_cache, block_tables, context_lens, scale, out);
    if (rc != KVC_OK) return rc;
    kvc::Workspace ws;
    rc = check_workspace(pl, workspace, workspace_bytes, &ws);
    if (rc != KVC_OK) return rc;
    return run_partial(q, k_cache, v_cache, block_tables, context_lens, scale, out, desc, pl, ws, false,
                       static_cast<hipStream_t>(hip_stream));
}

int kvc_paged_attention_decode_merge(const int32_t *context_lens, void *out,
                                     const kvc_attn_desc *desc, void *workspace,
                                     size_t workspace_bytes, void *hip_stream) {
    Plan pl;
    int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    if (desc->num_seqs == 0) return KVC_OK;
    if (!context_lens || !out) return KVC_ERR_NULL;
    if (!aligned16(out)) return KVC_ERR_ALIGN;
    kvc::Workspace ws;
    rc = check_workspace(pl, workspace, workspace_bytes, &ws);
    if (rc != KVC_OK) return rc;
    return run_merge(context_lens, out, desc, pl, ws, static_cast<hipStream_t>(hip_stream));
}

int kvc_paged_attention_decode(const void *q, const void *k_cache, const void *v_cache,
                               const int32_t *block_tables, const int32_t *context_lens,
                               float scale, void *out, const kvc_attn_desc *desc, void *workspace,
                               size_t workspace_bytes, void *hip_stream) {
    Plan pl;
    int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    if (desc->num_seqs == 0) return KVC_OK;
    rc = check_attn_args(q, k_cache, v_cache, block_tables, context_lens, scale, out);
    if (rc != KVC_OK) return rc;
    kvc::Workspace ws;
    rc = check_workspace(pl, workspace, workspace_bytes, &ws);
    if (rc != KVC_OK) return rc;
    const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const bool merge_here = merges_itself(*desc, pl);
    rc = run_partial(q, k_cache, v_cache, block_tables, context_lens, scale, out, desc, pl, ws, merge_here, stream);
    if (rc != KVC_OK || merge_here) return rc;
    return run_merge(context_lens, out, desc, pl, ws, stream);
}

int kvc_paged_attention_decode_noalloc(const void *q, const void *k_cache, const void *v_cache,
                                       const int32_t *block_tables, const int32_t *context_lens,
                                       float scale, void *out, const kvc_attn_desc *desc,
                                       void *hip_stream) {
    Plan pl;
    int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    if (pl.workspace_need > kScratchBytes) return KVC_ERR_WORKSPACE;
    if (desc->num_seqs == 0) return KVC_OK;
    rc = check_attn_args(q, k_cache, v_cache, block_tables, context_lens, scale, out);
    if (rc != KVC_OK) return rc;
    void *base = nullptr;
    const hipError_t e = scratch_of_current_device(&base);
    if (e != hipSuccess) return hip_failed(e);
    kvc::Workspace ws;
    rc = check_workspace(pl, base, kScratchBytes, &ws);
    if (rc != KVC_OK) return rc;
    const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const bool merge_here = merges_itself(*desc, pl);
    rc = run_partial(q, k_cache, v_cache, block_tables, context_lens, scale, out, desc, pl, ws, merge_here, stream);
    if (rc != KVC_OK || merge_here) return rc;
    return run_merge(context_lens, out, desc, pl, ws, stream);
}

size_t kvc_attn_schedule_bytes(const kvc_attn_desc *desc) {
    Plan pl;
    ScheduleLayout L;
    if (make_plan(desc, &pl) != KVC_OK || !schedule_layout(*desc, pl, &L)) return 0;
    return size_t(L.bytes);
}

int kvc_attn_schedule_build(const int32_t *block_tables, const int32_t *context_lens,
                            const kvc_attn_desc *desc, void *schedule, size_t schedule_bytes,
                            void *hip_stream) {
    Plan pl;
    int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    ScheduleLayout L;
    if (!schedule_layout(*desc, pl, &L)) return KVC_ERR_UNSUPPORTED;
    if (!schedule || schedule_bytes < L.bytes) return KVC_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(schedule) & 255u) return KVC_ERR_ALIGN;
    if (desc->num_seqs == 0) return KVC_OK;
    if (!block_tables || !context_lens) return KVC_ERR_NULL;
    const kvc::AttnParams p = make_params(*desc, pl, 1.0f);
    const hipError_t e = balanced_launcher(pl)(nullptr, nullptr, nullptr, block_tables, context_lens,
                                                         nullptr, kvc::Workspace{}, p, desc->head_dim, int(pl.partial_grid), 1,
                                                         schedule_view(schedule, L),
                                                         static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? KVC_OK : hip_failed(e);
}

int kvc_paged_attention_decode_scheduled(const void *q, const void *k_cache, const void *v_cache,
                                         const void *schedule, size_t schedule_bytes, float scale,
                                         void *out, const kvc_attn_desc *desc, void *workspace,
                                         size_t workspace_bytes, void *hip_stream) {
    Plan pl;
    int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    ScheduleLayout L;
    if (!schedule_layout(*desc, pl, &L)) return KVC_ERR_UNSUPPORTED;
    if (!schedule || schedule_bytes < L.bytes) return KVC_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(schedule) & 255u) return KVC_ERR_ALIGN;
    if (desc->num_seqs == 0) return KVC_OK;
    if (!q || !k_cache || !v_cache || !out) return KVC_ERR_NULL;
    if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(out)) return KVC_ERR_ALIGN;
    if (!isfinite(scale)) return KVC_ERR_BAD_SHAPE;
    kvc::Workspace ws;
    rc = check_workspace(pl, workspace, workspace_bytes, &ws);
    if (rc != KVC_OK) return rc;
    const kvc::AttnParams p = make_params(*desc, pl, scale);
    const hipError_t e = balanced_launcher(pl)(q, k_cache, v_cache, nullptr, nullptr, out, ws, p,
                                                         desc->head_dim, int(pl.partial_grid), 2,
                                                         schedule_view(const_cast<void *>(schedule), L),
                                                         static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? KVC_OK : hip_failed(e);
}

int kvc_validate_attention_inputs(const int32_t *block_tables, const int32_t *context_lens,
                                  const kvc_attn_desc *desc, void *hip_stream) {
    Plan pl;
    const int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    if (desc->num_seqs == 0) return KVC_OK;
    if (!block_tables || !context_lens) return KVC_ERR_NULL;
    const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    std::vector<int32_t> lens(desc->num_seqs);
    std::vector<int32_t> tables(size_t(desc->num_seqs) * desc->max_blocks_per_seq);
    hipError_t e = hipMemcpyAsync(lens.data(), context_lens, lens.size() * sizeof(int32_t),
                                  hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(tables.data(), block_tables, tables.size() * sizeof(int32_t),
                           hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return hip_failed(e);
    for (int n = 0; n < desc->num_seqs; ++n) {
        if (lens[n] < 0 || lens[n] > pl.max_context_len) return KVC_ERR_BAD_INDEX;
        const int nblk = int(ceil_div(lens[n], desc->block_size));
        for (int b = 0; b < nblk; ++b) {
            const int32_t id = tables[size_t(n) * desc->max_blocks_per_seq + b];
            if (id < 0 || id >= desc->num_pool_blocks) return KVC_ERR_BAD_INDEX;
        }
    }
    return KVC_OK;
}

int kvc_paged_attention_prefill(const void *q, const void *k_cache, const void *v_cache,
                                const int32_t *block_tables, const int32_t *context_lens,
                                const int32_t *q_start, float scale, void *out,
                                const kvc_attn_desc *desc, int32_t total_q, int32_t max_query_len,
                                void *hip_stream) {
    Plan pl;
    int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    if (total_q < 0 || max_query_len < 0) return KVC_ERR_BAD_SHAPE;
    if (desc->num_seqs == 0 || total_q == 0 || max_query_len == 0) return KVC_OK;
    if (!q_start) return KVC_ERR_NULL;
    rc = check_attn_args(q, k_cache, v_cache, block_tables, context_lens, scale, out);
    if (rc != KVC_OK) return rc;
    kvc::PrefillParams p;
    p.num_seqs = desc->num_seqs;
    p.num_q_heads = desc->num_q_heads;
    p.num_kv_heads = desc->num_kv_heads;
    p.group = desc->num_q_heads / desc->num_kv_heads;
    p.heads_per_chunk = p.group % 2 == 0 ? 2 : 1;
    p.block_size = desc->block_size;
    p.block_size_log2 = ilog2(desc->block_size);
    p.tiles_per_block_log2 = desc->block_size >= 16 ? ilog2(desc->block_size / 16) : 0;
    p.max_blocks_per_seq = desc->max_blocks_per_seq;
    p.max_query_tiles = int(ceil_div(max_query_len, 64));
    p.scale_log2e = float(double(scale) * 1.4426950408889634);
    const int64_t tile_grid = int64_t(p.num_q_heads / p.heads_per_chunk) * p.num_seqs * p.max_query_tiles;
    const bool on_mfma = desc->dtype == KVC_BF16 && desc->head_dim == 128 && p.group <= 16;
    if (desc->dtype == KVC_BF16 && desc->head_dim == 64 && prefill_d64_ok(p, total_q, max_query_len)) {
        // no sequence has more rows than there are
        const hipError_t e = kvc::launch_prefill_d64(q, k_cache, v_cache, block_tables, context_lens, q_start, out, p,
                                                     std::min(max_query_len, total_q), static_cast<hipStream_t>(hip_stream));
        return e == hipSuccess ? KVC_OK : hip_failed(e);
    }
    if (!on_mfma) {
        // vector-ALU kernel, one query row per "sequence" of its grid, one partition, no workspace
        kvc::AttnParams vp = make_params(*desc, pl, scale);
        vp.num_seqs = total_q;
        vp.partition_tokens = 1 << 30;
        vp.max_partitions = 1;
        vp.head_chunk = kvc::valu_head_chunk(vp.group);
        vp.max_context_len = desc->max_blocks_per_seq * desc->block_size;
        const int64_t grid = int64_t(total_q) * (desc->num_q_heads / kvc::valu_head_chunk(vp.group));
        if (grid > kMaxGrid) return KVC_ERR_BAD_SHAPE;
        const hipError_t e = kvc::launch_prefill_valu(q, k_cache, v_cache, block_tables, context_lens, q_start,
                                                      desc->num_seqs, max_query_len, out, vp, desc->dtype,
                                                      desc->head_dim, int(grid), static_cast<hipStream_t>(hip_stream));
        return e == hipSuccess ? KVC_OK : hip_failed(e);
    }
    if (tile_grid > kMaxGrid) return KVC_ERR_BAD_SHAPE;
    // KVC_KERNEL_MFMA asks for the 16x16-tile kernel whatever the shape
    const bool tiles32 = desc->kernel != KVC_KERNEL_MFMA && kvc::prefill_tiles32(p);
    const hipError_t e = tiles32 ? kvc::launch_prefill_mfma32(q, k_cache, v_cache, block_tables, context_lens, q_start,
                                                              out, p, total_q, static_cast<hipStream_t>(hip_stream))
                                 : kvc::launch_prefill_mfma(q, k_cache, v_cache, block_tables, context_lens, q_start,
                                                            out, p, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? KVC_OK : hip_failed(e);
}

int kvc_kv_cache_append(const void *k_new, const void *v_new, void *k_cache, void *v_cache,
                        const int32_t *block_tables, const int32_t *positions,
                        const kvc_attn_desc *desc, void *hip_stream) {
    Plan pl;
    const int rc = make_plan(desc, &pl);
    if (rc != KVC_OK) return rc;
    if (desc->num_seqs == 0) return KVC_OK;
    if (!k_new || !v_new || !k_cache || !v_cache || !block_tables || !positions) return KVC_ERR_NULL;
    if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_cache) || !aligned16(v_cache))
        return KVC_ERR_ALIGN;
    const int row_bytes = desc->head_dim * (desc->dtype == KVC_F32 ? 4 : 2);
    const hipError_t e = kvc::launch_cache_append(
        k_new, v_new, k_cache, v_cache, block_tables, positions, desc->num_seqs, desc->num_kv_heads,
        row_bytes, ilog2(desc->block_size), desc->max_blocks_per_seq, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? KVC_OK : hip_failed(e);
}

int kvc_kv_block_copy(const kvc_pool *src, const kvc_pool *dst, const int64_t *block_mapping,
                      int64_t num_pairs, void *hip_stream) {
    const int rc = check_pools(src, dst, block_mapping, num_pairs);
    if (rc != KVC_OK) return rc;
    if (num_pairs == 0) return KVC_OK;
    const hipError_t e = kvc::launch_block_copy(*src, *dst, block_mapping, num_pairs,
                                                static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? KVC_OK : hip_failed(e);
}

int kvc_validate_block_mapping(const kvc_pool *src, const kvc_pool *dst,
                               const int64_t *block_mapping, int64_t num_pairs, void *hip_stream) {
    const int rc = check_pools(src, dst, block_mapping, num_pairs);
    if (rc != KVC_OK) return rc;
    if (num_pairs == 0) return KVC_OK;
    const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    std::vector<int64_t> map(size_t(num_pairs) * 2);
    hipError_t e = hipMemcpyAsync(map.data(), block_mapping, map.size() * sizeof(int64_t),
                                  hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return hip_failed(e);
    std::vector<int64_t> srcs(num_pairs), dsts(num_pairs);
    for (int64_t i = 0; i < num_pairs; ++i) {
        srcs[i] = map[2 * i];
        dsts[i] = map[2 * i + 1];
        if (srcs[i] < 0 || srcs[i] >= src->num_blocks || dsts[i] < 0 || dsts[i] >= dst->num_blocks)
            return KVC_ERR_BAD_INDEX;
    }
    std::sort(dsts.begin(), dsts.end());
    if (std::adjacent_find(dsts.begin(), dsts.end()) != dsts.end()) return KVC_ERR_DUPLICATE;
    // Pools that share memory: a block that is both read and written would race.
    const auto *sb = static_cast<const unsigned char *>(src->base);
    const auto *db = static_cast<const unsigned char *>(dst->base);
    const int64_t s_extent = (src->num_planes > 1 ? (src->num_planes - 1) * src->plane_stride_bytes : 0) +
                             src->num_blocks * src->block_bytes;
    const int64_t d_extent = (dst->num_planes > 1 ? (dst->num_planes - 1) * dst->plane_stride_bytes : 0) +
                             dst->num_blocks * dst->block_bytes;
    if (sb < db + d_extent && db < sb + s_extent) {
        if (sb != db) return KVC_ERR_OVERLAP;  // partially overlapping pools: no safe reading
        std::sort(srcs.begin(), srcs.end());
        for (int64_t s : srcs)
            if (std::binary_search(dsts.begin(), dsts.end(), s)) return KVC_ERR_OVERLAP;
    }
    return KVC_OK;
}

}  // extern "C"

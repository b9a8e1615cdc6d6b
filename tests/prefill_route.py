"""The library's own rules for prefill calls on 32x32 tiles (csrc/prefill_route.h), compiled for the host."""
import ctypes
import os
import subprocess

from paper_2503_13773_amd.build import CSRC

FIELDS = ("num_seqs", "num_q_heads", "num_kv_heads", "block_size", "max_blocks_per_seq", "max_query_tiles")

SHIM = r'''
#include "prefill_route.h"
using namespace kvc;
static PrefillParams params(const int *v) {
    PrefillParams p{};
    p.num_seqs = v[0], p.num_q_heads = v[1], p.num_kv_heads = v[2], p.block_size = v[3], p.max_blocks_per_seq = v[4];
    p.max_query_tiles = v[5], p.group = v[1] / v[2], p.heads_per_chunk = p.group % 2 == 0 ? 2 : 1;
    return p;
}
extern "C" {
int wide(const int *v, long long total_q) { return prefill_wide(params(v), total_q); }
int by_units(const int *v) { return prefill_by_units(params(v)); }
int tiles32(const int *v, float scale) { PrefillParams p = params(v); p.scale_log2e = scale; return prefill_tiles32(p); }
int split(const int *v) { return prefill_split(params(v)); }
int split_steps() { return kMinSplitSteps; }
int chunk(int b, int chunks, int sharing) { return chunk_at(b, chunk_spread(chunks, sharing)); }
void places(int blocks, int group, int kv_heads, int *out) {
    for (int b = 0; b < blocks; ++b) {
        const HeadPlace at = head_place(b, blocks, group, kv_heads);
        out[3 * b] = at.kv_head, out[3 * b + 1] = at.head, out[3 * b + 2] = at.index;
    }
}
}
'''


def build(folder):
    src, out = os.path.join(folder, "route.cpp"), os.path.join(folder, "route.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, src, "-o", out])
    return ctypes.CDLL(out)


def values(hq, hkv, qlens, table_tokens, bs=16):
    """The numbers a call is judged by, in the order of FIELDS."""
    return (ctypes.c_int * len(FIELDS))(len(qlens), hq, hkv, bs, -(-table_tokens // bs), -(-max(qlens) // 64))

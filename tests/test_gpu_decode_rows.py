"""Decode attention of few rows (a workgroup per piece of a row) against the fp64 oracle: lengths around the tile, the
eight wavefronts, the uncut length of 20 tiles and the pieces; every merge layout; schedules; the counters."""
import numpy as np
import pytest
import torch

import kvc_workloads as W
from gpu_util import BF16_TOL, out_bits, out_to_f64, to_device
from test_gpu_attention import _scheduled_equals_direct, custom
from test_gpu_prefill_d64 import bound, poison

pytestmark = pytest.mark.gpu


def check(w, oracle_mod, label, max_context_len=0):
    import paper_2503_13773_amd as K
    print(f"[case] rows {label} D={w.head_dim} nseq={w.num_seqs} max={w.max_context_len}", flush=True)
    rows = w.num_seqs * w.num_kv_heads
    # above the bound of the whole-row layout; the table has room for it
    tokens = max(max_context_len, w.max_context_len, 641 if w.head_dim == 64 else 513)
    w.block_tables = np.pad(w.block_tables, ((0, 0), (0, max(0, -(-tokens // w.block_size) - w.max_blocks_per_seq))), constant_values=-1)
    assert rows <= 128 and w.num_seqs <= 64 and rows ** 3 * tokens <= 1 << 31   # the line of the dispatch
    d = to_device(w)
    desc = K.attn_desc(d["q"], d["k"], d["tables"], max_context_len=tokens)
    ws = K.new_workspace(desc)
    outs = [K.paged_attention_decode(d["q"], d["k"], d["v"], d["tables"], d["lens"], w.scale, desc=desc, workspace=ws)
            for _ in range(4)]
    torch.cuda.synchronize()
    assert ws is None or int(ws[:4096].max()) == 0
    assert all(np.array_equal(out_bits(o), out_bits(outs[0])) for o in outs)
    got, ref = out_to_f64(outs[0]), oracle_mod.attention_of_workload(w, num_threads=8)
    assert np.isfinite(got).all()
    if w.head_dim == 64:
        assert (np.abs(got - ref) <= bound(ref)).all(), label
    else:
        assert np.abs(got - ref).max() <= BF16_TOL, label


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv,bs", [(8, 2, 16), (7, 1, 8), (16, 1, 32), (9, 1, 4), (12, 12, 16), (1, 1, 64), (6, 3, 256)])
def test_lengths_around_tiles_waves_and_pieces(oracle_mod, d, hq, hkv, bs):
    t = 32 if d == 64 else 16
    for lens in ([1, 0, t - 1, t, t + 1, 7 * t, 8 * t, 8 * t + 1], [20 * t, 0, 3], [20 * t + 1, 40, 0, 0], [16 * t, 17 * t + 5, 33 * t]):
        w = custom(900 + hq + bs + d, dtype=W.BF16, lens=lens, hq=hq, hkv=hkv, d=d, bs=bs)
        poison(w)
        check(w, oracle_mod, f"{hq}/{hkv} bs={bs} {lens}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens,hq,hkv", [([3217], 32, 8), ([40000], 4, 1), ([40000, 9], 2, 1), ([12000, 100, 0, 7000], 8, 4),
                                         ([900] * 8, 32, 16), ([300] * 64, 4, 2), ([0] * 5, 4, 2), ([250000], 1, 1)])
def test_many_pieces_and_full_grids(oracle_mod, d, lens, hq, hkv):
    """Up to 64 pieces per row, pieces longer than the 64 tiles staged per wavefront, 128 rows, no row at all."""
    check(custom(920 + len(lens) + d, dtype=W.BF16, lens=lens, hq=hq, hkv=hkv, d=d, bs=16), oracle_mod, f"{lens[:4]}")


# numbers of heads and sequences that the placement and the merge divide by: one to 128 KV heads, one piece to spare or
# none per KV head, groups of any size
@pytest.mark.parametrize("hq,hkv,lens", [(128, 128, [1000]), (86, 43, [700, 513]), (15, 3, [2000] * 7 + [33]), (65, 13, [900, 40, 600]), (11, 11, [600] * 11),
                                         (77, 7, [5000, 17]), (26, 2, [3000, 100, 0, 700, 650]), (127, 127, [600])])
def test_heads_and_sequences_of_any_number(oracle_mod, hq, hkv, lens):
    for d in (128, 64):
        check(custom(930 + hq + d, dtype=W.BF16, lens=lens, hq=hq, hkv=hkv, d=d, bs=16), oracle_mod, f"{hq}/{hkv} {lens[:4]}")


def test_bound_far_above_the_lengths(oracle_mod):
    w = custom(940, dtype=W.BF16, lens=[70, 300, 5], hq=8, hkv=2, d=128, bs=16, lmax=4096)
    check(w, oracle_mod, "loose", max_context_len=65536)


def test_schedules(oracle_mod):
    for lens, hq, hkv, bs in [([3217], 32, 8, 16), ([0, 300, 0, 320, 321, 17], 8, 2, 8), ([20000, 37, 9000], 2, 1, 16),
                              ([0, 0], 4, 2, 16), ([500] * 16, 32, 8, 32), ([100, 250], 16, 1, 4)]:
        w = custom(950 + len(lens) + bs, dtype=W.BF16, lens=lens, hq=hq, hkv=hkv, d=128, bs=bs)
        if max(lens) <= 512:
            w.context_lens[-1] = 513      # out of the whole-row layout
            w = custom(950 + len(lens) + bs, dtype=W.BF16, lens=w.context_lens, hq=hq, hkv=hkv, d=128, bs=bs)
        _scheduled_equals_direct(w, oracle_mod, f"rows {lens[:4]} bs={bs}")


def test_one_workspace_for_few_rows_and_many(oracle_mod):
    """Calls of both kinds in turn on one workspace: each leaves the counters at 0 for the next."""
    import paper_2503_13773_amd as K
    few = custom(960, dtype=W.BF16, lens=[3000, 70], hq=32, hkv=8, d=128, bs=16)
    many = W.make_config("cfg3", num_seqs=40, ctx_scale=0.3)
    ws, seen = None, {}
    for turn in range(6):
        for w in (few, many):
            d = seen.setdefault(id(w), (to_device(w), oracle_mod.attention_of_workload(w, num_threads=8)))
            desc = K.attn_desc(d[0]["q"], d[0]["k"], d[0]["tables"], max_context_len=w.max_context_len)
            ws = ws if ws is not None else K.new_workspace(desc)
            out = K.paged_attention_decode(d[0]["q"], d[0]["k"], d[0]["v"], d[0]["tables"], d[0]["lens"], w.scale,
                                           desc=desc, workspace=ws)
            assert np.abs(out_to_f64(out) - d[1]).max() <= BF16_TOL
    assert int(ws[:4096].max()) == 0


# small calls at head_dim 64 are the vector ALUs' under a tight bound; this one makes them pieces
LOOSE64 = 65536


def check_pieces64(w, oracle_mod, label):
    import paper_2503_13773_amd as K
    d = K.AttnDesc(w.num_seqs, w.num_q_heads, w.num_kv_heads, 64, w.block_size, -(-LOOSE64 // w.block_size), w.num_pool_blocks, K.KVC_BF16,
                   LOOSE64, 0, 0, 0)
    plan = K.attn_plan(d)
    assert plan.kernel == K.KERNEL_MFMA_BALANCED and plan.partial_grid == 256 and plan.partition_tokens == 8 * 32   # pieces
    check(w, oracle_mod, label, max_context_len=LOOSE64)


@pytest.mark.parametrize("hq,hkv,bs", [(8, 2, 16), (7, 1, 8), (16, 1, 32), (9, 1, 4), (4, 4, 16), (2, 1, 64), (6, 3, 256)])
def test_pieces_at_head_dim_64(oracle_mod, hq, hkv, bs):
    t = 32
    for lens in ([1, 0, t - 1, t, t + 1, 7 * t, 8 * t, 8 * t + 1], [20 * t, 0, 3], [20 * t + 1, 40, 0, 0], [16 * t, 17 * t + 5, 33 * t], [300] * 7,
                 [9000, 5]):
        w = custom(980 + hq + bs, dtype=W.BF16, lens=lens, hq=hq, hkv=hkv, d=64, bs=bs)
        poison(w)
        check_pieces64(w, oracle_mod, f"{hq}/{hkv} bs={bs} {lens}")


def test_non_finite_values_in_pieces_at_head_dim_64(oracle_mod):
    w = custom(990, dtype=W.BF16, lens=[700, 300, 400], hq=4, hkv=2, d=64, bs=16, lmax=LOOSE64 // 16)
    for n, t, h, dim, what in [(0, 50, 0, 3, 0x7F80), (0, 650, 1, 40, 0x7FC0), (1, 299, 0, 63, 0xFF80)]:
        w.v_cache[w.block_tables[n, t // 16], h, t % 16, dim] = what
    w.q[:, :, 0] = 0x3F80                                       # q[0] = 1
    w.k_cache[w.block_tables[2, :4], :, :, 0] = 0xFF80          # scores of -inf for the first 64 tokens of sequence 2
    print("[case] pieces d64 non-finite values", flush=True)
    import paper_2503_13773_amd as K
    d = to_device(w)
    with np.errstate(all="ignore"):
        ref = oracle_mod.attention_of_workload(w, num_threads=8)
        got = out_to_f64(K.paged_attention_decode(d["q"], d["k"], d["v"], d["tables"], d["lens"], w.scale, max_context_len=LOOSE64))
        fine = np.isfinite(ref)
        assert np.array_equal(np.isfinite(got), fine) and (np.abs(got - ref)[fine] <= bound(ref)[fine]).all()
        assert np.array_equal(got[~fine], ref[~fine], equal_nan=True)

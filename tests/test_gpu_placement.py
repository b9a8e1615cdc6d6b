"""Where workers are placed in batches that plan as ranges of flat tiles: batch sizes at the passes of the placement, block
sizes on both sides of a tile in schedules, and repeated launches of pieces.  The layout is asserted from the plan."""
import numpy as np
import pytest
import torch

import kvc_workloads as W
from gpu_util import BF16_TOL, out_bits, out_to_f64, to_device
from test_gpu_attention import BALANCED, _scheduled_equals_direct, custom
from test_gpu_decode_d64 import check as check64

pytestmark = pytest.mark.gpu


def plan_of(w, **opts):
    import paper_2503_13773_amd as K
    d = to_device(w)
    return K.attn_plan(K.attn_desc(d["q"], d["k"], d["tables"], **opts))


@pytest.mark.parametrize("nseq", [63, 64, 65, 255, 256, 257, 1023, 1024, 1025])
def test_ranges_over_many_short_sequences(oracle_mod, nseq):
    """Contexts of 0 to 80 tokens in ranges of at least four tiles: up to 256 sequences a worker is placed by a count over
    the prefix table, 64 entries per pass, beyond that by a binary search; up to 1024 the smaller prefix table."""
    import paper_2503_13773_amd as K
    lens = np.random.default_rng(1800 + nseq).integers(0, 81, nseq).astype(np.int32)
    w = custom(1800 + nseq, dtype=W.BF16, lens=lens, hq=8, hkv=2, d=128, bs=16)
    opts = dict(max_context_len=80, partition_tokens=64)
    plan = plan_of(w, **opts)
    assert (plan.kernel, plan.partial_grid, plan.partition_tokens) == (BALANCED, 256, 64)
    print(f"[case] ranges over {nseq} short sequences", flush=True)
    d = to_device(w)
    out = K.paged_attention_decode(d["q"], d["k"], d["v"], d["tables"], d["lens"], w.scale, **opts)
    torch.cuda.synchronize()
    assert np.abs(out_to_f64(out) - oracle_mod.attention_of_workload(w, num_threads=8)).max() <= BF16_TOL


@pytest.mark.parametrize("nseq", [63, 64, 65, 255, 256, 257, 1023, 1024, 1025])
@pytest.mark.parametrize("longest", [80, 400])          # a worker per row, and ranges that cross rows
def test_ranges_at_head_dim_64(oracle_mod, nseq, longest):
    lens = np.random.default_rng(1810 + nseq).integers(0, longest + 1, nseq).astype(np.int32)
    w = custom(1810 + nseq, dtype=W.BF16, lens=lens, hq=8, hkv=2, d=64, bs=16, lmax=4096)
    plan = plan_of(w, max_context_len=4096)
    assert (plan.kernel, plan.partial_grid, plan.partition_tokens) == (BALANCED, 256, 128)   # pieces would say 256
    check64(w, oracle_mod, f"{nseq} sequences of up to {longest}", max_context_len=4096)


@pytest.mark.parametrize("bs", [4, 8, 32])
@pytest.mark.parametrize("chunk", [16, 64])
def test_schedules_of_ranges_at_other_block_sizes(oracle_mod, bs, chunk):
    """Several units per tile and several units per block, in ranges that the schedule holds."""
    w = custom(1820 + bs, dtype=W.BF16, lens=[1, 3, 9, 17, 100, 257, 1000, 0, 2000], hq=8, hkv=2, d=128, bs=bs)
    plan = plan_of(w, max_context_len=w.max_context_len, kernel=BALANCED, partition_tokens=chunk)
    assert (plan.kernel, plan.partial_grid, plan.partition_tokens) == (BALANCED, 256, chunk)
    _scheduled_equals_direct(w, oracle_mod, f"bs={bs} chunk={chunk}", partition_tokens=chunk)


@pytest.mark.parametrize("d", [64, 128])
def test_pieces_merge_the_same_bits_launch_after_launch(d):
    """The partials of a row's pieces travel between workgroups on different XCDs inside one launch: 300 launches over
    rotating replicas (cold caches, another arrival order) must all give the bits of the first."""
    import paper_2503_13773_amd as K
    w = custom(1830 + d, dtype=W.BF16, lens=[9000, 700, 0, 12000, 3000, 1, 8000, 5000], hq=32, hkv=4, d=d, bs=16)
    plan = plan_of(w, max_context_len=w.max_context_len)
    assert (plan.kernel, plan.partial_grid, plan.partition_tokens) == (BALANCED, 256, 8 * (16 if d == 128 else 32))   # 8 tiles; ranges would say 384
    devs = [to_device(w) for _ in range(4)]
    desc = K.attn_desc(devs[0]["q"], devs[0]["k"], devs[0]["tables"], max_context_len=w.max_context_len)
    ws = K.new_workspace(desc)
    outs = [torch.empty_like(devs[0]["q"]) for _ in range(300)]
    for i, o in enumerate(outs):
        x = devs[i % 4]
        K.paged_attention_decode(x["q"], x["k"], x["v"], x["tables"], x["lens"], w.scale, o, desc=desc, workspace=ws)
    torch.cuda.synchronize()
    first = out_bits(outs[0])
    bad = [i for i, o in enumerate(outs) if not np.array_equal(out_bits(o), first)]
    assert not bad, bad[:10]
    assert int(ws[:4096].max()) == 0

"""Decode attention of short contexts (a workgroup per row) against the fp64 oracle: lengths around the tile and the four
wavefronts up to the bound, every block size (up to 64 units per wavefront), tables with no spare entry, groups around the
merge layouts, more rows than the device holds at once, schedules."""
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
    print(f"[case] whole rows {label} D={w.head_dim} nseq={w.num_seqs} max={w.max_context_len}", flush=True)
    d = to_device(w)
    desc = K.attn_desc(d["q"], d["k"], d["tables"], max_context_len=max_context_len or max(1, w.max_context_len))
    assert K.attn_plan(desc).partial_grid == w.num_seqs * w.num_kv_heads      # the layout under test
    ws = K.new_workspace(desc)
    outs = [K.paged_attention_decode(d["q"], d["k"], d["v"], d["tables"], d["lens"], w.scale, desc=desc, workspace=ws)
            for _ in range(2)]
    torch.cuda.synchronize()
    assert np.array_equal(out_bits(outs[0]), out_bits(outs[1]))
    got, ref = out_to_f64(outs[0]), oracle_mod.attention_of_workload(w, num_threads=8)
    assert np.isfinite(got).all()
    if w.head_dim == 64:
        assert (np.abs(got - ref) <= bound(ref)).all(), label
    else:
        assert np.abs(got - ref).max() <= BF16_TOL, label


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bs", [4, 8, 16, 32, 64, 256])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (7, 1), (16, 1), (5, 5)])
def test_edges(oracle_mod, d, bs, hq, hkv):
    t, cap = (32, 640) if d == 64 else (16, 512)
    lens = [cap, 0, 1, 2, 3, 4, 5, 15, 16, 17, t - 1, t, t + 1, 2 * t, 3 * t + 1, 4 * t, 4 * t + 1, 8 * t - 1, 12 * t + 5, cap - 1]
    w = custom(1200 + d + bs + hq, dtype=W.BF16, lens=lens, hq=hq, hkv=hkv, d=d, bs=bs, lmax=-(-cap // bs))
    poison(w)
    check(w, oracle_mod, f"{hq}/{hkv} bs={bs}")


@pytest.mark.parametrize("d,nseq,hkv,cap", [(64, 130, 1, 1024), (64, 17, 8, 1023), (128, 500, 4, 300), (128, 1000, 1, 90), (64, 1500, 2, 60)])
def test_many_rows(oracle_mod, d, nseq, hkv, cap):
    lens = np.random.default_rng(1250 + nseq).integers(0, cap + 1, nseq)
    lens[nseq // 2] = cap
    check(custom(1250 + nseq, dtype=W.BF16, lens=lens, hq=2 * hkv, hkv=hkv, d=d, bs=4 if cap > 1000 else 16), oracle_mod, f"{nseq} rows x {hkv}")


def test_bound_above_the_lengths_and_no_workspace(oracle_mod):
    check(custom(1290, dtype=W.BF16, lens=[70, 300, 5], hq=8, hkv=2, d=64, bs=16, lmax=60), oracle_mod, "loose", 600)


def test_schedules(oracle_mod):
    for lens, hq, hkv, bs in [([512, 0, 1, 300, 47], 32, 8, 16), ([0, 0], 4, 2, 16), ([100] * 300, 4, 2, 8), ([33, 500], 16, 1, 4),
                              ([511, 2], 8, 2, 64)]:
        w = custom(1295 + len(lens) + bs, dtype=W.BF16, lens=lens, hq=hq, hkv=hkv, d=128, bs=bs)
        _scheduled_equals_direct(w, oracle_mod, f"whole {lens[:4]} bs={bs}")

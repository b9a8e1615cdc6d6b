"""Scores of -inf (a K of -inf against a positive q) over whole tiles and partitions: they weigh nothing wherever these fall in
the split of the row, as long as some score of the row is finite.  Every layout and kernel against the fp64 oracle."""
import numpy as np
import pytest

import kvc_workloads as W
from gpu_util import BF16_TOL, out_to_f64, run_gpu
from test_gpu_attention import custom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opts", [dict(), dict(max_context_len=4096), dict(partition_tokens=64), dict(partition_tokens=16), dict(kernel=2),
                                  dict(kernel=1)], ids=["whole", "pieces", "ranges", "cut", "fixed", "valu"])
def test_tiles_of_minus_infinity(oracle_mod, opts):
    w = custom(1700, dtype=W.BF16, lens=[200, 500, 64, 333], hq=8, hkv=2, d=128, bs=16, lmax=256)
    w.q[:, :, 5] = 0x3F80                                                # q[5] = 1
    for n, tiles in enumerate([(1, 2, 6), (0, 5, 9, 30), (3,), range(0, 20)]):
        for t in tiles:
            w.k_cache[w.block_tables[n, t], :, :, 5] = 0xFF80            # -inf
    print(f"[case] decode scores of -inf {opts}", flush=True)
    with np.errstate(all="ignore"):
        ref = oracle_mod.attention_of_workload(w, num_threads=8)
    assert np.isfinite(ref).all()
    assert np.abs(out_to_f64(run_gpu(w, **opts)) - ref).max() <= BF16_TOL


@pytest.mark.parametrize("opts", [dict(max_context_len=640), dict(), dict(max_context_len=65536), dict(kernel=1, partition_tokens=64)],
                         ids=["whole", "valu", "pieces", "partitions"])
def test_head_dim_64(oracle_mod, opts):
    w = custom(1710, dtype=W.BF16, lens=[600, 500, 64, 333], hq=4, hkv=2, d=64, bs=16, lmax=4096)
    w.q[:, :, 5] = 0x3F80
    for n, tiles in enumerate([(1, 2, 6), range(0, 30), (3,), range(0, 20)]):
        for t in tiles:
            w.k_cache[w.block_tables[n, t], :, :, 5] = 0xFF80
    print(f"[case] decode d64 scores of -inf {opts}", flush=True)
    with np.errstate(all="ignore"):
        ref = oracle_mod.attention_of_workload(w, num_threads=8)
    assert np.isfinite(ref).all()
    assert np.abs(out_to_f64(run_gpu(w, **opts)) - ref).max() <= BF16_TOL

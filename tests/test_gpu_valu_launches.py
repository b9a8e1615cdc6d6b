"""The launch shapes of the vector-ALU attention kernel that the other files do not reach, against the fp64 oracle."""
import numpy as np
import pytest

import kvc_workloads as W
from gpu_util import F32_TOL, out_to_f64, run_gpu, tol_of
from test_gpu_attention import custom
from test_gpu_prefill import make, run
from test_gpu_prefill_d64 import reference

pytestmark = pytest.mark.gpu


# fp32 with two and four heads per workgroup: table entries ahead of their use up to 512 workgroups (rows x hq / heads) over
# tables of 512 tokens and more (make() adds a block to the longest context)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv,rows", [(8, 4, 128), (8, 4, 129), (8, 2, 256), (8, 2, 257)])
@pytest.mark.parametrize("longest,bs", [(479, 16), (495, 16), (510, 1), (511, 1), (700, 2)])
def test_prefill_of_two_and_four_heads(oracle_mod, d, hq, hkv, rows, longest, bs):
    lens, qlens = [longest, 33, longest - 1, 16, rows], [3, 2, rows - 25, 1, 19]
    w, q, qs = make(1600 + rows + longest + d, lens, qlens, hq, hkv, bs=bs, dtype=W.F32, d=d)
    for cache in (w.k_cache, w.v_cache):  # what no context covers is NaN
        covered = np.zeros((w.num_pool_blocks, bs), dtype=bool)
        for n, length in enumerate(lens):
            for t in range(length):
                covered[w.block_tables[n, t // bs], t % bs] = True
        cache.transpose(0, 2, 1, 3)[~covered] = np.nan
    print(f"[case] valu prefill f32 D={d} {hq}/{hkv} rows={rows} longest={longest} bs={bs}", flush=True)
    got, ref = out_to_f64(run(w, q, qs, max(qlens))), reference(oracle_mod, w, q, qs)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= F32_TOL


# more partials than a wavefront weighs at once: whole batches of eight and what is left, in the first 64 and behind
@pytest.mark.parametrize("dtype,d,kernel", [(W.F32, 64, 1), (W.F32, 128, 1), (W.BF16, 64, 1), (W.BF16, 128, 2)])
@pytest.mark.parametrize("cap", [1040, 1041, 1152, 1160, 2049, 3200])
def test_merges_of_many_partials(oracle_mod, dtype, d, kernel, cap):
    w = custom(1700 + cap + d, dtype=dtype, lens=[cap, 1025, 0, 16, 1024, 33], hq=6, hkv=2, d=d, bs=16)
    print(f"[case] merge of {cap / 16} partials {dtype} D={d} kernel={kernel}", flush=True)
    got = out_to_f64(run_gpu(w, kernel=kernel, partition_tokens=16, max_context_len=cap))
    assert np.abs(got - oracle_mod.attention_of_workload(w, num_threads=8)).max() <= tol_of(w)

"""kv_cache_append of more sequences than it gives a workgroup each: several per workgroup where their words are
few, bit-exact over both whole caches, at widths that do and do not divide a workgroup and a last one partly filled."""
import numpy as np
import pytest
import torch

import kvc_workloads as W
from gpu_util import dev_tensor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,hkv,nseq", [(W.BF16, 64, 1, 1025), (W.BF16, 64, 3, 1031), (W.BF16, 128, 2, 1100),
                                              (W.F32, 64, 1, 1027), (W.F32, 128, 1, 1024), (W.BF16, 128, 3, 1100)])
def test_many_sequences_of_few_words_append_bit_exactly(oracle_mod, dtype, d, hkv, nseq):
    import paper_2503_13773_amd as K
    print(f"[case] append {dtype} d={d} hkv={hkv} nseq={nseq}", flush=True)
    rng = np.random.default_rng(nseq + hkv)
    ctx = rng.integers(1, 50, nseq).astype(np.int32)
    w = W.build_workload("append-many", rng, dtype=dtype, context_lens=ctx, num_q_heads=hkv, num_kv_heads=hkv,
                         head_dim=d, block_size=16, max_blocks_per_seq=4, num_pool_blocks=None, occupancy=0.8)
    pos = (ctx - 1).astype(np.int32)
    pos[rng.random(nseq) < 0.2] = -1                       # skipped by request
    past = rng.random(nseq) < 0.05                         # skipped because the table has no entry for them
    host_pos = np.where(past, -1, pos).astype(np.int32)
    pos[past] = 4 * 16 + 3
    new = [rng.standard_normal((nseq, hkv, d)).astype(np.float32) for _ in "kv"]
    if dtype == W.BF16:
        new = [W.f32_to_bf16_bits(x) for x in new]
    wk, wv = w.k_cache.copy(), w.v_cache.copy()
    oracle_mod.kv_cache_append(*new, wk, wv, w.block_tables, host_pos)
    dk, dv = dev_tensor(w.k_cache, dtype), dev_tensor(w.v_cache, dtype)
    K.kv_cache_append(*(dev_tensor(x, dtype) for x in new), dk, dv,
                      torch.from_numpy(w.block_tables).cuda(), torch.from_numpy(pos).cuda())
    torch.cuda.synchronize()
    bits, np_bits = (torch.int16, np.int16) if dtype == W.BF16 else (torch.int32, np.int32)
    for got, want in ((dk, wk), (dv, wv)):
        assert np.array_equal(got.view(bits).cpu().numpy(), want.view(np_bits))

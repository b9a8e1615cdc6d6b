"""The vector-ALU decode kernel around its launch shapes: one head or several per workgroup (256 to 768 (head,
partition) pairs), four or sixteen wavefronts (256 workgroups), rows of 128, 256 and 512 bytes (sums over 8, 16 and 32 lanes)."""
import numpy as np
import pytest

import kvc_workloads as W
from gpu_util import out_to_f64, run_gpu, tol_of
from test_gpu_attention import custom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [(W.F32, 64), (W.F32, 128), (W.BF16, 64)])
@pytest.mark.parametrize("hq,hkv,nseq,cap", [(16, 4, 23, 256), (16, 4, 24, 256), (16, 4, 25, 256), (8, 8, 31, 240), (8, 8, 33, 240),
                                             (16, 2, 5, 1100), (6, 2, 3, 700), (1, 1, 1, 33), (12, 12, 22, 200)])
def test_launch_shapes(oracle_mod, dtype, d, hq, hkv, nseq, cap):
    rng = np.random.default_rng(1300 + nseq + cap)
    lens = rng.integers(0, cap + 1, nseq)
    lens[:3] = [cap, 1, 17][:nseq]
    w = custom(1300 + nseq, dtype=dtype, lens=lens, hq=hq, hkv=hkv, d=d, bs=16)
    print(f"[case] valu {dtype} D={d} {hq}/{hkv} nseq={nseq} cap={cap}", flush=True)
    got = out_to_f64(run_gpu(w, kernel=1, max_context_len=cap))
    assert np.isfinite(got).all()
    assert np.abs(got - oracle_mod.attention_of_workload(w, num_threads=8)).max() <= tol_of(w)


# two heads per KV head: 256 pairs where a row is 256 bytes or more, 384 below; four of bf16 and 128 in several partitions: 320
@pytest.mark.parametrize("dtype,d,hq,hkv,nseq,cap,limit", [
    (W.F32, 64, 16, 8, 16, 256, 256), (W.F32, 64, 16, 8, 17, 256, 256), (W.BF16, 128, 16, 8, 16, 256, 256), (W.BF16, 128, 16, 8, 17, 256, 256),
    (W.BF16, 64, 16, 8, 24, 256, 384), (W.BF16, 64, 16, 8, 25, 256, 384), (W.BF16, 128, 16, 4, 24, 256, 384), (W.BF16, 128, 16, 4, 10, 512, 320),
    (W.BF16, 128, 16, 4, 11, 512, 320), (W.BF16, 128, 12, 1, 16, 512, 384), (W.F32, 128, 16, 4, 12, 512, 384)])
def test_where_heads_part(oracle_mod, dtype, d, hq, hkv, nseq, cap, limit):
    import paper_2503_13773_amd as K
    lens = np.random.default_rng(1350 + nseq).integers(0, cap, nseq)
    w = custom(1350 + nseq + d, dtype=dtype, lens=lens, hq=hq, hkv=hkv, d=d, bs=16, lmax=512)
    code, parts = K.KVC_F32 if dtype == W.F32 else K.KVC_BF16, cap // 256
    plan = K.attn_plan(K.AttnDesc(nseq, hq, hkv, d, 16, 32, 64, code, cap, 0, 1, 0))
    chunk = {2: 2, 4: 4, 12: 4}[hq // hkv]
    assert plan.partial_grid == nseq * parts * (hq if nseq * hq * parts <= limit else hq // chunk)   # a head each, or several together
    print(f"[case] valu {dtype} D={d} {hq}/{hkv} nseq={nseq} cap={cap} of {limit} pairs", flush=True)
    got = out_to_f64(run_gpu(w, kernel=1, max_context_len=cap))
    assert np.abs(got - oracle_mod.attention_of_workload(w, num_threads=8)).max() <= tol_of(w)


# rows merged by their last partition (few partitions, or many rows, up to 64 and 1024) or by a launch of its own: the same bits
@pytest.mark.parametrize("dtype,d,hq,hkv,nseq,cap,pt", [
    (W.F32, 64, 4, 4, 3, 1024, 16), (W.F32, 64, 4, 4, 3, 1040, 16), (W.F32, 128, 16, 4, 5, 700, 16), (W.F32, 128, 8, 1, 30, 300, 32),
    (W.BF16, 64, 6, 2, 9, 500, 32), (W.BF16, 128, 4, 4, 7, 260, 16), (W.F32, 64, 8, 8, 128, 64, 16), (W.F32, 64, 8, 8, 129, 64, 16),
    (W.F32, 64, 32, 8, 40, 550, 0), (W.BF16, 64, 16, 16, 2, 5000, 0)])
def test_the_last_partition_merges_the_row(oracle_mod, dtype, d, hq, hkv, nseq, cap, pt):
    import paper_2503_13773_amd as K
    import torch
    from gpu_util import to_device
    lens = np.random.default_rng(1400 + nseq + cap).integers(0, cap + 1, nseq)
    lens[:4] = [cap, 0, 17, 16][:nseq]
    w = custom(1400 + nseq, dtype=dtype, lens=lens, hq=hq, hkv=hkv, d=d, bs=16)
    t = to_device(w)
    desc = K.attn_desc(t["q"], t["k"], t["tables"], max_context_len=cap, kernel=1, partition_tokens=pt)
    ws = K.new_workspace(desc)
    print(f"[case] valu merge {dtype} D={d} {hq}/{hkv} nseq={nseq} cap={cap} pt={pt}", flush=True)
    apart = torch.full_like(t["q"], float("nan"))
    K.paged_attention_decode_partial(t["q"], t["k"], t["v"], t["tables"], t["lens"], w.scale, apart, desc, ws)
    K.paged_attention_decode_merge(t["lens"], apart, desc, ws)
    assert np.abs(out_to_f64(apart) - oracle_mod.attention_of_workload(w, num_threads=8)).max() <= tol_of(w)
    for _ in range(5):
        ws[4096:].fill_(0xff)  # NaN in every slot: a partial fetched before it was written shows
        got = torch.full_like(t["q"], float("nan"))
        K.paged_attention_decode(t["q"], t["k"], t["v"], t["tables"], t["lens"], w.scale, got, desc=desc, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(got, apart)
        assert not ws[:4096].any()


@pytest.mark.parametrize("dtype,d,hq,hkv,nseq,cap", [(W.F32, 64, 16, 2, 24, 512), (W.F32, 64, 16, 2, 25, 512), (W.F32, 128, 64, 8, 12, 256),
                                                     (W.F32, 128, 64, 8, 13, 256), (W.BF16, 128, 32, 4, 8, 700), (W.BF16, 64, 8, 1, 33, 700)])
def test_where_eight_heads_part(oracle_mod, dtype, d, hq, hkv, nseq, cap):
    """Eight heads of a KV head together above 768 (head, partition) pairs."""
    import paper_2503_13773_amd as K
    lens = np.random.default_rng(1450 + nseq).integers(0, cap + 1, nseq)
    lens[0] = cap
    w = custom(1450 + nseq + d, dtype=dtype, lens=lens, hq=hq, hkv=hkv, d=d, bs=16, lmax=64)
    code, pairs = K.KVC_F32 if dtype == W.F32 else K.KVC_BF16, nseq * hq * -(-cap // 256)
    plan = K.attn_plan(K.AttnDesc(nseq, hq, hkv, d, 16, 64, 64, code, cap, 0, 1, 0))
    assert plan.partial_grid == (pairs if pairs <= 768 else pairs // 8)
    print(f"[case] valu eight heads {dtype} D={d} {hq}/{hkv} nseq={nseq} cap={cap}", flush=True)
    got = out_to_f64(run_gpu(w, kernel=1, max_context_len=cap))
    assert np.abs(got - oracle_mod.attention_of_workload(w, num_threads=8)).max() <= tol_of(w)

"""The launch shapes of the vector-ALU attention kernel that the other files do not reach, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import kvc_workloads as W
from gpu_util import F32_TOL, out_to_f64, run_gpu, to_device, tol_of
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


# the vector-ALU kernel merges a row itself (sequences x heads of a workgroup rows): up to 8 partitions, bf16 6, or from 32 rows, bf16
# 64, and never eight heads; both ways give the same bits, leave the counters zero, and can be captured
@pytest.mark.parametrize("dtype,d,hq,hkv,nseq,cap", [
    (W.F32, 64, 4, 4, 7, 128), (W.F32, 64, 4, 4, 7, 129), (W.F32, 64, 4, 4, 8, 129), (W.F32, 128, 8, 2, 31, 300), (W.F32, 128, 32, 8, 60, 300),
    (W.BF16, 64, 7, 1, 9, 96), (W.BF16, 64, 7, 1, 9, 97), (W.BF16, 64, 8, 8, 8, 97), (W.BF16, 64, 16, 2, 100, 64), (W.F32, 64, 16, 2, 100, 64)])
def test_who_merges_a_row(oracle_mod, dtype, d, hq, hkv, nseq, cap):
    import paper_2503_13773_amd as K
    lens = np.random.default_rng(1800 + nseq + cap).integers(0, cap + 1, nseq)
    lens[:4] = [cap, 17, 0, 16]
    w = custom(1800 + nseq + cap, dtype=dtype, lens=lens, hq=hq, hkv=hkv, d=d, bs=16)
    t = to_device(w)
    desc = K.attn_desc(t["q"], t["k"], t["tables"], max_context_len=cap, kernel=1, partition_tokens=16)
    ws = K.new_workspace(desc)
    print(f"[case] valu who merges {dtype} D={d} {hq}/{hkv} nseq={nseq} cap={cap}", flush=True)
    apart, got = torch.empty_like(t["q"]), torch.empty_like(t["q"])
    K.paged_attention_decode_partial(t["q"], t["k"], t["v"], t["tables"], t["lens"], w.scale, apart, desc, ws)
    K.paged_attention_decode_merge(t["lens"], apart, desc, ws)
    assert np.abs(out_to_f64(apart) - oracle_mod.attention_of_workload(w, num_threads=8)).max() <= tol_of(w)

    def call():
        K.paged_attention_decode(t["q"], t["k"], t["v"], t["tables"], t["lens"], w.scale, got, desc=desc, workspace=ws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for step in range(4):
        got.fill_(float("nan"))
        ws[4096:].fill_(0xff)  # NaN in every slot: a partial fetched before it was written shows
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, apart) and not ws[:4096].any(), step
        got.fill_(float("nan"))
        call()  # eager, between the replays
        torch.cuda.synchronize()
        assert torch.equal(got, apart) and not ws[:4096].any(), step
        t["q"].copy_(t["q"].flip(0))  # other inputs for the next replay
        K.paged_attention_decode_partial(t["q"], t["k"], t["v"], t["tables"], t["lens"], w.scale, apart, desc, ws)
        K.paged_attention_decode_merge(t["lens"], apart, desc, ws)
        torch.cuda.synchronize()


# eight tokens a lane group: fp32, a head per workgroup, up to 256 workgroups and partitions that sixteen wavefronts of four
# tokens a lane group do not cover (256 tokens of 64 dims, 128 of 128), which at 64 dims only the caller's own can be
@pytest.mark.parametrize("d,pt", [(64, 272), (64, 512), (64, 1024), (128, 144), (128, 512), (128, 1024)])
@pytest.mark.parametrize("cap", [272, 511, 512, 513, 1024, 1025, 3000])
def test_eight_tokens_a_lane_group(oracle_mod, d, pt, cap):
    w = custom(1900 + cap + d, dtype=W.F32, lens=[cap, cap - 1, 1, 0, 257, 17], hq=4, hkv=2, d=d, bs=8)
    for cache in (w.k_cache, w.v_cache):  # what no context covers is NaN
        covered = np.zeros((w.num_pool_blocks, 8), dtype=bool)
        for n, length in enumerate(w.context_lens.tolist()):
            for t in range(length):
                covered[w.block_tables[n, t // 8], t % 8] = True
        cache.transpose(0, 2, 1, 3)[~covered] = np.nan
    print(f"[case] valu eight tokens D={d} pt={pt} cap={cap}", flush=True)
    got = out_to_f64(run_gpu(w, kernel=1, partition_tokens=pt, max_context_len=cap))
    assert np.isfinite(got).all()
    assert np.abs(got - oracle_mod.attention_of_workload(w, num_threads=8)).max() <= tol_of(w)

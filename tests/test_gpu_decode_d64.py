"""Decode attention at head_dim 64 on the balanced matrix-core kernel (32-token tiles, weights kept to 16 bits) against
the fp64 oracle.  Tolerance as in test_gpu_prefill_d64: one rounding of the output to bf16 plus weights that enter the
product as two bf16 values (2^-16 relative each)."""
import numpy as np
import pytest
import torch

import kvc_workloads as W
from gpu_util import out_bits, out_to_f64, run_gpu, to_device
from test_gpu_attention import custom
from test_gpu_prefill_d64 import bound, poison

pytestmark = pytest.mark.gpu

VALU, BALANCED = 1, 4


def check(w, oracle_mod, label, max_context_len=0):
    """Bound 0: enough tokens for a large batch's kernel (the table has room for it)."""
    import paper_2503_13773_amd as K
    print(f"[case] decode d64 {label} nseq={w.num_seqs} max={w.max_context_len}", flush=True)
    rows = w.num_seqs * w.num_kv_heads
    bound_tokens = max_context_len or max(w.max_context_len, 1025, -(-(1 << 17) // rows), (1 << 31) // rows ** 3 + 1)
    w.block_tables = np.pad(w.block_tables, ((0, 0), (0, max(0, -(-bound_tokens // w.block_size) - w.max_blocks_per_seq))),
                            constant_values=-1)
    d = to_device(w)
    desc = K.attn_desc(d["q"], d["k"], d["tables"], max_context_len=bound_tokens)
    assert K.attn_plan(desc).kernel == BALANCED and K.attn_plan(desc).merge_grid == 0
    ws = K.new_workspace(desc)
    got = [K.paged_attention_decode(d["q"], d["k"], d["v"], d["tables"], d["lens"], w.scale, desc=desc, workspace=ws)
           for _ in range(3)]
    torch.cuda.synchronize()
    assert int(ws[:4096].max()) == 0
    assert all(np.array_equal(out_bits(g), out_bits(got[0])) for g in got)
    ref = oracle_mod.attention_of_workload(w, num_threads=8)
    got = out_to_f64(got[0])
    assert np.isfinite(got).all()
    assert (np.abs(got - ref) <= bound(ref)).all(), label


EDGES = [0, 1, 15, 16, 17, 31, 32, 33, 0, 63, 64, 65, 95, 96, 97, 127, 128, 129, 300, 511, 513, 1000, 2049]


# groups around the 4, 8 and 16 heads of the three merge layouts; blocks from 4 tokens (8 units per tile) to 256
@pytest.mark.parametrize("hq,hkv,bs", [(8, 2, 16), (32, 8, 16), (14, 2, 8), (3, 1, 32), (4, 4, 4), (16, 1, 16), (9, 1, 64),
                                       (5, 1, 256), (12, 12, 16)])
def test_shapes_and_edges(oracle_mod, hq, hkv, bs):
    w = custom(800 + hq + bs, dtype=W.BF16, lens=EDGES, hq=hq, hkv=hkv, d=64, bs=bs)
    poison(w)
    check(w, oracle_mod, f"{hq}/{hkv} bs={bs}")


@pytest.mark.parametrize("lens", [[3000], [20000, 5], [257], [40, 70], [0, 0, 300]])
def test_few_sequences(oracle_mod, lens):
    """Rows cut over many wavefronts, and a bound far above the lengths."""
    check(custom(830 + len(lens), dtype=W.BF16, lens=lens, hq=4, hkv=2, d=64, bs=16), oracle_mod, f"{lens}")


@pytest.mark.parametrize("nseq", [255, 257, 1100, 4096])
def test_many_sequences(oracle_mod, nseq):
    lens = np.random.default_rng(840 + nseq).integers(0, 90, nseq)
    lens[3] = 280
    check(custom(840 + nseq, dtype=W.BF16, lens=lens, hq=4, hkv=2, d=64, bs=16), oracle_mod, f"{nseq} short")


def test_long_ranges_per_wavefront(oracle_mod):
    """A bound of 320000 tokens makes a wavefront take at least 313 tiles: more than the 256 staged at a time."""
    check(custom(850, dtype=W.BF16, lens=[9000, 17000, 33], hq=2, hkv=1, d=64, bs=16), oracle_mod, "long ranges",
          max_context_len=320000)


@pytest.mark.parametrize("bound_tokens", [700, 1 << 24])   # pieces / ranges of flat tiles
def test_non_finite_values(oracle_mod, bound_tokens):
    """Inf / NaN in V reach their dim of their sequence with the sign they have, scores of -inf weigh nothing."""
    w = custom(860, dtype=W.BF16, lens=[700, 300, 400], hq=4, hkv=2, d=64, bs=16, lmax=1 << 20)
    bits = {"inf": 0x7F80, "-inf": 0xFF80, "nan": 0x7FC0}
    for n, t, h, dim, what in [(0, 50, 0, 3, "inf"), (0, 650, 1, 40, "nan"), (1, 299, 0, 63, "-inf")]:
        w.v_cache[w.block_tables[n, t // 16], h, t % 16, dim] = bits[what]
    w.q[:, :, 0] = 0x3F80                                # q[0] = 1
    w.k_cache[w.block_tables[2, :4], :, :, 0] = bits["-inf"]   # the first 64 tokens of sequence 2
    print("[case] decode d64 non-finite values", flush=True)
    with np.errstate(all="ignore"):
        got, ref = out_to_f64(run_gpu(w, max_context_len=bound_tokens)), oracle_mod.attention_of_workload(w, num_threads=8)
        fine = np.isfinite(ref)
        assert 0.5 < fine.mean() < 1.0 and np.array_equal(np.isfinite(got), fine)
        assert (np.abs(got - ref)[fine] <= bound(ref)[fine]).all()
        assert np.array_equal(got[~fine], ref[~fine], equal_nan=True)

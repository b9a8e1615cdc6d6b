"""Causal multi-query attention at head_dim 64 (32x32 matrix-core tiles, weights kept to 16 bits) against the
fp64 oracle.

Tolerance: the output is one rounding to bf16 (2^-9 relative) of a value whose own error is that of fp32 sums and of
weights that enter the product as two bf16 values (2^-16 relative each, so at most 2^-16 * max|V|, with |V| < 6 here:
9e-5).  2^-8 |ref| + 2e-4 covers both twice over."""
import numpy as np
import pytest
import torch

import kvc_workloads as W
from gpu_util import dev_tensor, out_to_f64
from test_gpu_prefill import make, run

pytestmark = pytest.mark.gpu


def bound(ref):
    return np.abs(ref) * 2.0 ** -8 + 2e-4


def reference(oracle_mod, w, q, qs):
    return oracle_mod.paged_attention_prefill(q, w.k_cache, w.v_cache, w.block_tables, w.context_lens, qs, w.scale,
                                              dtype=w.dtype, num_threads=8)


def poison(w):
    """NaN in every slot of the pools that no context covers."""
    bs = w.block_size
    covered = np.zeros((w.num_pool_blocks, bs), dtype=bool)
    for n, length in enumerate(w.context_lens.tolist()):
        for t in range(length):
            covered[w.block_tables[n, t // bs], t % bs] = True
    for cache in (w.k_cache, w.v_cache):
        cache.transpose(0, 2, 1, 3)[~covered] = np.uint16(0x7FC0)


# steps of 64 tokens in halves of 32, column sets of 16 or 32 rows, workgroups of 64 or 128 rows; groups of every
# kind (even: two heads per wavefront, odd: one; above 16), blocks below and above the 8 rows of one load
@pytest.mark.parametrize("hq,hkv,bs", [(8, 2, 16), (32, 8, 16), (14, 2, 8), (3, 1, 32), (4, 4, 16), (40, 2, 16), (8, 2, 1),
                                       (8, 4, 2), (6, 2, 4), (8, 2, 64), (8, 2, 256)])
def test_matches_oracle(oracle_mod, hq, hkv, bs):
    lens = [1, 31, 32, 33, 63, 64, 65, 97, 127, 128, 129, 200, 257, 450, 300, 700]
    qlens = [1, 31, 32, 33, 63, 64, 65, 97, 17, 128, 1, 130, 257, 16, 0, 33]
    w, q, qs = make(700 + hq + bs, lens, qlens, hq, hkv, bs=bs, d=64)
    poison(w)
    print(f"[case] prefill d64 {hq}/{hkv} bs={bs}", flush=True)
    got = out_to_f64(run(w, q, qs, max(qlens)))
    ref = reference(oracle_mod, w, q, qs)
    assert np.isfinite(got).all()
    assert (np.abs(got - ref) <= bound(ref)).all()


@pytest.mark.parametrize("rows", [1, 2])
def test_one_and_two_query_rows(oracle_mod, rows):
    """One row per sequence stays on the vector ALUs, from two on the matrix cores take the call."""
    lens = [2, 64, 65, 500, 1000]
    w, q, qs = make(750 + rows, lens, [rows] * 5, 8, 2, d=64)
    print(f"[case] prefill d64 rows={rows}", flush=True)
    got, ref = out_to_f64(run(w, q, qs, rows)), reference(oracle_mod, w, q, qs)
    assert (np.abs(got - ref) <= bound(ref)).all()


@pytest.mark.parametrize("scale", [0.0, -0.125, 3.0, 40.0])
def test_scales(oracle_mod, scale):
    """Any finite scale: zero (a plain mean), negative, and scores far outside the range of the weights."""
    import dataclasses
    w, q, qs = make(760, [150, 64, 333], [150, 20, 333], 8, 2, d=64)
    w = dataclasses.replace(w, scale=scale)
    print(f"[case] prefill d64 scale={scale}", flush=True)
    got = out_to_f64(run(w, q, qs, 333))
    ref = reference(oracle_mod, w, q, qs)
    # a score of magnitude s has an absolute error of about s * 2^-22 in fp32, relative error of its weight
    big = abs(scale) * float(np.abs(W.bf16_bits_to_f32(q)).max()) * 64 * 4
    assert (np.abs(got - ref) <= bound(ref) + 6 * big * 2.0 ** -22).all()


def test_rows_past_the_callers_bound_are_not_computed(oracle_mod):
    import paper_2503_13773_amd as K
    w, q, qs = make(770, [200, 90], [200, 90], 4, 2, d=64)
    out = torch.full((290, 4, 64), 7.0, dtype=torch.bfloat16, device="cuda")
    K.paged_attention_prefill(dev_tensor(q, w.dtype), dev_tensor(w.k_cache, w.dtype), dev_tensor(w.v_cache, w.dtype),
                              torch.from_numpy(w.block_tables).cuda(), torch.from_numpy(w.context_lens).cuda(),
                              torch.from_numpy(qs).cuda(), w.scale, 100, out)
    got, ref = out_to_f64(out), reference(oracle_mod, w, q, qs)
    seen = np.zeros(290, dtype=bool)
    seen[:100] = seen[200:] = True
    assert (np.abs(got - ref)[seen] <= bound(ref)[seen]).all()
    assert (got[~seen] == 7.0).all()


def test_infinities_stay_with_the_rows_that_see_them(oracle_mod):
    """Inf / NaN in V at a token reaches the rows at and after it (in that dim) and none before; a K row whose
    scores are -inf weighs nothing, also when it is all a row has seen in its first tokens."""
    lens = [100, 170]
    w, q, qs = make(780, lens, lens, 4, 2, d=64)
    bits = {"inf": 0x7F80, "-inf": 0xFF80, "nan": 0x7FC0}
    for n, t, h, dim, what in [(0, 50, 0, 3, "inf"), (0, 99, 1, 40, "nan"), (1, 64, 0, 63, "-inf"), (1, 169, 1, 0, "inf"),
                               (1, 33, 1, 17, "nan")]:
        w.v_cache[w.block_tables[n, t // 16], h, t % 16, dim] = bits[what]
    q[:, :, 0] = 0x3F80                                        # q[0] = 1
    w.k_cache[w.block_tables[1, 3], 0, 5, 0] = bits["-inf"]    # token 53 of sequence 1, KV head 0
    print("[case] prefill d64 non-finite values", flush=True)
    with np.errstate(all="ignore"):
        got, ref = out_to_f64(run(w, q, qs, max(lens))), reference(oracle_mod, w, q, qs)
        fine = np.isfinite(ref)
        assert 0.5 < fine.mean() < 1.0
        assert np.array_equal(np.isfinite(got), fine)
        assert (np.abs(got - ref)[fine] <= bound(ref)[fine]).all()
        assert np.array_equal(got[~fine], ref[~fine], equal_nan=True)


@pytest.mark.parametrize("hq,hkv,bs", [(8, 2, 16), (3, 1, 8), (8, 2, 64), (4, 2, 4)])
def test_windows_of_row_places(oracle_mod, hq, hkv, bs):
    """The places of 64 steps (4096 tokens) are looked up at once, and a turn asks four steps ahead: contexts that end around
    the points where the next 64 are fetched, and in the second and third window."""
    lens = [4096 - 256, 4096 - 255, 4095, 4096, 4097, 4096 + 257, 8192 - 192, 8193, 9000]
    qlens = [40, 70, 33, 64, 65, 40, 130, 20, 90]
    w, q, qs = make(770 + bs, lens, qlens, hq, hkv, bs=bs, d=64)
    poison(w)
    print(f"[case] prefill d64 windows {hq}/{hkv} bs={bs}", flush=True)
    got, ref = out_to_f64(run(w, q, qs, max(qlens))), reference(oracle_mod, w, q, qs)
    assert np.isfinite(got).all()
    assert (np.abs(got - ref) <= bound(ref)).all()


def test_reference_point_moves_in_every_turn(oracle_mod):
    """Scores that rise along the context move the reference point of the weights again and again, by less and by more than
    the weights of a step can hold, in turns that hold the scores of two steps."""
    for up in (0.02, 1.0, 40.0):
        w, q, qs = make(780, [700, 333], [700, 40], 4, 2, d=64)
        bits = lambda x: (np.ascontiguousarray(x, np.float32).view(np.uint32) >> 16).astype(np.uint16)
        q[...] = bits(np.full(q.shape, 1.0))
        for n, length in enumerate(w.context_lens.tolist()):
            for t in range(length):
                w.k_cache[w.block_tables[n, t // w.block_size], :, t % w.block_size] = bits(np.full((2, 64), up * t / 64))
        print(f"[case] prefill d64 rising {up}", flush=True)
        got, ref = out_to_f64(run(w, q, qs, 700)), reference(oracle_mod, w, q, qs)
        # a score of magnitude s has an absolute error of about s * 2^-22 in fp32, relative error of its weight
        assert (np.abs(got - ref) <= bound(ref) + 6 * (up * 700) * w.scale * 2.0 ** -22 * 4).all()

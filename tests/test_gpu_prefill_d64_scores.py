"""Scores and weights of head_dim 64 prefill at the ends of their ranges: reference points beyond 2^20, where the product of a
score and the scale is rounded before the reference point is taken off, and sums of weights far below their total."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_util import out_to_f64
from test_gpu_prefill import make, run
from test_gpu_prefill_d64 import bound, reference

pytestmark = pytest.mark.gpu


def bits(x):
    return (np.ascontiguousarray(x, np.float32).view(np.uint32) >> 16).astype(np.uint16)


# Scores so far apart that a token weighs 1 or nothing; those of one level are exact ties.  Against the heads of positive q the
# reference point starts beyond 2^20 in magnitude, comes inside, and leaves again, in steps that every column of a wavefront sees whole and
# in such that the causal mask cuts; against those of negative q it is outside from the first token on.  Inside, where a product with
# the scale is not rounded by itself, the levels are powers of two (the product is exact); outside they are not.
FRACTION = 1.6875
LEVELS = [-FRACTION * 2 ** 30, -FRACTION * 2 ** 24, -1.5 * 2 ** 22, -2.0 ** 12, 8.0, 2.0 ** 12, 2.0 ** 20, FRACTION * 2 ** 23,
          FRACTION * 2 ** 26, FRACTION * 2 ** 33]


@pytest.mark.parametrize("scale", [0.125, -0.125, 0.37, 1e5, -1e5])
@pytest.mark.parametrize("hq,hkv,bs", [(4, 2, 16), (3, 1, 8), (4, 1, 4)])
@pytest.mark.parametrize("segment", [29, 64, 101])
def test_reference_points_beyond_2_to_the_20(oracle_mod, scale, hq, hkv, bs, segment):
    lens = [700, 333, 1100, 64]
    qlens = [700, 40, 300, 64]
    w, q, qs = make(790 + segment + bs, lens, qlens, hq, hkv, bs=bs, d=64)
    w = dataclasses.replace(w, scale=scale)
    q[...] = 0
    q[:, :, 0] = bits(np.where(np.arange(hq) % 2 == 0, 1.0, -1.0))
    for n, length in enumerate(lens):
        for t in range(length):
            w.k_cache[w.block_tables[n, t // bs], :, t % bs, 0] = bits(LEVELS[min(t // segment, len(LEVELS) - 1)])
    print(f"[case] prefill d64 beyond 2^20 scale={scale} {hq}/{hkv} bs={bs} segment={segment}", flush=True)
    got, ref = out_to_f64(run(w, q, qs, max(qlens))), reference(oracle_mod, w, q, qs)
    assert np.isfinite(got).all()
    assert (np.abs(got - ref) <= bound(ref)).all()


def test_many_small_weights_reach_the_sum():
    """2^23 tokens that weigh 2^-26 beside four that weigh 1: a pair of them is lost on a running sum of 1 (half an ulp is 2^-24),
    the sixteen of a lane's step are not.  Tokens 0, 4, 32 and 36 weigh 1, one for every lane that sums a column, their V is 0, that of
    all others 1; the output is one rounding to bf16 (2^-9) of S / (4 + S)."""
    import paper_2503_13773_amd as K
    bs, blocks, hq = 256, 1 << 15, 4
    k = torch.zeros((2, 1, bs, 64), dtype=torch.bfloat16, device="cuda")
    v = torch.ones_like(k)
    k[:, :, :, 0] = -26.0
    for t in (0, 4, 32, 36):
        k[0, :, t, 0] = 0.0
        v[0, :, t] = 0.0
    q = torch.zeros((2, hq, 64), dtype=torch.bfloat16, device="cuda")
    q[:, :, 0] = 1.0
    tables = torch.ones((1, blocks), dtype=torch.int32, device="cuda")
    tables[0, 0] = 0
    lens = torch.tensor([bs * blocks], dtype=torch.int32, device="cuda")
    starts = torch.tensor([0, 2], dtype=torch.int32, device="cuda")
    print(f"[case] prefill d64 small weights, {bs * blocks} tokens", flush=True)
    got = out_to_f64(K.paged_attention_prefill(q, k, v, tables, lens, starts, float(np.float32(np.log(2.0))), 2))
    for row in range(2):
        small = (bs * blocks - 1 + row - 4) * 2.0 ** -26
        ref = small / (4 + small)
        assert np.abs(got[row] - ref).max() <= ref * 2.0 ** -8

"""Scores and weights of head_dim 64 prefill at the ends of their ranges: reference points beyond 2^20, where the product of a
score and the scale is rounded before the reference point is taken off."""
import dataclasses

import numpy as np
import pytest

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

"""Long requests: the prefill kernel of 64-column wavefronts (four query heads and 64 query rows per workgroup), against
attention in float64 on the dense sequence.

Sizes are near the lines between which that kernel takes a call, with row counts that leave wavefronts with part of
their rows or none, contexts longer than the rows, blocks of 4 to 256 tokens, and NaN wherever no context reaches.

Tolerance: weights are rounded to bf16 (2^-9 relative, with |V| < 6 at most 0.012) and so is the output (2^-9 relative)."""
import math

import numpy as np
import pytest
import torch

import kvc_workloads as W
from gpu_util import BF16_TOL, dev_tensor, out_to_f64
from test_gpu_prefill import make, run
from test_gpu_prefill_d64 import poison

pytestmark = pytest.mark.gpu


# (query heads, KV heads, contexts, query rows, block size); a test on the host asks the library whether they take this kernel
SHAPES = [(64, 8, [1985], [1985], 16), (64, 8, [2111], [1999], 4), (64, 4, [2049], [2040], 8),
          (64, 8, [2301, 2000, 1990, 1500, 33], [2000, 2000, 1990, 1500, 33], 64),
          (32, 8, [3457], [3457], 16), (32, 8, [3601], [3490], 2), (48, 4, [2321], [2321], 256)]
SPECIAL = (64, 8, [2000])


def exact(w, q, qs):
    qd, k, v = (dev_tensor(x, w.dtype) for x in (q, w.k_cache, w.v_cache))
    out = np.zeros(q.shape)
    group = w.num_q_heads // w.num_kv_heads
    for n, S in enumerate(w.context_lens.tolist()):
        rows = int(qs[n + 1] - qs[n])
        ids = torch.from_numpy(w.block_tables[n, :-(-S // w.block_size)].astype(np.int64)).cuda()
        for h in range(w.num_kv_heads):
            kd, vd = (x[ids, h].reshape(-1, x.shape[3])[:S].double() for x in (k, v))
            hidden = torch.arange(S, device="cuda")[None] > torch.arange(S - rows, S, device="cuda")[:, None]
            for g in range(group):
                score = qd[int(qs[n]):int(qs[n + 1]), h * group + g].double() @ kd.t().contiguous() * w.scale
                out[int(qs[n]):int(qs[n + 1]), h * group + g] = (
                    torch.softmax(score.masked_fill(hidden, -math.inf), dim=1) @ vd).cpu().numpy()
    return out


def check(w, q, qs, qlens, what):
    print(f"[case] prefill wide {what}", flush=True)
    got = out_to_f64(run(w, q, qs, max(qlens)))
    ref = exact(w, q, qs)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= BF16_TOL


@pytest.mark.parametrize("hq,hkv,lens,qlens,bs", SHAPES)
def test_matches_float64(hq, hkv, lens, qlens, bs):
    w, q, qs = make(1300 + hq + bs, lens, qlens, hq, hkv, bs=bs)
    poison(w)
    check(w, q, qs, qlens, f"{hq}/{hkv} {lens} {qlens} bs={bs}")


def test_scores_that_keep_growing_move_the_reference_point():
    """Every few steps the largest score so far is passed by more than the reference point allows, in all columns."""
    hq, hkv, lens = SPECIAL
    w, q, qs = make(1350, lens, lens, hq, hkv)
    q[:, :, 1] = 0x3F80                                   # q[1] = 1
    ramp = np.linspace(-40.0, 40.0, lens[0]).astype(np.float32)
    for t in range(lens[0]):
        w.k_cache[w.block_tables[0, t // 16], :, t % 16, 1] = W.f32_to_bf16_bits(ramp[t:t + 1] * 8)[0]
    check(w, q, qs, lens, "ramp")


def test_scores_of_minus_infinity_weigh_nothing():
    """The first two steps' scores are -inf in every column, and single ones later."""
    hq, hkv, lens = SPECIAL
    w, q, qs = make(1360, lens, lens, hq, hkv)
    q[:, :, 0] = 0x3F80
    for t in [*range(64), 100, 511, 999]:
        w.k_cache[w.block_tables[0, t // 16], :, t % 16, 0] = 0xFF80
    print("[case] prefill wide -inf", flush=True)
    got, ref = out_to_f64(run(w, q, qs, lens[0]))[64:], exact(w, q, qs)[64:]  # earlier rows see nothing else
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= BF16_TOL

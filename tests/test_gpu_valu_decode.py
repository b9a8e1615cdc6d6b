"""The vector-ALU decode kernel around its launch shapes: one head or several per workgroup (384 (head, partition)
pairs), four or sixteen wavefronts (256 workgroups), rows of 128, 256 and 512 bytes (sums over 8, 16 and 32 lanes)."""
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

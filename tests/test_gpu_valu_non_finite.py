"""Infinities in V at the last token of a context on the vector ALUs: lanes without a token load that one again, with a weight
of 0, and must not turn it into NaN.  Decode and prefill, rows of 128, 256 and 512 bytes, against the fp64 oracle."""
import numpy as np
import pytest

import kvc_workloads as W
from gpu_util import out_to_f64, run_gpu, tol_of
from test_gpu_attention import custom
from test_gpu_prefill import make, run

pytestmark = pytest.mark.gpu

LENS = [1, 5, 31, 32, 33, 130, 257, 600]


def put_infinities(w):
    """-inf in one dim of the last token's V of every sequence, +inf in another; what a row's ref then holds follows."""
    neg, pos = (np.uint16(0xFF80), np.uint16(0x7F80)) if w.dtype == W.BF16 else (-np.inf, np.inf)
    for n, length in enumerate(w.context_lens.tolist()):
        block, slot = w.block_tables[n, (length - 1) // w.block_size], (length - 1) % w.block_size
        w.v_cache[block, :, slot, 7] = neg
        w.v_cache[block, :, slot, 41] = pos


def compare(got, ref, tol):
    assert np.array_equal(np.isfinite(got), np.isfinite(ref)) and not np.isfinite(ref).all()
    fine = np.isfinite(ref)
    assert np.abs(got - ref)[fine].max() <= tol
    assert np.array_equal(got[~fine], ref[~fine])


@pytest.mark.parametrize("dtype,d", [(W.BF16, 64), (W.BF16, 128), (W.F32, 64), (W.F32, 128)])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (3, 3)])
def test_decode(oracle_mod, dtype, d, hq, hkv):
    w = custom(1500 + d + hq, dtype=dtype, lens=LENS, hq=hq, hkv=hkv, d=d, bs=16)
    put_infinities(w)
    print(f"[case] valu infinities decode {dtype} D={d} {hq}/{hkv}", flush=True)
    with np.errstate(all="ignore"):
        compare(out_to_f64(run_gpu(w, kernel=1)), oracle_mod.attention_of_workload(w, num_threads=8), tol_of(w))


@pytest.mark.parametrize("dtype,d,hq,hkv", [(W.BF16, 64, 3, 3), (W.F32, 64, 8, 2), (W.F32, 128, 3, 3)])
def test_prefill(oracle_mod, dtype, d, hq, hkv):
    w, q, qs = make(1520 + d + hq, LENS, [1, 2, 2, 1, 2, 2, 2, 2], hq, hkv, dtype=dtype, d=d)
    put_infinities(w)
    print(f"[case] valu infinities prefill {dtype} D={d} {hq}/{hkv}", flush=True)
    with np.errstate(all="ignore"):
        ref = oracle_mod.paged_attention_prefill(q, w.k_cache, w.v_cache, w.block_tables, w.context_lens, qs, w.scale, dtype=dtype,
                                                 num_threads=8)
        compare(out_to_f64(run(w, q, qs, 2)), ref, tol_of(w))

"""Which prefill calls at head_dim 64 take the matrix-core kernel and which the vector ALUs: both sides of every line of
the rule against the fp64 oracle, the tolerance as in test_gpu_prefill_d64."""
import numpy as np
import pytest

import kvc_workloads as W  # noqa: F401
from gpu_util import out_to_f64
from test_gpu_prefill import make, run
from test_gpu_prefill_d64 import bound, poison, reference

pytestmark = pytest.mark.gpu


def check(oracle_mod, lens, qlens, hq, hkv, max_q, label):
    w, q, qs = make(1400 + len(lens) + hq, lens, qlens, hq, hkv, d=64)
    poison(w)
    print(f"[case] prefill d64 {label} {hq}/{hkv} nseq={len(lens)} rows={sum(qlens)} max={max_q}", flush=True)
    got, ref = out_to_f64(run(w, q, qs, max_q)), reference(oracle_mod, w, q, qs)
    assert (np.abs(got - ref) <= bound(ref)).all(), label     # not for NaN either


@pytest.mark.parametrize("max_q", [8128, 8192])   # just below and at 2^32 threads for 4096 sequences of 16 head pairs
def test_many_sequences_with_a_loose_bound(oracle_mod, max_q):
    lens = np.random.default_rng(1410).integers(2, 9, 4096).tolist()
    qlens = [2] * 4095 + [1]
    check(oracle_mod, lens, qlens, 32, 8, max_q, "loose bound")

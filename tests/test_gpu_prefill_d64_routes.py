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


# one or two heads per workgroup of the vector ALUs, rows x heads at and above 512
@pytest.mark.parametrize("hq,hkv,rows", [(8, 8, 64), (8, 8, 65), (7, 1, 73), (7, 1, 74), (16, 8, 32), (16, 8, 33), (6, 1, 85), (6, 1, 86)])
def test_small_launches(oracle_mod, hq, hkv, rows):
    check(oracle_mod, [rows + 130, 3], [rows - 1, 1], hq, hkv, rows - 1, "small")


# rows per sequence around the lines of 1.75 (one or four heads) and 1.1 (two), more than two workgroups a compute unit
@pytest.mark.parametrize("hq,hkv,ones,long", [(8, 2, 64, 49), (8, 2, 64, 50), (15, 5, 64, 49), (15, 5, 64, 50), (36, 18, 64, 7), (36, 18, 64, 8),
                                              (16, 1, 64, 2), (16, 2, 64, 40)])
def test_mostly_one_row_per_sequence(oracle_mod, hq, hkv, ones, long):
    rng = np.random.default_rng(1420 + hq)
    lens, qlens = rng.integers(1, 200, ones + 1), [1] * (ones // 2) + [0, 1 + long] + [1] * (ones // 2 - 1)
    lens[ones // 2 + 1] = 300
    check(oracle_mod, lens.tolist(), qlens, hq, hkv, 1 + long, f"mixed {sum(qlens) / len(qlens):.3f}")


@pytest.mark.parametrize("max_q", [64 * 31, 64 * 33])     # tiles at most and more than eight times the row workgroups
def test_mostly_empty_tiles(oracle_mod, max_q):
    lens = np.random.default_rng(1430).integers(8, 60, 1024).tolist()
    check(oracle_mod, lens, [8] * 1024, 8, 2, max_q, "empty tiles")

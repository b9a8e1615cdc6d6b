"""Prefill of several sequences under a block table that reaches far past their contexts, as an engine with tables of one
width passes it: which order the query tiles are handed out in depends on the real lengths, and no order changes a bit."""
import numpy as np
import pytest

import kvc_workloads as W  # noqa: F401
from gpu_util import out_bits
from test_gpu_prefill import check, make, run

pytestmark = pytest.mark.gpu


def widen(w, tokens):
    w.block_tables = np.pad(w.block_tables, ((0, 0), (0, max(0, tokens // w.block_size - w.block_tables.shape[1]))),
                            constant_values=-1)


# `longest` against four times the 64-row tiles of the longest chunk (1024 and 512 tokens here); up to eight
# sequences are looked over by scalar loads, more of them by a wavefront
@pytest.mark.parametrize("lens,rows,bs", [
    ([250, 200, 250, 130, 64], 0, 16), ([120, 128, 65] * 3 + [1], 0, 8),            # recomputations
    ([1023, 300, 700, 900, 260], 256, 16), ([1024, 300, 700, 900, 260], 256, 16),
    ([511] + [130] * 8, 128, 16), ([130] * 8 + [512], 128, 16), ([200] * 8 + [4000], 128, 32),
])
def test_wide_tables(oracle_mod, lens, rows, bs):
    qlens = [min(n, rows or n) for n in lens]
    tiles = -(-max(qlens) // 64)
    assert 256 < len(lens) * tiles * 16 and len(lens) * tiles <= 64   # the launches that may rank
    w, q, qs = make(1300 + len(lens) + rows, lens, qlens, 32, 8, bs=bs)
    tight = out_bits(run(w, q, qs, max(qlens)))
    widen(w, 8192)
    check(oracle_mod, w, q, qs, f"wide table {lens[:4]} rows={rows}")
    assert np.array_equal(out_bits(run(w, q, qs, max(qlens))), tight)

"""Decode at head_dim 64 on ranges of flat tiles under a bound far above the lengths: short rows go to a worker each,
longer ones get ranges by their own lengths.  Both sides of every line against the fp64 oracle."""
import numpy as np
import pytest

import kvc_workloads as W
from test_gpu_attention import custom
from test_gpu_decode_d64 import check
from test_gpu_prefill_d64 import poison

pytestmark = pytest.mark.gpu


# 8 tiles of 32 tokens a row and 1024 workers: at the lines and past them, empty rows first, last and between
@pytest.mark.parametrize("nseq,hq,hkv,longest", [(70, 8, 2, 256), (70, 8, 2, 257), (512, 4, 2, 256), (513, 4, 2, 256), (1024, 2, 1, 200),
                                                 (1025, 2, 1, 200), (300, 9, 3, 1), (70, 16, 1, 256), (66, 14, 2, 255)])
@pytest.mark.parametrize("bs", [4, 16, 64])
def test_short_rows(oracle_mod, nseq, hq, hkv, longest, bs):
    lens = np.random.default_rng(1600 + nseq).integers(0, longest + 1, nseq)
    lens[[0, 1, nseq // 2, nseq - 1]] = [0, longest, 0, 0]
    w = custom(1600 + nseq + bs, dtype=W.BF16, lens=lens, hq=hq, hkv=hkv, d=64, bs=bs)
    poison(w)
    check(w, oracle_mod, f"short {hq}/{hkv} longest={longest} bs={bs}", max_context_len=4096)


# the smallest range by powers of two of the longest row (128, 256, 512 tiles), by all rows together, by the bound
@pytest.mark.parametrize("longest", [4096, 4097, 8192, 8193, 16384, 16385])
@pytest.mark.parametrize("tokens", [20000, 200000])
def test_long_rows(oracle_mod, longest, tokens):
    lens = [300, longest, 0, 33, 700] + [64] * 65
    check(custom(1650, dtype=W.BF16, lens=lens, hq=4, hkv=2, d=64, bs=16), oracle_mod, f"longest={longest}", max_context_len=tokens)


def test_one_row_and_a_bound_above_any_length(oracle_mod):
    check(custom(1660, dtype=W.BF16, lens=[5000] + [0] * 64, hq=4, hkv=1, d=64, bs=16), oracle_mod, "one row", max_context_len=1 << 20)

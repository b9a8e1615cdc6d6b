"""Prefill launches of at most one workgroup per compute unit: from 1569 tokens (50 steps of 32) on, the two groups of a
workgroup share its context.  Lengths around that line, and below it, and around odd and even numbers of steps, row counts that leave
wavefronts without rows, every head layout, blocks of 8 tokens and more, against the oracle.  A test on the host asks the
library which of these launches it splits."""
import numpy as np
import pytest

import kvc_workloads as W  # noqa: F401
from gpu_util import BF16_TOL, out_to_f64
from test_gpu_prefill import check, make, run
from test_gpu_prefill_d64 import poison, reference

pytestmark = pytest.mark.gpu

HEADS = [(8, 2, 16), (3, 1, 16), (3, 1, 32), (4, 4, 8), (2, 1, 32), (16, 1, 64)]   # query heads, KV heads, block size
AROUND = [1567, 1600, 1568, 1569, 1633, 1601, 1602, 1632, 1665, 1750]
BELOW = [735, 736, 737, 767, 768, 769, 800, 801, 833, 1000]
CROSSING = [(8, 2, [1800, 40], [1800, 40]), (5, 1, [1800, 40], [1800, 40])]
LONG = (4, 2, [20000, 3001], [37, 1])
RAMP = (4, 2, [2100], [64])
MINUS_INF = [(32, 8, [300, 200], [300, 200]), (8, 2, [1800], [1800])]     # whole; split


def fives(lens):
    """Five contexts at a time: the launch stays within 256 workgroups."""
    qlens = [64, 1, 17, 33, 64, 65, 128, 5, 63, 130]
    return [(lens[i:i + 5], qlens[i:i + 5]) for i in range(0, len(lens), 5)]


@pytest.mark.parametrize("hq,hkv,bs", HEADS)
def test_contexts_below_the_line(oracle_mod, hq, hkv, bs):
    for i, (lens, qlens) in enumerate(fives(BELOW)):
        w, q, qs = make(1100 + hq + bs + 5 * i, lens, qlens, hq, hkv, bs=bs)
        poison(w)
        check(oracle_mod, w, q, qs, f"below the line {hq}/{hkv} bs={bs}")


@pytest.mark.parametrize("hq,hkv,lens,qlens", CROSSING)
def test_recompute_crosses_the_line_inside_one_launch(oracle_mod, hq, hkv, lens, qlens):
    """The first query tiles of a request walk too few steps to share, the last ones share."""
    w, q, qs = make(1150 + hq, lens, qlens, hq, hkv)
    check(oracle_mod, w, q, qs, f"recompute {hq}/{hkv}")


def test_long_context_short_chunk(oracle_mod):
    hq, hkv, lens, qlens = LONG
    w, q, qs = make(1160, lens, qlens, hq, hkv)
    check(oracle_mod, w, q, qs, "long")


def test_scores_that_keep_growing_reach_both_parts(oracle_mod):
    """Rising scores keep the reference points of the two parts far apart."""
    hq, hkv, lens, qlens = RAMP
    w, q, qs = make(1170, lens, qlens, hq, hkv)
    ramp = np.linspace(-40.0, 40.0, lens[0]).astype(np.float32)
    q[:, :, 1] = 0x3F80                                   # q[1] = 1
    for t in range(lens[0]):
        w.k_cache[w.block_tables[0, t // 16], :, t % 16, 1] = W.f32_to_bf16_bits(ramp[t:t + 1] * 8)[0]
    check(oracle_mod, w, q, qs, "ramp")


@pytest.mark.parametrize("nseq,rows,longest", [(6, 130, 2500), (8, 260, 1300)])   # at most / more than 512 workgroups
def test_chunks_of_several_sequences_are_ranked(oracle_mod, nseq, rows, longest):
    """Tiles are handed out by the steps they walk; sequences without rows, with few, and of equal lengths among them."""
    lens = [longest, 300, longest, 700, 64, 1200, 555, 40][:nseq]
    qlens = [rows, 33, rows, 1, 0, 100, rows, 40][:nseq]
    w, q, qs = make(1180 + nseq, lens, qlens, 32, 8)
    items = nseq * -(-rows // 64)
    assert items <= 64 and items * 16 > 256 and w.max_blocks_per_seq * 16 >= 4 * 64 * -(-rows // 64)
    check(oracle_mod, w, q, qs, f"ranked {nseq}")


@pytest.mark.parametrize("hq,hkv,bs", HEADS)
def test_contexts_around_the_line_from_which_they_are_shared(oracle_mod, hq, hkv, bs):
    for i, (lens, qlens) in enumerate(fives(AROUND)):
        w, q, qs = make(1190 + hq + bs + 5 * i, lens, qlens, hq, hkv, bs=bs)
        poison(w)
        check(oracle_mod, w, q, qs, f"split line {hq}/{hkv} bs={bs}")


@pytest.mark.parametrize("hq,hkv,lens,qlens", MINUS_INF)
def test_scores_of_minus_infinity_weigh_nothing(oracle_mod, hq, hkv, lens, qlens):
    """The first two steps' scores are -inf in every column of the first sequence."""
    w, q, qs = make(1195 + hq, lens, qlens, hq, hkv)
    q[:, :, 0] = 0x3F80
    for t in range(64):
        w.k_cache[w.block_tables[0, t // 16], :, t % 16, 0] = 0xFF80
    print(f"[case] prefill -inf {hq}/{hkv}", flush=True)
    got = out_to_f64(run(w, q, qs, max(qlens)))
    ref = reference(oracle_mod, w, q, qs)
    assert np.isfinite(got[64:]).all()     # earlier rows see nothing else
    assert np.abs(got[64:] - ref[64:]).max() <= BF16_TOL

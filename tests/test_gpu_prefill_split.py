"""Prefill launches of at most one workgroup per compute unit: from 1121 tokens (36 steps of 32) on, the two groups of a
workgroup share its context.  Lengths around that line, and below it, and around odd and even numbers of steps, row counts that leave
wavefronts without rows, every head layout, blocks of 8 tokens and more, against the oracle."""
import numpy as np
import pytest

import kvc_workloads as W  # noqa: F401
from gpu_util import BF16_TOL, out_to_f64
from test_gpu_prefill import check, make, run
from test_gpu_prefill_d64 import poison, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,bs", [(8, 2, 16), (3, 1, 16), (4, 4, 8), (2, 1, 32), (16, 1, 64)])
def test_contexts_around_the_line_and_odd_shares(oracle_mod, hq, hkv, bs):
    lens = [735, 736, 737, 767, 768, 769, 800, 801, 833, 1000]
    qlens = [64, 1, 17, 33, 64, 65, 128, 5, 63, 130]
    for i in range(0, len(lens), 5):      # five at a time: the launch stays within 256 workgroups
        w, q, qs = make(1100 + hq + bs + i, lens[i:i + 5], qlens[i:i + 5], hq, hkv, bs=bs)
        poison(w)
        assert len(lens[i:i + 5]) * 3 * hq <= 256
        check(oracle_mod, w, q, qs, f"split {hq}/{hkv} bs={bs}")


@pytest.mark.parametrize("hq,hkv", [(8, 2), (5, 1)])
def test_recompute_crosses_the_line_inside_one_launch(oracle_mod, hq, hkv):
    """The first query tiles of a request walk too few steps to share, the last ones share."""
    w, q, qs = make(1150 + hq, [1300, 40], [1300, 40], hq, hkv)
    check(oracle_mod, w, q, qs, f"recompute {hq}/{hkv}")


def test_long_context_short_chunk(oracle_mod):
    w, q, qs = make(1160, [20000, 3001], [37, 1], 4, 2)
    check(oracle_mod, w, q, qs, "long")


def test_scores_that_keep_growing_reach_both_parts(oracle_mod):
    """Rising scores keep the reference points of the two parts far apart."""
    w, q, qs = make(1170, [1500], [64], 4, 2)
    ramp = np.linspace(-40.0, 40.0, 1500).astype(np.float32)
    q[:, :, 1] = 0x3F80                                   # q[1] = 1
    for t in range(1500):
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


@pytest.mark.parametrize("hq,hkv,bs", [(8, 2, 16), (3, 1, 32), (4, 4, 8)])
def test_contexts_around_the_line_from_which_they_are_shared(oracle_mod, hq, hkv, bs):
    lens = [1119, 1120, 1121, 1152, 1153, 1154, 1184, 1185, 1217, 1300]
    qlens = [64, 1, 17, 33, 64, 65, 128, 5, 63, 130]
    for i in range(0, len(lens), 5):      # five at a time: the launch stays within 256 workgroups
        w, q, qs = make(1190 + hq + bs + i, lens[i:i + 5], qlens[i:i + 5], hq, hkv, bs=bs)
        poison(w)
        assert len(lens[i:i + 5]) * 3 * hq <= 256
        check(oracle_mod, w, q, qs, f"split line {hq}/{hkv} bs={bs}")


@pytest.mark.parametrize("hq,hkv,lens,qlens", [(32, 8, [300, 200], [300, 200]), (8, 2, [1400], [1400])])  # plain; shared
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

"""Prefill of odd groups in launches of more than 1024 workgroups of one head: the heads of a KV head go to one XCD.
KV heads in multiples of eight and others (whose last units are dealt out singly), tiles ranked and not, against the oracle."""
import pytest

import kvc_workloads as W  # noqa: F401
from test_gpu_prefill import check, make
from test_gpu_prefill_d64 import poison

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,bs,nseq", [(24, 8, 16, 44), (27, 9, 8, 40), (50, 10, 32, 22), (33, 11, 4, 34)])
def test_every_row_is_computed_once(oracle_mod, hq, hkv, bs, nseq):
    lens = [(37 * i) % 150 + 1 for i in range(nseq - 1)] + [200]
    qlens = [max(1, n - 40 * (i % 3)) for i, n in enumerate(lens)]
    qlens[3] = 0
    assert hq * nseq * -(-max(qlens) // 128) > 1024
    w, q, qs = make(1500 + hq, lens, qlens, hq, hkv, bs=bs)
    poison(w)
    check(oracle_mod, w, q, qs, f"units {hq}/{hkv} bs={bs}")


def test_chunks_are_ranked(oracle_mod):
    nseq = 22
    lens = [1100 - 50 * (i % 20) for i in range(nseq)]
    qlens = [130 if n >= 130 else n for n in lens]
    w, q, qs = make(1590, lens, qlens, 24, 8)
    assert 24 * nseq * 2 > 1024 and nseq * 2 <= 64 and w.max_blocks_per_seq * 16 >= 4 * 64 * 3 and max(lens) >= 768
    poison(w)
    check(oracle_mod, w, q, qs, "units ranked")

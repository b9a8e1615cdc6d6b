"""Prefill over blocks of 8 tokens, whose ids come through the scalar cache as those of larger blocks do: the same
tokens in blocks of 8 and of 16 give the same bits, for every workgroup shape, and the oracle's values."""
import numpy as np
import pytest
import torch

import kvc_workloads as W
from gpu_util import out_bits
from test_gpu_prefill import check, make
from test_gpu_prefill_d64 import poison

pytestmark = pytest.mark.gpu


def paged(dense, bs, seed):
    """[tokens][heads][D] of every sequence scattered over blocks of `bs` tokens; slots past the end hold NaN."""
    rng = np.random.default_rng(seed)
    need = [-(-len(d) // bs) for d in dense]
    ids = rng.permutation(sum(need) + 3)
    tables = np.full((len(dense), max(need) + 1), -1, dtype=np.int32)
    pool = torch.full((sum(need) + 3, dense[0].shape[1], bs, dense[0].shape[2]), float("nan"), dtype=torch.bfloat16)
    at = 0
    for n, d in enumerate(dense):
        tables[n, :need[n]] = ids[at:at + need[n]]
        at += need[n]
        for i in range(need[n]):
            part = d[i * bs:(i + 1) * bs]
            pool[tables[n, i], :, :len(part)] = part.transpose(0, 1)
    return tables, pool


# two heads and one head per workgroup, launches that fit the device at once and long ones, 64 columns per wavefront (the last)
SHAPES = [(8, 2, [1, 7, 8, 9, 25, 200, 333], [1, 7, 8, 9, 25, 100, 333]), (7, 1, [1, 8, 15, 17, 130, 300], [1, 8, 15, 17, 130, 40]),
          (32, 2, [3100, 3073], [3100, 3073]), (28, 4, [3333, 70], [3333, 70]), (32, 2, [3600], [3577])]


@pytest.mark.parametrize("hq,hkv,lens,qlens", SHAPES)
def test_blocks_of_8_equal_blocks_of_16(hq, hkv, lens, qlens):
    import paper_2503_13773_amd as K
    gen = torch.Generator().manual_seed(11)
    k = [torch.randn((n, hkv, 128), generator=gen).to(torch.bfloat16) for n in lens]
    v = [torch.randn((n, hkv, 128), generator=gen).to(torch.bfloat16) for n in lens]
    starts = torch.tensor(np.concatenate([[0], np.cumsum(qlens)]), dtype=torch.int32, device="cuda")
    q = torch.randn((sum(qlens), hq, 128), generator=gen).to(torch.bfloat16).cuda()
    out = {}
    for bs in (8, 16):
        tables, kp = paged(k, bs, 3)
        _, vp = paged(v, bs, 3)
        print(f"[case] prefill blocks of {bs} {hq}/{hkv} {lens}", flush=True)
        out[bs] = out_bits(K.paged_attention_prefill(q, kp.cuda(), vp.cuda(), torch.from_numpy(tables).cuda(),
                                                     torch.tensor(lens, dtype=torch.int32, device="cuda"), starts, 128 ** -0.5,
                                                     max(qlens)))
    assert np.array_equal(out[8], out[16])


@pytest.mark.parametrize("hq,hkv", [(8, 2), (3, 1)])
def test_against_the_oracle(oracle_mod, hq, hkv):
    lens = [1, 8, 9, 16, 17, 63, 64, 65, 130, 300]
    w, q, qs = make(650 + hq, lens, [1, 8, 3, 16, 17, 20, 64, 1, 130, 129], hq, hkv, bs=8)
    poison(w)
    check(oracle_mod, w, q, qs, f"blocks of 8 {hq}/{hkv}")

"""kv_cache_append of more sequences than the threads of one launch serve (2^32 of them, 256 to a sequence)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv", [5])
def test_more_sequences_than_one_launch_serves(hkv):
    import paper_2503_13773_amd as K
    nseq = (1 << 24) + 3                                                 # 40 words of 16 bytes each: a workgroup per sequence
    print(f"[case] append of {nseq} sequences, {hkv} heads", flush=True)
    rows = [0, 1, (1 << 24) - 2, (1 << 24) - 1, 1 << 24, nseq - 1]
    new = torch.empty(nseq, hkv, 64, dtype=torch.bfloat16, device="cuda")
    for r in rows:
        new[r] = torch.randn(hkv, 64, device="cuda")
    tables = torch.zeros(nseq, 1, dtype=torch.int32, device="cuda")
    positions = torch.full((nseq,), -1, dtype=torch.int32, device="cuda")
    for i, r in enumerate(rows):
        tables[r], positions[r] = 1 + i, i
    k, v = (torch.zeros(len(rows) + 1, hkv, 16, 64, dtype=torch.bfloat16, device="cuda") for _ in "kv")
    want = torch.zeros_like(k)
    for i, r in enumerate(rows):
        want[1 + i, :, i] = new[r]
    K.kv_cache_append(new, new, k, v, tables, positions)
    assert torch.equal(k, want) and torch.equal(v, want)
    # shifted by one row: which launch serves a sequence does not matter
    k.zero_()
    K.kv_cache_append(new[1:], new[1:], k, v, tables[1:], positions[1:])
    want[1] = 0
    assert torch.equal(k, want)

"""Which head_dim 64 decode calls take the balanced kernel, and what the others keep (no GPU needed)."""
import pytest

from test_abi_cpu import K, desc, plan_status  # noqa: F401


def test_auto_takes_the_balanced_kernel_for_large_batches(K):  # noqa: F811
    d = desc(K, head_dim=64)
    rc, p = plan_status(K, d)
    slots = 256 * 4 * 2
    assert rc == 0 and p.kernel == K.KERNEL_MFMA_BALANCED and p.merge_grid == 0 and p.partial_grid == 256
    assert p.workspace_bytes == 4096 + slots * 4 * 64 * 4 + slots * 4 * 2 * 4
    assert p.workspace_bytes <= K.NOALLOC_WORKSPACE_BYTES


@pytest.mark.parametrize("kw", [
    dict(num_q_heads=16, num_kv_heads=16, max_context_len=200),   # 1024 rows of one head each, up to 200 tokens
    dict(partition_tokens=512),           # the caller's own split
    dict(dtype=0), dict(block_size=2), dict(num_q_heads=136), dict(num_seqs=4097), dict(kernel=1),
])
def test_the_others_stay_on_the_vector_alus(K, kw):  # noqa: F811
    rc, p = plan_status(K, desc(K, head_dim=64, **kw))
    assert rc == 0 and p.kernel == K.KERNEL_VALU
    if kw.get("max_context_len") == 200:
        assert p.workspace_bytes == 0


def test_whole_rows_need_no_workspace_and_pieces_do(K):  # noqa: F811
    for kw, need in [(dict(num_seqs=4, max_context_len=4000), True), (dict(num_seqs=16, max_context_len=641), True),
                     (dict(num_seqs=16, max_context_len=640), False), (dict(num_seqs=17, max_context_len=1024), False),
                     (dict(num_seqs=17, max_context_len=1025), True), (dict(num_seqs=1, max_context_len=7), False)]:
        rc, p = plan_status(K, desc(K, head_dim=64, **kw))
        assert rc == 0 and p.kernel == K.KERNEL_MFMA_BALANCED and (p.workspace_bytes > 0) == need
        assert p.partial_grid == (256 if need else kw["num_seqs"] * 8)


def test_layouts_of_head_dim_128(K):  # noqa: F811
    for kw, grid in [(dict(num_seqs=64, max_context_len=512), 512), (dict(num_seqs=64, max_context_len=513), 256),
                     (dict(num_seqs=126, max_context_len=200), 256), (dict(num_seqs=126, max_context_len=201), 1008),
                     (dict(num_seqs=125, max_context_len=200), 1000), (dict(num_seqs=64, max_context_len=512, partition_tokens=64), 256)]:
        rc, p = plan_status(K, desc(K, **kw))
        assert rc == 0 and p.kernel == K.KERNEL_MFMA_BALANCED and p.merge_grid == 0 and p.partial_grid == grid
        assert p.workspace_bytes == K.workspace_bytes(desc(K)) and K.schedule_bytes(desc(K, **kw)) > 0


def test_explicit_kernels_and_schedules_stay_refused(K):  # noqa: F811
    for kernel in (2, 3, 4):
        assert plan_status(K, desc(K, head_dim=64, kernel=kernel))[0] == -4
    assert K.schedule_bytes(desc(K, head_dim=64)) == 0

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
                     (dict(num_seqs=16, max_context_len=640), False), (dict(num_seqs=17, max_context_len=640), False),
                     (dict(num_seqs=17, max_context_len=1025), True), (dict(num_seqs=1, max_context_len=7), False)]:
        rc, p = plan_status(K, desc(K, head_dim=64, **kw))
        assert rc == 0 and p.kernel == K.KERNEL_MFMA_BALANCED and (p.workspace_bytes > 0) == need
        assert p.partial_grid == (256 if need else kw["num_seqs"] * 8)
    rc, p = plan_status(K, desc(K, head_dim=64, num_seqs=17, max_context_len=1024))
    assert rc == 0 and p.partial_grid == 17 * 8 and p.workspace_bytes > 0  # whole rows; 16 of them would be pieces


@pytest.mark.parametrize("heads", [(32, 8), (16, 16), (14, 2), (12, 12), (1, 1), (2, 1), (64, 4), (256, 128)])
@pytest.mark.parametrize("block_size", [4, 8, 16, 32])
def test_buffers_do_for_smaller_batches_and_lower_bounds(K, heads, block_size):  # noqa: F811
    """Workspaces and schedules: at every (batch, bound) the size is at least that of the next smaller batch and
    of the next lower bound, whichever layouts these have."""
    seqs = [0, 1, 2, 3, 8, 10, 11, 16, 17, 32, 33, 63, 64, 65, 66, 96, 125, 126, 127, 128, 129, 500, 1001, 4096]
    bounds = [1, 16, 200, 201, 256, 257, 500, 512, 513, 560, 640, 641, 1000, 1024, 1025, 1100, 2000, 2049, 4096, 8192]
    for size, dim in ((K.workspace_bytes, 64), (K.workspace_bytes, 128), (K.schedule_bytes, 128)):
        table = [[size(desc(K, head_dim=dim, num_q_heads=heads[0], num_kv_heads=heads[1], num_seqs=n, block_size=block_size,
                            max_blocks_per_seq=8192 // block_size, max_context_len=b)) for b in bounds] for n in seqs]
        for i, n in enumerate(seqs):
            for j, b in enumerate(bounds):
                assert i < 2 or table[i][j] >= table[i - 1][j], (size.__name__, dim, n, b)
                assert not j or table[i][j] >= table[i][j - 1], (size.__name__, dim, n, b)


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


def test_whole_rows_of_head_dim_128_end_at_2048_rows(K):  # noqa: F811
    for n, heads, grid in [(256, 8, 2048), (257, 8, 256), (64, 32, 2048), (65, 32, 256), (2048, 1, 2048), (2049, 1, 256)]:
        d = desc(K, num_seqs=n, num_q_heads=heads, num_kv_heads=heads, max_context_len=300)
        rc, p = plan_status(K, d)
        assert rc == 0 and p.kernel == K.KERNEL_MFMA_BALANCED and p.partial_grid == grid


def test_few_rows_of_head_dim_64(K):  # noqa: F811
    """The vector ALUs keep up to 384 (query head, 256-token partition) pairs, 512 with two heads per KV head, 1024
    with one and less than 128 rows."""
    for n, hq, hkv, ctx, balanced in [(1, 14, 2, 6912, False), (1, 14, 2, 6913, True), (3, 32, 8, 1024, False), (4, 32, 8, 1024, True),
                                      (1, 16, 8, 8192, False), (1, 16, 8, 8193, True), (4, 16, 16, 4096, False), (5, 16, 16, 4096, True), (8, 16, 16, 768, False), (8, 16, 16, 769, True),
                                      (1, 1, 1, 65536, False), (64, 1, 1, 8192, True)]:
        rc, p = plan_status(K, desc(K, head_dim=64, num_seqs=n, num_q_heads=hq, num_kv_heads=hkv, max_blocks_per_seq=8192, max_context_len=ctx))
        assert rc == 0 and (p.kernel == K.KERNEL_MFMA_BALANCED) == balanced, (n, hq, hkv, ctx)


def test_one_head_per_kv_head_and_many_short_rows(K):  # noqa: F811
    for n, ctx, kernel in [(40, 256, 4), (41, 256, 1), (41, 257, 4)]:
        rc, p = plan_status(K, desc(K, head_dim=64, num_seqs=n, num_q_heads=16, num_kv_heads=16, max_context_len=ctx))
        assert rc == 0 and p.kernel == kernel and (kernel == 1 or p.partial_grid == n * 16)


@pytest.mark.parametrize("heads", [(32, 8), (16, 16), (14, 2), (1, 1), (64, 4)])
def test_workspaces_of_batches_beyond_the_balanced_kernel_do_for_smaller_ones(K, heads):  # noqa: F811
    """4097 and more sequences are the vector ALUs', often without a workspace of their own: what the query answers for them
    is enough for the batches below, bound by bound, and the call itself still runs with what it needs."""
    import ctypes
    kw = dict(head_dim=64, num_q_heads=heads[0], num_kv_heads=heads[1], max_blocks_per_seq=512, num_pool_blocks=64)
    for bound in (600, 640, 641, 1000, 1024, 1025, 4096, 8192):
        below = max(K.workspace_bytes(desc(K, num_seqs=n, max_context_len=b, **kw)) for n in (1, 3, 20, 65, 129, 2000, 4096)
                    for b in (600, 640, 641, 1000, bound) if b <= bound)
        for n in (4097, 5000, 8192, 20000):
            d = desc(K, num_seqs=n, max_context_len=bound, **kw)
            rc, p = plan_status(K, d)
            assert rc == 0 and p.kernel == K.KERNEL_VALU and p.workspace_bytes >= below, (n, bound)
            if p.merge_grid == 0:   # one partition: no workspace is needed, and none is missed
                a = ctypes.c_void_p(4096)
                assert K.lib().kvc_paged_attention_decode_merge(a, a, ctypes.byref(d), None, 0, None) == 0, (n, bound)


def test_sizes_of_the_vector_alu_kernel_are_its_own(K):  # noqa: F811
    """fp32 is never the balanced kernel's: what the query answers is what the call needs."""
    for n in (1, 512, 513, 4097):
        rc, p = plan_status(K, desc(K, dtype=0, head_dim=64, num_seqs=n, max_context_len=1000))
        parts = p.max_partitions
        want = 0 if parts == 1 else (4096 + n * 32 * parts * 64 * 4 + 255) // 256 * 256 + n * 32 * parts * 8
        assert rc == 0 and p.workspace_bytes == want

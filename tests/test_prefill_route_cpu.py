"""Where the workgroups of a prefill launch on 32x32 tiles go, asked of the library's own rules (no GPU needed)."""
import ctypes

import numpy as np
import pytest

import prefill_route


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    return prefill_route.build(str(tmp_path_factory.mktemp("route")))


@pytest.mark.parametrize("group,kv_heads,indexes", [(5, 8, 58), (3, 16, 7), (7, 8, 1), (5, 10, 129), (3, 9, 43), (15, 8, 9), (3, 33, 5),
                                                    (7, 11, 2), (3, 8, 1)])
def test_units_cover_every_workgroup_and_share_an_xcd(route, group, kv_heads, indexes):
    blocks = group * kv_heads * indexes
    out = (ctypes.c_int * (3 * blocks))()
    route.places(blocks, group, kv_heads, out)
    kv, head, index = np.frombuffer(out, dtype=np.int32).reshape(blocks, 3).T
    assert (head // group == kv).all() and head.min() == 0 and head.max() < group * kv_heads and index.min() == 0
    assert len(set(zip(head.tolist(), index.tolist()))) == blocks and index.max() == indexes - 1
    # the device hands block b to XCD b % 8; fewer than eight units at the end are dealt out as they come
    whole = blocks // (8 * group) * 8 * group
    for b in range(0, whole, 8 * group):
        for x in range(8):
            unit = slice(b + x, b + 8 * group, 8)
            assert len(set(zip(kv[unit].tolist(), index[unit].tolist()))) == 1 and len(set(head[unit])) == group
    if kv_heads % 8 == 0:
        assert whole == blocks and all(len(set(np.arange(blocks)[kv == k] % 8)) == 1 for k in range(kv_heads))
    else:
        # no XCD gets the longer tiles throughout: mean tile index per XCD, over the runs that come in pairs
        pairs = blocks // (16 * group) * 16 * group
        means = [index[:pairs][np.arange(pairs) % 8 == x].mean() for x in range(8)] if pairs else [0]
        assert max(means) - min(means) <= 1.0


@pytest.mark.parametrize("hq,hkv,qlens,units", [
    (40, 8, [4096] * 4, True), (40, 8, [3600] * 2, True), (56, 8, [4096] * 4, True), (50, 10, [4096] * 4, True),
    (40, 8, [128 * 25], False), (40, 8, [128 * 26], True),          # 1000 and 1040 workgroups
    (28, 4, [4096] * 4, False), (35, 5, [3600] * 2, False), (49, 7, [4096] * 4, False),   # fewer than eight KV heads
    (32, 32, [4096] * 4, False), (32, 8, [4096] * 4, False)])       # nothing to share; two heads per workgroup
def test_odd_groups_place_long_launches_by_units(route, hq, hkv, qlens, units):
    assert bool(route.by_units(prefill_route.values(hq, hkv, qlens, max(qlens)))) == units


@pytest.mark.parametrize("heads,bs,scale,yes", [(65535, 256, 0.1, True), (65536, 256, 0.1, False), (131071, 128, 0.1, True),
                                                (131072, 128, 0.1, False), (8, 16, 0.1, True), (8, 16, 0.0, False), (8, 16, -0.1, False)])
def test_blocks_of_4_gib_and_other_scales_take_16x16_tiles(route, heads, bs, scale, yes):
    assert bool(route.tiles32(prefill_route.values(heads, heads, [40], bs, bs), ctypes.c_float(scale))) == yes


@pytest.mark.parametrize("hq,hkv,qlens,tokens,bs,yes", [
    (32, 8, [64], 1568, 16, False), (32, 8, [64], 1569, 16, True), (32, 8, [64], 1200, 16, False),   # 49 and 50 steps
    (32, 8, [16 * 64], 4000, 16, True), (32, 8, [16 * 64 + 1], 4000, 16, False),                     # workgroups
    (28, 4, [9 * 128], 4000, 16, True), (28, 4, [9 * 128 + 1], 4000, 16, False),
    (32, 8, [64], 4000, 8, True), (32, 8, [64], 4000, 4, False)])                                    # blocks
def test_which_launches_are_split(route, hq, hkv, qlens, tokens, bs, yes):
    assert bool(route.split(prefill_route.values(hq, hkv, qlens, tokens, bs))) == yes


def test_device_tests_of_split_workgroups_reach_them(route):
    import test_gpu_prefill_split as T

    def split(hq, hkv, lens, qlens, bs=16):
        blocks = -(-max(lens) // bs) + 1     # of their tables
        return bool(route.split(prefill_route.values(hq, hkv, qlens, blocks * bs, bs)))

    line = 32 * (route.split_steps() - 1)
    for hq, hkv, bs in T.HEADS:
        for lens, qlens in T.fives(T.AROUND):
            assert split(hq, hkv, lens, qlens, bs) and min(lens) <= line + 200 and max(lens) > line
        for lens, qlens in T.fives(T.BELOW):
            assert max(lens) <= line and not split(hq, hkv, lens, qlens, bs)
    assert min(T.AROUND) < line and {line, line + 1} <= set(T.AROUND)
    for hq, hkv, lens, qlens in [*T.CROSSING, T.LONG, T.RAMP, T.MINUS_INF[1]]:
        assert split(hq, hkv, lens, qlens) and max(lens) > line + 64
    assert not split(*T.MINUS_INF[0])


def wide(route, hq, hkv, qlens, bs=16):
    return bool(route.wide(prefill_route.values(hq, hkv, qlens, max(qlens), bs), ctypes.c_longlong(sum(qlens))))


def test_shapes_of_the_device_tests_reach_the_kernel_of_64_columns(route):
    import test_gpu_large_pool as P
    import test_gpu_prefill_block8 as B
    import test_gpu_prefill_wide as T
    for hq, hkv, _, qlens, bs in T.SHAPES:
        assert wide(route, hq, hkv, qlens, bs), (hq, hkv, qlens, bs)
    assert wide(route, *T.SPECIAL[:2], T.SPECIAL[2])
    assert [wide(route, hq, hkv, qlens) for hq, hkv, _, qlens in B.SHAPES].count(True) >= 1
    assert wide(route, *P.WIDE)


def test_replayed_prefills_are_of_the_kinds_they_name(route):
    import test_gpu_graph_replay as G
    for kind, (hq, hkv, lens, qlens) in G.PREFILLS.items():
        v = prefill_route.values(hq, hkv, qlens, (-(-max(lens) // 16) + 1) * 16)
        assert [wide(route, hq, hkv, qlens), bool(route.split(v)), bool(route.by_units(v))] == [kind == k for k in ("wide", "split", "units")]


# both sides of every line of the rule, with the shapes that were slower on 64 columns
@pytest.mark.parametrize("hq,hkv,qlens,yes", [
    (32, 8, [54 * 64], True), (32, 8, [52 * 64], False),              # rounds of 1.65 (one request)
    (32, 8, [65 * 64], True), (32, 8, [66 * 64], False), (32, 8, [5000], False), (32, 8, [6500], False),      # of 2
    (32, 8, [109 * 64], True), (32, 8, [108 * 64], False), (32, 8, [16384], True),                            # of 3.4
    (64, 8, [32 * 64], True), (96, 8, [31 * 64], False), (128, 16, [31 * 64], False), (128, 16, [32 * 64], True),  # 32 tiles
    (64, 8, [2500], False), (16, 2, [6500], False), (16, 2, [7300], True),
    (32, 8, [3500, 3000, 3400, 2900], False), (32, 8, [4900, 4000, 4800, 4100], False), (32, 8, [4096, 3700] * 3, True),  # heads times requests
    (64, 8, [4096, 3500], False), (64, 8, [4096, 3500, 4000], True), (16, 2, [6500, 5000], False), (24, 2, [5000, 4500], False),
    (64, 8, [4096] * 2, True), (16, 2, [3600] * 2, True), (16, 2, [5000] * 2, False), (32, 8, [4096] * 2, True),  # equal rows
    (32, 8, [100 * 64, 94 * 64], True), (32, 8, [100 * 64, 93 * 64], False), (32, 8, [2048] * 2, False), (32, 2, [2048] * 2, True),
    (32, 8, [55 * 64, 50 * 64] * 5, True), (32, 8, [54 * 64, 50 * 64] * 5, False),                              # tiles
    (64, 8, [32 * 64, 30 * 64] * 2, True), (64, 8, [31 * 64, 29 * 64] * 3, False),
    (64, 8, [32 * 64] * 3 + [16 * 64], True), (64, 8, [32 * 64] * 3 + [15 * 64], False),                      # seven rounds
    (8, 2, [8000, 6000], True), (8, 1, [5000, 4000], False), (8, 2, [54 * 64] * 2, False),                    # two of eight heads
    (128, 8, [8000] * 3 + [10] * 4, False), (128, 8, [8000] * 4 + [10] * 3, True),                            # a mean of half
    (24, 8, [8000], False), (40, 8, [8000], False), (48, 8, [8000], False)])                                  # groups
def test_which_calls_take_64_columns(route, hq, hkv, qlens, yes):
    assert wide(route, hq, hkv, qlens) == yes


@pytest.mark.parametrize("hq,hkv,qlens,yes", [
    (32, 8, [5000], False), (32, 8, [95 * 64], False), (32, 8, [96 * 64], True), (32, 8, [65 * 64], True), (32, 8, [66 * 64], False),
    (32, 8, [4096, 3500, 3800], True), (32, 8, [45 * 64, 40 * 64] * 3, True), (32, 8, [44 * 64, 40 * 64] * 3, False),
    (32, 8, [46 * 64, 43 * 64], False), (32, 8, [47 * 64, 43 * 64], True),                    # 2.8 rounds
    (16, 2, [8000, 7000], False), (16, 2, [8000, 7000, 7500], True), (8, 2, [9000, 8000] * 2, False),  # XCDs of their own
    (64, 8, [3600, 2700], False), (64, 8, [58 * 64, 54 * 64], True), (64, 8, [2600, 2300, 2400], True), (64, 8, [31 * 64] * 3, False),
    (24, 8, [8000], False)])
@pytest.mark.parametrize("bs", [1, 4])
def test_which_calls_take_64_columns_on_blocks_of_few_tokens(route, hq, hkv, qlens, yes, bs):
    assert wide(route, hq, hkv, qlens, bs) == yes


def test_blocks_of_8_tokens_and_more_are_judged_alike(route):
    for shape in [(32, 8, [6500]), (32, 8, [4096, 3500, 3800]), (64, 8, [2600, 2300, 2400]), (64, 8, [2600] * 5)]:
        assert len({wide(route, *shape, bs) for bs in (8, 16, 256)}) == 1


@pytest.mark.parametrize("chunks,sharing", [(16, 2), (8, 1), (32, 4), (24, 6), (40, 5), (64, 8), (12, 2), (7, 7), (16, 1), (2, 2)])
def test_head_chunks_of_a_kv_head_are_on_one_xcd(route, chunks, sharing):
    at = np.array([route.chunk(b, chunks, sharing) for b in range(chunks)])
    assert sorted(at) == list(range(chunks))
    if sharing > 1 and chunks % 8 == 0:
        for x in range(8):  # neighbours, so no more KV heads than that many chunks can hold
            assert (np.diff(at[x::8]) == 1).all() and len(at[x::8]) == chunks // 8
    else:
        assert (at == np.arange(chunks)).all()

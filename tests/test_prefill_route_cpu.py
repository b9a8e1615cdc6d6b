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
    v = prefill_route.values(hq, hkv, qlens, max(qlens))
    heads = 2 if hq // hkv % 2 == 0 else 1
    grid = hq // heads * len(qlens) * -(-max(qlens) // (128 // heads))
    assert bool(route.by_units(v, ctypes.c_longlong(grid))) == units

"""Sizes that the attention workspace queries return: work lists, and partial results of split items for
the units that end with the sequence only, however many segments a layer is cut into."""
import ctypes as C

import pytest

from paper_2608_29058_amd import _rs

MIB = 1 << 20


def _sizes(n, seg, hq, hkv, d=128, first=0):
    segs = [(s, min(n, s + seg)) for s in range(first, n, seg)]
    units = [(h, s0, s1, 0, i) for i, (s0, s1, h) in enumerate((*s, h) for s in segs for h in range(hq))]
    qkv = _rs.RsQkv(q=16, k=16, v=16, n=n, hq=hq, hkv=hkv, d=d, sq_h=n * d, sq_t=d, sk_h=n * d, sk_t=d, sv_h=n * d,
                    sv_t=d)
    u = _rs.make_units(units)
    tiles = sum((s1 - 1) // 128 - s0 // 128 + 1 for _, s0, s1, _, _ in units)
    L = _rs.lib()
    return (L.rs_attn_workspace_size(C.byref(qkv), u, len(units)),
            L.rs_routed_attn_workspace_size(C.byref(qkv), u, len(units)), len(units), tiles)


@pytest.mark.parametrize("n,seg,hq,hkv", [(16384, 2048, 32, 8), (65536, 2048, 32, 8), (131072, 4096, 32, 8)])
def test_layers_of_short_segments_stay_below_100_mib(n, seg, hq, hkv):
    grouped, routed, _, _ = _sizes(n, seg, hq, hkv)
    assert grouped < 100 * MIB and routed < 100 * MIB, (grouped / MIB, routed / MIB)


@pytest.mark.parametrize("n,seg,hq,hkv,d", [
    (131072, 2048, 32, 8, 128), (131072, 1024, 16, 16, 128), (131072, 512, 32, 8, 128), (262144, 2048, 16, 16, 128),
    (262144, 128, 8, 2, 64), (65536, 128, 1, 1, 128), (50001, 700, 28, 4, 128), (777, 777, 32, 8, 128),
])
def test_partial_results_are_bounded(n, seg, hq, hkv, d):
    """At most 1536 slots of 128 rows x (d + 2) floats and two counters beside the lists (an item in each
    family's list, a unit record in each)."""
    grouped, routed, units, tiles = _sizes(n, seg, hq, hkv, d)
    parts = 1536 * (128 * (d + 2) * 4 + 8) + 8192
    items = tiles + 1536
    assert grouped <= parts + 4 * items + 64 * units
    assert routed <= parts + 16 * items + 4 * 64 * units + 32 * units


def test_a_chunk_at_the_end_has_room_for_its_pieces():
    whole, _, units, tiles = _sizes(65536, 512, 32, 8, first=65536 - 512)
    assert whole > tiles * 2 * 128 * 130 * 4  # at least two pieces an item


def test_fp32_copies_cover_the_units_only():
    """One head's first 2048 tokens of a long fp32 context: its rows, not the layer's; and none for a
    call that reads too little to gain from copies."""
    n, hq, hkv, d = 131072, 32, 8, 128
    qkv = _rs.RsQkv(q=16, k=16, v=16, dtype=1, n=n, hq=hq, hkv=hkv, d=d, sq_h=n * d, sq_t=d, sk_h=n * d, sk_t=d,
                    sv_h=n * d, sv_t=d)
    L = _rs.lib()

    def size(units):
        u = _rs.make_units(units)
        return (L.rs_attn_workspace_size(C.byref(qkv), u, len(units)),
                L.rs_routed_attn_workspace_size(C.byref(qkv), u, len(units)))

    rows = 3 * 2048 * d * 2
    for got in size([(3, 0, 2048)]):
        assert rows <= got <= rows + 16384
    for got in size([(3, 0, 64)]):
        assert got <= 4096
    whole = (hq + 2 * hkv) * n * d * 2
    for got in size([(h, 0, n) for h in range(hq)]):
        assert whole <= got <= whole + MIB


@pytest.mark.parametrize("hq,hkv,n,d", [(1999, 1000, 4096, 128), (5, 2, 4096, 128), (2, 5, 4096, 64), (7, 7, 0, 128), (3, 0, 100, 64)])
def test_size_queries_of_refused_layers_return(hq, hkv, n, d):
    """Layers and units that the calls refuse: the queries read nothing outside their lists."""
    qkv = _rs.RsQkv(q=16, k=16, v=16, dtype=1, n=n, hq=hq, hkv=hkv, d=d)
    L = _rs.lib()
    for units in ([(h, 0, 4096) for h in range(hq)], [(-1, 0, 10)], [(99, 5, 10)], [(0, 90, 10)], [(0, -5, 10)]):
        u = _rs.make_units(units)
        assert L.rs_attn_workspace_size(C.byref(qkv), u, len(units)) > 0
        assert L.rs_routed_attn_workspace_size(C.byref(qkv), u, len(units)) > 0

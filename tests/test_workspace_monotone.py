"""A workspace sized for the largest graph serves the smaller ones: no size query gets smaller
past the counts where the sorts' tiles, the lanes per body and the bodies per thread change."""
import ctypes as C

import pytest

L = pytest.importorskip("paper_2108_00529_amd._lib", reason="libbgv.so not built")

LINES = [1 << 14, 16_384 * 5 // 4, 1 << 15, 45_056, 1 << 16, 1 << 17, 184_320, 1 << 18, 1 << 20]
COEF = (C.c_uint64 * 24)()


def community(**kw):
    p = L.CdParams(16, kw.get("passes", 1), 2, kw.get("method", 0), kw.get("chunk", 1 << 40), 0, kw.get("rule", 0))
    return lambda n, m: L.bgv_community_workspace(n, m, C.byref(p))


def supergraph(rows, cols):
    coef = C.cast(COEF, C.c_void_p)
    p = L.SketchParams(rows, cols, coef, coef)
    return lambda n, m: L.bgv_supergraph_workspace(n, m, C.byref(p))


def layout(exact):
    p = L.Fa2Params(1, exact, 1.2, 1, 1, 1, 0.1, 10)
    return lambda K, E: L.bgv_fa2_workspace(K, E, C.byref(p))


QUERIES = {
    "draw": lambda n, m: L.bgv_draw_workspace(n),
    "tree": lambda n, m: L.bgv_bh_tree_workspace(n),
    "layout exact": layout(1),
    "layout Barnes-Hut": layout(0),
    "energy": lambda n, m: L.bgv_fa2_energy_workspace(n, m),
    "batched": lambda n, m: L.bgv_batched_workspace(8, n, m),
    "supergraph small sketch": supergraph(4, 1024),
    "supergraph large sketch": supergraph(5, 1 << 20),
    "community": community(),
    "community chunks": community(chunk=4096, passes=3),
    "community back-pointers": community(method=2, chunk=1, passes=2),
    "community volume": community(rule=1, chunk=1 << 16),
}


@pytest.mark.parametrize("name", QUERIES)
def test_never_smaller_for_more(name):
    query = QUERIES[name]
    for line in LINES:
        for half in (line // 2, line):  # a sort of both ends of every edge has twice as many keys
            around = [half + d for d in (-33, -1, 0, 1, 2, 33)]
            for other in (1000, 200_000, 3_000_000):
                for sizes in ([query(x, other) for x in around], [query(other, x) for x in around]):
                    assert sizes == sorted(sizes), (half, other, sizes)

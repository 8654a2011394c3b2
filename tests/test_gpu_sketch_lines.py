"""Where sketch 2 goes over to the grouped form by edges alone or by fewer additions into a large
sketch: the size query shows which form a call takes, and both give the oracle's integers."""
import ctypes as C

import numpy as np
import pytest
import torch

import graphgen
import oracle

L = pytest.importorskip("paper_2108_00529_amd._lib", reason="libbgv.so not built")

#        edges, rows, cols, grouped
CASES = [((1 << 20) - 1, 1, 1 << 18, False), (1 << 20, 1, 1 << 18, True), (1 << 20, 1, (1 << 18) - 1, False),
         (700_000, 3, 349_526, True), (700_000, 3, 349_525, False), (699_050, 3, 349_526, False)]


@pytest.mark.parametrize("m,rows,cols,grouped", CASES)
def test_form(m, rows, cols, grouped):
    coef = C.cast((C.c_uint64 * 24)(), C.c_void_p)
    size = lambda c: L.bgv_supergraph_workspace(20_000, m, C.byref(L.SketchParams(rows, c, coef, coef)))
    # the grouped form holds an entry of 4 bytes per (edge, row); 200,000 cells never take it
    assert (size(cols) - size(200_000 // rows) >= 4 * rows * m) == grouped


@pytest.mark.gpu
@pytest.mark.parametrize("m,rows,cols,grouped", CASES)
def test_same_integers(m, rows, cols, grouped):
    import paper_2108_00529_amd as bgv
    n = 20_000
    rng = np.random.default_rng(m + rows)
    e = rng.integers(0, n, (m, 2)).astype(np.int32)
    lab = np.arange(n, dtype=np.int32)
    deg = np.bincount(e[e[:, 0] != e[:, 1]].ravel(), minlength=n).astype(np.int32)
    c1, c2 = graphgen.hash_coeffs(rows, 5), graphgen.hash_coeffs(rows, 6)
    ref = oracle.supergraph(n, e, lab, deg, rows, cols, c1, c2)
    sg = bgv.supergraph(torch.from_numpy(e).cuda(), torch.from_numpy(lab).cuda(), torch.from_numpy(deg).cuda(), rows,
                        cols, c1, c2, exact_counts=True)
    for k in ("M2", "se_weight", "se_count"):
        np.testing.assert_array_equal(sg[k].cpu().numpy().view(np.uint32), ref[k], err_msg=k)

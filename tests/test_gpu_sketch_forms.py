"""The forms of sketch 2 against the oracle on both sides of each line between them: in LDS up
to 16,384 cells, by device atomics, and grouped by buckets from 2^18 cells and 2^22 additions
on (buckets of 2^14 cells and, from 2^23 on, 2^15; tiles of 2,048 pairs above five rows), with
pairs of more edges than a grouped entry's count field holds."""
import numpy as np
import pytest
import torch

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


@pytest.mark.parametrize("m,rows,cols", [
    (40_000, 4, 4096), (40_000, 4, 4097), (900_000, 1, 16_384), (900_000, 1, 16_385), (900_000, 3, 7),
    (838_860, 5, 52_429), (838_861, 5, 52_428), (838_861, 5, 52_429), (700_000, 6, 43_691), (700_000, 8, 1 << 20),
    (4_194_303, 1, 1 << 18), (4_194_304, 1, 1 << 18)])
def test_sketch_two_forms(bgv, m, rows, cols):
    n = 20_000
    rng = np.random.default_rng(m + rows)
    e = rng.integers(0, n, (m, 2)).astype(np.int32)
    e[: m // 8] = e[m // 8: m // 8 + 1]              # one pair of very many edges
    e[m // 8: m // 4] = e[m // 4: m // 4 + 1000][np.arange(m // 4 - m // 8) % 1000]  # and many of some
    lab = np.arange(n, dtype=np.int32)
    deg = np.bincount(e[e[:, 0] != e[:, 1]].ravel(), minlength=n).astype(np.int32)
    c1, c2 = graphgen.hash_coeffs(rows, 5), graphgen.hash_coeffs(rows, 6)
    ref = oracle.supergraph(n, e, lab, deg, rows, cols, c1, c2)
    sg = bgv.supergraph(torch.from_numpy(e).cuda(), torch.from_numpy(lab).cuda(), torch.from_numpy(deg).cuda(), rows,
                        cols, c1, c2, exact_counts=True)
    assert sg["E"] == len(ref["superedges"])
    for k in ("M2", "se_weight", "se_count"):
        np.testing.assert_array_equal(sg[k].cpu().numpy().view(np.uint32), ref[k], err_msg=k)
    np.testing.assert_array_equal(sg["superedges"].cpu().numpy(), ref["superedges"])

"""The automatic choice of the community method on both sides of its line (16 + m / 2^17 chunk
steps with one pass, 15 + (passes + 1) m / 2^18 with more): the labels, degrees and volumes
are the oracle's whichever method it takes."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


@pytest.mark.parametrize("m,passes,line", [(5_000, 1, 16), (5_000, 3, 15), (200_000, 4, 18), (2_000_000, 1, 31),
                                           (2_000_000, 2, 37)])
@pytest.mark.parametrize("past", [0, 1])
def test_both_sides_of_the_line(bgv, m, passes, line, past):
    n, chunks = m // 8, (line + past * passes) // passes  # the most chunks at the line, or one more
    rng = np.random.default_rng(m + passes)
    u = rng.integers(0, n, m)
    e = np.stack([u, (u + rng.integers(0, 50, m)) % n], 1).astype(np.int32)
    chunk = -(-m // chunks)
    lab, cnt = oracle.bs_community(n, e, 16, passes, 2, chunk)
    deg, vol = oracle.degree_volume(lab, cnt, passes)
    got = bgv.community(torch.from_numpy(e).cuda(), n, 16, passes, 2, chunk, volume=True)
    for a, b in zip(got, (lab, deg, vol)):
        np.testing.assert_array_equal(a.cpu().numpy(), b)

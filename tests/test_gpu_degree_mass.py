"""The energy's degree-based masses, counted without the rows: equal to a call that is given
the same masses, and to the sum of the definition, for no superedge, a hub of every superedge,
repeated superedges and more nodes than a counting workgroup's table holds."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


@pytest.mark.parametrize("K,E,kind", [(1, 0, "none"), (2, 1, "random"), (50, 0, "none"), (2047, 30_000, "random"),
                                      (2049, 30_000, "hub"), (20_479, 200_000, "random"), (20_481, 5_000, "random"),
                                      (5_000, 300_000, "repeated")])
def test_energy_with_counted_masses(bgv, K, E, kind):
    rng = np.random.default_rng(K)
    e = np.sort(rng.integers(0, K, (E, 2)), 1)
    e = e[e[:, 0] != e[:, 1]] if kind != "hub" else np.stack([np.zeros(E, np.int64), rng.integers(1, K, E)], 1)
    if kind == "repeated":
        e[: E // 2] = (0, 1)
    se = torch.from_numpy(e.astype(np.int32)).cuda()
    pos = torch.from_numpy(rng.uniform(-50, 50, (K, 2)).astype(np.float32)).cuda()
    mass = np.bincount(e.ravel(), minlength=K).astype(np.float32) + 1.0
    counted = bgv.fa2_energy(se, pos, kr=1.0, kg=1.0)
    given = bgv.fa2_energy(se, pos, kr=1.0, kg=1.0, mass=torch.from_numpy(mass).cuda())
    assert float(counted) == float(given)

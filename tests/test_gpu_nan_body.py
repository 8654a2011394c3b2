"""A body with one coordinate that is not a number: every pair with it is dropped along the
other axis (the test |x_i - x_j|^2 > 0 fails), so the other bodies' forces there are those
without it, in every kernel (one workgroup, segments, two bodies per thread)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

SE = np.zeros((0, 2), np.int32)


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("K", [2, 9, 448, 449, 4001, 16385, 45057])
def test_other_axis(K, axis):
    import paper_2108_00529_amd as bgv
    rng = np.random.default_rng(K)
    pos, mass = rng.uniform(-4, 4, (K, 2)).astype(np.float32), rng.uniform(1, 9, K).astype(np.float32)
    bad = K // 2
    pos[bad, axis] = np.nan
    x, m, se = (torch.from_numpy(a).cuda() for a in (pos, mass, SE))
    keep = np.arange(K) != bad
    grad = bgv.fa2_grad(se, x, mass=m).cpu().numpy()
    _, force, _ = bgv.fa2_layout(se, x.clone(), 1, exact=True, mass=m)
    ref = oracle.fa2_forces(pos[keep].astype(np.float64), SE, mass[keep].astype(np.float64), exact=True)
    # the tolerance of the other tests of these kernels: 1e-4 of the largest force
    for f in (-grad, force.cpu().numpy()):
        assert np.abs(f[keep, 1 - axis] - ref[:, 1 - axis]).max() <= 1e-4 * np.linalg.norm(ref, axis=1).max()

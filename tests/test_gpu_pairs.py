"""The all-pairs kernels at the sizes where their shape changes (tiles of 256 bodies,
segments of 512, two bodies per thread from 16,384 on) with coincident bodies and pairs
whose squared distance is subnormal, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

SE = np.zeros((0, 2), np.int32)


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


def bodies(K):
    rng = np.random.default_rng(K)
    pos = rng.uniform(-4, 4, (K, 2)).astype(np.float32)
    pos[K // 3] = pos[0]                                   # coincident, in another tile
    pos[K // 2: K // 2 + 3] = pos[K - 1]                   # and three in a row with the last
    if K > 8:
        pos[5] = 0.0                                       # and two so near that d^2 is subnormal
        pos[7] = (1e-20, 0.0)
    return pos, rng.uniform(1, 9, K).astype(np.float32)


# FP32 terms of either sign, summed 256 (energy) or 512 (force) at a time: the rounding of a
# sum stays below 1e-6 of the sum of its terms' sizes, which the energy's and the largest
# force's scales exceed here; the tolerance of the other layout tests is 1e-4.
@pytest.mark.parametrize("K", [7, 8, 9, 255, 256, 257, 511, 512, 513, 769, 4001, 16383, 16384, 16385, 16641, 17000])
def test_pairs(bgv, K):
    pos, mass = bodies(K)
    x, m, se = (torch.from_numpy(a).cuda() for a in (pos, mass, SE))
    near = 7 if K > 8 else None                            # its force is about 1e20: checked for being finite
    keep = np.ones(K, bool)
    if near:
        keep[[5, 7]] = False
    ref = oracle.fa2_forces(pos.astype(np.float64), SE, mass.astype(np.float64), exact=True)
    scale = np.linalg.norm(ref[keep], axis=1).max()
    grad = bgv.fa2_grad(se, x, mass=m).cpu().numpy()
    _, force, _ = bgv.fa2_layout(se, x.clone(), 1, exact=True, mass=m)
    for f in (-grad, force.cpu().numpy()):
        assert np.linalg.norm(f[keep] - ref[keep], axis=1).max() <= 1e-4 * scale
    e_ref = oracle.fa2_energy(pos.astype(np.float64), SE, mass.astype(np.float64))
    e = float(bgv.fa2_energy(se, x, mass=m))
    assert abs(e - e_ref) <= 1e-5 * max(1.0, abs(e_ref))


@pytest.mark.parametrize("K", [45_055, 45_056, 45_313])
def test_forces_around_two_bodies_per_thread(bgv, K):
    """The layout's forces where it goes over to two bodies per thread against the gradient
    kernel's, which has gone over long before; the tolerance is that of test_pairs."""
    pos, mass = bodies(K)
    x, m, se = (torch.from_numpy(a).cuda() for a in (pos, mass, SE))
    keep = np.ones(K, bool)
    keep[[5, 7]] = False
    grad = bgv.fa2_grad(se, x, mass=m).cpu().numpy()
    _, force, _ = bgv.fa2_layout(se, x.clone(), 1, exact=True, mass=m)
    scale = np.linalg.norm(grad[keep], axis=1).max()
    assert np.linalg.norm(force.cpu().numpy()[keep] + grad[keep], axis=1).max() <= 1e-4 * scale

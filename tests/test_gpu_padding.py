"""The loops over all pairs take bodies in groups of eight; a last group that is not full must
add nothing, also to a body close to the origin.  Forces, gradient and energy of one body at
(1e-20, 0) among bodies that are not near it, at counts that leave groups partly filled in
every kernel (one workgroup, segments, two bodies per thread, the batched form's three),
against the FP64 oracle and against the same bodies filled up with massless far ones."""
import numpy as np
import pytest
import torch

import graphgen
import oracle

pytestmark = pytest.mark.gpu

SE = np.zeros((0, 2), np.int32)


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


def bodies(K):
    rng = np.random.default_rng(K)
    r, a = rng.uniform(1, 4, K), rng.uniform(0, 2 * np.pi, K)  # none within 1 of the origin
    pos = np.stack([r * np.cos(a), r * np.sin(a)], 1).astype(np.float32)
    pos[0] = (1e-20, 0.0)
    return pos, rng.uniform(1, 9, K).astype(np.float32)


def forces(bgv, pos, mass):
    x, m, se = (torch.from_numpy(a).cuda() for a in (pos, mass, SE))
    grad = bgv.fa2_grad(se, x, mass=m).cpu().numpy()
    _, force, _ = bgv.fa2_layout(se, x.clone(), 1, exact=True, mass=m)
    return -grad, force.cpu().numpy(), float(bgv.fa2_energy(se, x, mass=m))


# the tolerances of the other tests of these kernels: 1e-4 of the largest force, 1e-5 of the
# energy's terms
@pytest.mark.parametrize("K", [1, 7, 9, 255, 257, 449, 513, 4001, 16385, 45057])
def test_forces_and_energy(bgv, K):
    pos, mass = bodies(K)
    grad, force, energy = forces(bgv, pos, mass)
    ref = oracle.fa2_forces(pos.astype(np.float64), SE, mass.astype(np.float64), exact=True)
    scale = np.linalg.norm(ref, axis=1).max()
    for f in (grad, force):
        assert np.linalg.norm(f - ref, axis=1).max() <= 1e-4 * scale
    e_ref = oracle.fa2_energy(pos.astype(np.float64), SE, mass.astype(np.float64))
    assert abs(energy - e_ref) <= 1e-5 * max(1.0, abs(e_ref))


@pytest.mark.parametrize("K", [1, 7, 9, 257, 513])
def test_filled_up_by_the_caller(bgv, K):
    pos, mass = bodies(K)
    more = -K % 8
    far = np.tile(np.float32([[1e3, 1e3]]), (more, 1))
    a = forces(bgv, pos, mass)
    b = forces(bgv, np.concatenate([pos, far]), np.concatenate([mass, np.zeros(more, np.float32)]))
    for f, g in zip(a[:2], b[:2]):
        assert np.isfinite(f).all()
        np.testing.assert_array_equal(f, g[:K])


@pytest.mark.parametrize("wg_threads,big_k", [(256, 0), (512, 0), (1024, 0), (512, 1)])
def test_batched(bgv, wg_threads, big_k):
    # threshold 0: every node is a supernode; a path, so masses are 2 and 3
    sizes = [2, 7, 9, 257, 513, 1025]
    wl = dict(graphgen.WORKLOADS["batched_512"], threshold=0, fa2_iters=1)
    c1 = graphgen.hash_coeffs(wl["rows"], 3)
    path = lambda n: np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32)
    edges, noff, eoff, noff_h, _ = bgv.pack_graphs([(n, path(n)) for n in sizes], torch.device("cuda"))
    pos0 = np.concatenate([bodies(n)[0] for n in sizes])
    out = bgv.batched(edges, noff, eoff, int(noff_h[-1]), wl, c1, c1, torch.from_numpy(pos0).cuda(),
                      wg_threads=wg_threads, big_k=big_k)
    assert out["K"].tolist() == sizes
    for g, n in enumerate(sizes):
        a, b = int(noff_h[g]), int(noff_h[g + 1])
        ref = oracle.fa2_forces(pos0[a:b].astype(np.float64), path(n), oracle.fa2_mass(n, path(n)), kr=wl["kr"],
                                kg=wl["kg"], exact=True)
        err = np.linalg.norm(out["fprev"][a:b].cpu().numpy() - ref, axis=1).max()
        assert err <= 1e-4 * np.linalg.norm(ref, axis=1).max(), n

"""Exact layouts small enough for one workgroup (up to 448 supernodes) and the first ones
past it: one step against the FP64 oracle, run-to-run and split-run equality, with rows of
no entry, of more than 64 and more than 1,024 entries and more neighbour ids than LDS holds."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def superedges(K, kind):
    rng = np.random.default_rng(K)
    if K < 2 or kind == "none":
        return np.zeros((0, 2), np.int32)
    if kind == "star":  # one row of K - 1 entries, and the last node alone
        return np.stack([np.zeros(K - 2, np.int64), np.arange(1, K - 1)], 1).astype(np.int32)
    E = 20_000 if kind == "many" else 12 * K
    u = rng.integers(0, K - 1, E)
    e = np.stack([u, u + 1 + rng.integers(0, 2**31, E) % (K - 1 - u)], 1).astype(np.int32)
    if kind == "many":
        e[:1500] = (0, 1)  # two rows cut into blocks
    return e


# the layout tests' tolerance: 1e-4 of the largest sum of a node's force components
@pytest.mark.parametrize("K", [1, 2, 3, 63, 64, 65, 255, 256, 257, 447, 448, 449])
@pytest.mark.parametrize("kind", ["none", "star", "plain", "many"])
@pytest.mark.parametrize("weighted", [False, True])
def test_step(bgv, K, kind, weighted):
    rng = np.random.default_rng(7 * K)
    se = superedges(K, kind)
    w = rng.uniform(0.5, 2, len(se)).astype(np.float32) if weighted and len(se) else None
    pos = rng.uniform(-5, 5, (K, 2)).astype(np.float32)
    fprev = rng.uniform(-3, 3, (K, 2)).astype(np.float32)
    kw = dict(exact=True, attr_w=None if w is None else dev(w))
    args = lambda: dict(fprev=dev(fprev), speed=torch.full((1,), 0.7, device="cuda"), **kw)
    p, f, s = bgv.fa2_layout(dev(se), dev(pos), 1, **args())
    mass = oracle.fa2_mass(K, se)
    x64 = pos.astype(np.float64)
    parts = [oracle.fa2_forces(x64, se, mass, w, kr=kr, kg=kg, exact=True) for kr, kg in ((1, 0), (0, 1), (0, 0))]
    scale = max(np.linalg.norm(parts[0] - parts[2], axis=1).max(), np.linalg.norm(parts[2], axis=1).max(), 1e-3)
    ref = parts[0] + parts[1] - parts[2]
    assert np.linalg.norm(f.cpu().numpy() - ref, axis=1).max() <= 1e-4 * scale
    # the step itself, from the forces that were returned
    F, Fp = f.cpu().numpy().astype(np.float64), fprev.astype(np.float64)
    swing, trac = np.linalg.norm(F - Fp, axis=1), 0.5 * np.linalg.norm(F + Fp, axis=1)
    sp = min((mass * trac).sum() / (mass * swing).sum(), 1.5 * 0.7)
    assert abs(float(s) - sp) <= 1e-5 * sp
    fn = np.linalg.norm(F, axis=1)
    local = np.minimum(0.1 * sp / (1 + sp * np.sqrt(swing)), 10 / np.maximum(fn, 1e-30))
    want = x64 + local[:, None] * F
    assert np.abs(p.cpu().numpy() - want).max() <= 1e-5 * max(1.0, np.abs(want).max())
    # five iterations, and two and three
    a = bgv.fa2_layout(dev(se), dev(pos), 5, **args())
    b = bgv.fa2_layout(dev(se), dev(pos), 2, **args())
    b = bgv.fa2_layout(dev(se), b[0], 3, fprev=b[1], speed=b[2], **kw)
    for u, v in zip(a, b):
        assert torch.equal(u, v)

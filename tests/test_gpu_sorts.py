"""The one-sweep sorts at the key counts where their tiles change (65,536 and 2^20 keys) and
one key to either side, through the calls that run them: back-pointer communities (32- and
64-bit keys with values) against the chunk-by-chunk form, and superedge rows with and
without weights (keys of 32 and 64 bits) against sums in FP64."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


# 512 edges fill a wavefront's tile
@pytest.mark.parametrize("n,chunk", [(3000, 5000), (200_000, 40)])
@pytest.mark.parametrize("m", [1, 511, 512, 513, 32_767, 32_768, 32_769, 524_288, 524_289])
def test_occurrence_and_event_sorts(bgv, n, chunk, m):
    rng = np.random.default_rng(m)
    e = rng.integers(0, n, (m, 2)).astype(np.int32)
    e[rng.random(m) < 0.2, 0] = rng.integers(0, 5)
    e = torch.from_numpy(e).cuda()
    got = bgv.community(e, n, 9, 2, 2, max(1, min(chunk, m)), volume=True, method=2)
    want = bgv.community(e, n, 9, 2, 2, max(1, min(chunk, m)), volume=True, method=1)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_events_past_one_workgroups_scan(bgv):
    """16,384 tiles of 512 proposals is the most that one workgroup scans."""
    test_occurrence_and_event_sorts(bgv, 200_000, 300_000, 16_384 * 512 // 2 + 1)


# rows of up to a few thousand FP32 terms: far inside the 1e-4 of the other force tests
@pytest.mark.parametrize("K", [300, 70_000])
@pytest.mark.parametrize("E", [32_767, 32_768, 32_769, 524_289])
@pytest.mark.parametrize("weighted", [False, True])
def test_row_sorts(bgv, K, E, weighted):
    rng = np.random.default_rng(E)
    pos = rng.uniform(-3, 3, (K, 2)).astype(np.float32)
    u = rng.integers(0, K - 1, E)
    se = np.stack([u, u + 1 + rng.integers(0, 2**31, E) % (K - 1 - u)], 1).astype(np.int32)
    w = rng.uniform(0.5, 4, E).astype(np.float32) if weighted else None
    mass = np.full(K, 1e-3, np.float32)  # attraction alone decides the force
    _, f, _ = bgv.fa2_layout(torch.from_numpy(se).cuda(), torch.from_numpy(pos).cuda(), 1, exact=False,
                             kr=0.0, kg=0.0, mass=torch.from_numpy(mass).cuda(),
                             attr_w=None if w is None else torch.from_numpy(w).cuda())
    x, a = pos.astype(np.float64), np.ones(E) if w is None else w.astype(np.float64)
    ref = np.zeros((K, 2))
    d = a[:, None] * (x[se[:, 1]] - x[se[:, 0]])
    np.add.at(ref, se[:, 0], d)
    np.add.at(ref, se[:, 1], -d)
    assert np.abs(f.cpu().numpy() - ref).max() <= 1e-4 * np.abs(ref).max()

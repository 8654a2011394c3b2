"""The Morton order of the Barnes-Hut bodies at the sizes where its sort changes (tiles of 256
bodies, one or four bodies per thread, the largest bucket count, the radix sort above), for
positions that make buckets of every size: the order is that of a stable sort of the codes,
and it does not depend on the order that the sample was taken from."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


def spread(v):
    v = v.astype(np.uint32)
    for s, m in ((8, 0x00FF00FF), (4, 0x0F0F0F0F), (2, 0x33333333), (1, 0x55555555)):
        v = (v | (v << np.uint32(s))) & np.uint32(m)
    return v


def codes(p):
    lo, hi = p.min(0), p.max(0)
    s0 = np.float32(max(hi[0] - lo[0], hi[1] - lo[1]))
    s0 = s0 if s0 > 0 else np.float32(1)
    q = np.minimum(((p - lo) / s0 * np.float32(65536)).astype(np.int32), 65535)
    return spread(q[:, 0]) | (spread(q[:, 1]) << np.uint32(1))


def positions(K, kind):
    rng = np.random.default_rng(K)
    p = rng.uniform(-50, 50, (K, 2)).astype(np.float32)
    if kind == "equal":
        p[:] = p[0]
    elif kind == "clustered":  # a few points hold almost everything
        c = rng.integers(0, min(K, 5), K)
        p = np.where(rng.random((K, 1)) < 0.05, p, p[c])
    elif kind == "grid":
        w = int(np.sqrt(K)) + 1
        i = np.arange(K)
        p = np.stack([i % w, i // w], 1).astype(np.float32)
    elif kind == "unsampled":  # the sampled bodies in one spot: one bucket holds the others
        NB = min(1024, -(-K // 192))
        q = np.arange(1, NB, dtype=np.uint64)
        b = (q * 2654435761 % 2**32 * np.uint64(K)) >> np.uint64(32)
        p[b.astype(np.int64)] = (-50.0, -50.0)
    return p


@pytest.mark.parametrize("kind", ["uniform", "equal", "clustered", "grid", "unsampled"])
@pytest.mark.parametrize("K", [1, 2, 191, 192, 193, 255, 256, 257, 4000, 17_000, 65_536, 65_537, 98_305, 184_320, 184_321, 262_144, 262_145])
def test_order_is_the_stable_sort_of_the_codes(bgv, K, kind):
    p = positions(K, kind)
    t = bgv.bh_tree(torch.from_numpy(p).cuda(), torch.ones(K, device="cuda"))
    c = codes(p)
    want = np.argsort(c, kind="stable")
    body = t["body"].cpu().numpy()
    assert np.array_equal(t["codes"].cpu().numpy().view(np.uint32), c[want])
    assert np.array_equal(body[:, 3].view(np.int32), want)
    assert np.array_equal(body[:, :2], p[want])


@pytest.mark.parametrize("K,ks", [(300, 0.1), (5_000, 0.1), (5_000, 50.0), (70_000, 50.0)])
def test_one_call_equals_calls_of_one_iteration(bgv, K, ks):
    """A call's later iterations sample the order before them, a call's first one does not."""
    rng = np.random.default_rng(K)
    se = rng.integers(0, K, (4 * K, 2))
    se = np.unique(np.sort(se[se[:, 0] != se[:, 1]], 1), axis=0).astype(np.int32)
    e, p0 = torch.from_numpy(se).cuda(), torch.from_numpy(positions(K, "clustered")).cuda()
    kw = dict(exact=False, theta=1.2, ks=ks, ksmax=100.0 * ks)
    one = bgv.fa2_layout(e, p0.clone(), 4, **kw)
    p, f, s = bgv.fa2_layout(e, p0.clone(), 1, **kw)
    for _ in range(3):
        p, f, s = bgv.fa2_layout(e, p, 1, fprev=f, speed=s, **kw)
    assert torch.equal(one[0], p) and torch.equal(one[1], f) and float(one[2]) == float(s)


# a node's centre is a difference of FP64 prefix sums (error below K * 50 * 2^-52 over its
# mass) rounded to float32 (50 * 2^-24): 1e-5 holds both; masses of 1 sum exactly
@pytest.mark.parametrize("K", [2, 255, 256, 257, 4000, 65_536, 65_537, 70_000, 262_145])
def test_node_masses_and_centres(bgv, K):
    p = positions(K, "clustered")
    t = bgv.bh_tree(torch.from_numpy(p).cuda(), torch.ones(K, device="cuda"))
    a, r = t["nodeA"].cpu().numpy(), t["nodeB"].cpu().numpy()
    body = t["body"].cpu().numpy().astype(np.float64)
    first, last = r[:, 2], r[:, 3]
    assert np.array_equal(a[:, 2], (last - first + 1).astype(np.float32))
    for c in (0, 1):
        s = np.concatenate([[0.0], np.cumsum(body[:, c])])
        np.testing.assert_allclose(a[:, c], (s[last + 1] - s[first]) / (last - first + 1), rtol=0, atol=1e-5)

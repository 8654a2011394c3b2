"""Community volumes where one community holds most nodes and thousands of others collide
in the workgroups' tables, against a plain count over the returned labels and degrees."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


def giant_and_pairs(n, seed):
    """Two thirds of the nodes meet one of three hubs; the others meet a neighbour."""
    rng = np.random.default_rng(seed)
    name = rng.permutation(n)
    k = 2 * n // 3
    u = np.concatenate([np.arange(3, k), np.arange(k, n - 1)])
    v = np.concatenate([rng.integers(0, 3, max(0, k - 3)), np.arange(k + 1, n)])
    e = np.stack([name[u], name[v]], 1)
    return np.concatenate([e, e[::2]])[rng.permutation(len(u) + (len(u) + 1) // 2)].astype(np.int32)


# 1,024 nodes fill one workgroup's threads, 524,288 the whole grid
@pytest.mark.parametrize("n", [5, 1023, 1025, 20_000, 524_288 + 1_100])
@pytest.mark.parametrize("method,rule,chunk", [(1, 0, 4096), (2, 0, 64), (0, 1, 100_000)])
def test_volume_is_the_sum_of_degrees(bgv, n, method, rule, chunk):
    e = torch.from_numpy(giant_and_pairs(n, n)).cuda()
    labels, degree, volume = bgv.community(e, n, 1 << 20, 2, 2, chunk, volume=True, method=method, rule=rule)
    lab, deg = labels.cpu().numpy(), degree.cpu().numpy().astype(np.int64)
    want = np.zeros(n, np.int64)
    np.add.at(want, lab, deg)
    assert np.array_equal(deg, np.bincount(e.cpu().numpy().ravel(), minlength=n))
    assert np.array_equal(volume.cpu().numpy(), want)


# the grouped form of the volume rule takes chunks of at least n / 8192 edges above 2^20
# nodes, and buckets of 2^13 ids from 2^21 nodes on
@pytest.mark.parametrize("n,chunk", [((1 << 20) + 1, 129), ((1 << 20) + 1, 128), ((1 << 21) - 1, 256),
                                     ((1 << 21) + 3, 257), ((1 << 21) + 3, 256), ((1 << 21) + 3, 3000),
                                     (1 << 20, 70)])
def test_volume_rule_forms(bgv, n, chunk):
    rng = np.random.default_rng(chunk)
    ids = np.concatenate([rng.integers(0, 2000, 700), rng.integers(n - 9000, n, 900), rng.integers(0, n, 900)])
    e = ids[rng.integers(0, len(ids), (9_000, 2))].astype(np.int32)
    e[rng.random(len(e)) < 0.1, 0] = n - 1
    ref = [oracle.bs_community(n, e, 5, p, 2, chunk, rule=1) for p in (1, 2)]
    deg, vol = oracle.degree_volume(*ref[1], 2)
    labels, degree, volume, rows = bgv.community_passes(torch.from_numpy(e).cuda(), n, 5, 2, 2, chunk, volume=True,
                                                        rule=1)
    assert np.array_equal(rows.cpu().numpy(), np.stack([r[0] for r in ref]))
    assert np.array_equal(labels.cpu().numpy(), ref[1][0])
    assert np.array_equal(degree.cpu().numpy(), deg)
    assert np.array_equal(volume.cpu().numpy(), vol)
    again, _, _ = bgv.community_resume(torch.from_numpy(e).cuda(), n, rows[0].contiguous(), 1, 5, 2, 2, chunk, rule=1)
    assert torch.equal(again, labels)

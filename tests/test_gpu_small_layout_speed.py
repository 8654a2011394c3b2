"""Where the layouts of a few hundred supernodes by one workgroup cost more than another form or
size, they were taken all the same; the bounds leave the measured times a factor of 1.5 and
more (shortest of several runs)."""
import numpy as np
import pytest
import torch

import graphgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


def shortest(run, n=5):
    times = []
    for _ in range(n):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        torch.cuda.synchronize()
        a.record()
        run()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


@pytest.mark.parametrize("wg_threads", [0, 1024])
def test_batched_440_no_longer_than_500(bgv, wg_threads):
    """440 supernodes leave one of 512 threads' wavefronts to the rows, 500 none (so all take
    them): the smaller graphs took three times as long."""
    wl = dict(graphgen.WORKLOADS["batched_512"], threshold=0, fa2_iters=100)  # every node a supernode
    c1 = graphgen.hash_coeffs(wl["rows"], 3)
    ms = []
    for n in (440, 500):
        rng = np.random.default_rng(n)
        u = rng.integers(0, n, 16 * n)
        e = np.stack([u, (u + 1 + rng.integers(0, n - 1, 16 * n)) % n], 1).astype(np.int32)
        edges, noff, eoff, noff_h, _ = bgv.pack_graphs([(n, e)] * 32, torch.device("cuda"))
        pos = torch.from_numpy(np.random.default_rng(1).uniform(-1, 1, (32 * n, 2)).astype(np.float32)).cuda()
        ms.append(shortest(lambda: bgv.batched(edges, noff, eoff, 32 * n, wl, c1, c1, pos.clone(),
                                               wg_threads=wg_threads)))
    assert ms[0] <= 1.3 * ms[1], ms


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("K", [192, 448])
def test_dense_layout_of_one_graph(bgv, K, weighted):
    """Every pair eight times: one workgroup took two to twelve times as long as three launches
    per iteration, which 449 supernodes have always taken."""
    ms = []
    for n in (K, 449):
        u, v = np.triu_indices(n, 1)
        se = torch.from_numpy(np.tile(np.stack([u, v], 1), (8, 1)).astype(np.int32)).cuda()
        w = torch.full((se.shape[0],), 0.5, device="cuda") if weighted else None
        pos = torch.from_numpy(np.random.default_rng(1).uniform(-1, 1, (n, 2)).astype(np.float32)).cuda()
        ms.append(shortest(lambda: bgv.fa2_layout(se, pos.clone(), 100, exact=True, attr_w=w)))
    assert ms[0] <= 1.3 * ms[1], ms

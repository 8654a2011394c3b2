"""The batched form at the supergraph sizes where its layout changes hands: 512 (state on
chip in the persistent launch), whole segments of 512 bodies, 2,048 (positions in LDS for
the attraction) and 4,096 (the multi-workgroup kernels' largest), with rows of one, of more
than 64 and of more than 1,024 entries and more neighbour ids than LDS holds.  Positions,
forces and speeds equal a plain layout's bit for bit: the additions are the same."""
import numpy as np
import pytest
import torch

import graphgen
import oracle

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 65, 256, 511, 512, 513, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097]


@pytest.fixture(scope="module")
def bgv():
    import paper_2108_00529_amd as b
    return b


@pytest.fixture(scope="module")
def batch():
    # threshold 0: no node ever moves, so the supergraph has every node of the graph
    wl = dict(graphgen.WORKLOADS["batched_512"], threshold=0, fa2_iters=3)
    c1 = graphgen.hash_coeffs(wl["rows"], wl["sketch_seed"])
    c2 = graphgen.hash_coeffs(wl["rows"], wl["sketch_seed"] ^ 0x9E3779B97F4A7C15)
    graphs = []
    for n in SIZES:
        rng = np.random.default_rng(n)
        e = rng.integers(0, n, ((20 if n == 512 else 4) * n, 2))
        star = np.stack([np.zeros(n, np.int64), np.arange(n)], 1)  # one row of n - 1 entries
        e = np.concatenate([e, star]).astype(np.int32)
        lab, cnt = oracle.bs_community(n, e, wl["threshold"], wl["passes"], wl["growth"], wl["chunk"])
        deg, _ = oracle.degree_volume(lab, cnt, wl["passes"])
        ref = oracle.supergraph(n, e, lab, deg, wl["rows"], wl["cols"], c1, c2)
        assert ref["K"] == n
        graphs.append((n, e, ref["superedges"], graphgen.initial_positions(n, 5 + n)))
    return wl, c1, c2, graphs


@pytest.mark.parametrize("wg_threads,big_k", [(256, 0), (512, 0), (1024, 0), (512, 1), (1024, 512)])
def test_every_size_equals_the_plain_layout(bgv, batch, wg_threads, big_k):
    wl, c1, c2, graphs = batch
    dev = torch.device("cuda")
    edges, noff, eoff, noff_h, _ = bgv.pack_graphs([(n, e) for n, e, _, _ in graphs], dev)
    pos = torch.from_numpy(np.concatenate([p for _, _, _, p in graphs])).to(dev)
    out = bgv.batched(edges, noff, eoff, int(noff_h[-1]), wl, c1, c2, pos, wg_threads=wg_threads, big_k=big_k)
    for g, (n, _, se, p0) in enumerate(graphs):
        a, b = int(noff_h[g]), int(noff_h[g + 1])
        p, f, s = bgv.fa2_layout(torch.from_numpy(se).cuda(), torch.from_numpy(p0).cuda(), wl["fa2_iters"], exact=True,
                                 kr=wl["kr"], kg=wl["kg"], tau=wl["tau"], ks=wl["ks"], ksmax=wl["ksmax"])
        assert int(out["K"][g]) == n
        assert torch.equal(out["pos"][a:b], p), n
        assert torch.equal(out["fprev"][a:b], f) and float(out["speed"][g]) == float(s), n


@pytest.mark.parametrize("chunk", [1, 2, 255, 256, 257, 512, 1024, 1025, 100_000])
@pytest.mark.parametrize("wg_threads,passes,tie", [(256, 3, 0), (1024, 2, 1)])
def test_chunks_of_one_edge_per_thread_and_of_more(bgv, chunk, wg_threads, passes, tie):
    """Chunks that leave each thread one edge at most and larger ones: labels and degrees are
    the oracle's (graphs of no, fewer than, just as many and more edges than a chunk, loops,
    repeated edges)."""
    wl = dict(graphgen.WORKLOADS["batched_512"], passes=passes, chunk=chunk, tie=tie, fa2_iters=0)
    c1 = graphgen.hash_coeffs(wl["rows"], 3)
    rng = np.random.default_rng(chunk)
    graphs = [(5, np.zeros((0, 2), np.int32))]
    for n, m in ((3, 1), (40, 255), (40, 256), (40, 257), (300, 1024), (300, 1025), (900, 6000)):
        e = rng.integers(0, n, (m, 2))
        e[m // 2: m // 2 + m // 8] = e[0]
        graphs.append((n, e.astype(np.int32)))
    dev = torch.device("cuda")
    edges, noff, eoff, noff_h, _ = bgv.pack_graphs(graphs, dev)
    pos = torch.zeros((int(noff_h[-1]), 2), device=dev)
    out = bgv.batched(edges, noff, eoff, int(noff_h[-1]), wl, c1, c1, pos, wg_threads=wg_threads)
    for g, (n, e) in enumerate(graphs):
        lab, cnt = oracle.bs_community(n, e, wl["threshold"], passes, wl["growth"], chunk, tie)
        deg, _ = oracle.degree_volume(lab, cnt, passes)
        a, b = int(noff_h[g]), int(noff_h[g + 1])
        np.testing.assert_array_equal(out["labels"][a:b].cpu().numpy(), lab)
        np.testing.assert_array_equal(out["degree"][a:b].cpu().numpy(), deg)

"""Kernels whose workgroups wait for one another within a launch: a workgroup may wait only for
such as have started, and workgroup numbers do not say who has (the XCDs start theirs
independently of each other, and a kernel on another stream can hold one of them up)."""
import os
import re

import numpy as np
import pytest

import graphgen

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2108_00529_amd", "csrc")


def kernels():
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        for m in re.finditer(r"__global__[^;{]*?\b(k_\w+)\(", text):
            at = text.index("{", m.end())
            depth, end = 1, at + 1
            while depth:
                depth += {"{": 1, "}": -1}.get(text[end], 0)
                end += 1
            yield m.group(1), text[at:end]


def test_waiting_kernels_number_their_workgroups_by_start():
    """The place a waiting workgroup takes comes from a counter that workgroups raise as they
    start, and after that its number in the launch is not used."""
    waiting = {name: body for name, body in kernels() if re.search(r"\+\+spins|spins\+\+", body)}
    assert {"k_os_pass", "k_os_pass_keys", "k_bh_prefix"} <= set(waiting)
    for name, body in waiting.items():
        ticket = re.search(r"= (\(int32_t\))?atomicAdd\((counter|started), 1u\);", body)
        assert ticket, name
        assert "blockIdx" not in body[ticket.end():], name


@pytest.mark.gpu
def test_layout_beside_another_streams_work():
    """A Barnes-Hut layout beside a persistent launch that holds every compute unit: the same
    bits as alone."""
    import torch

    import paper_2108_00529_amd as bgv
    K, dev = 30_000, torch.device("cuda")
    rng = np.random.default_rng(5)
    u = rng.integers(0, K, 4 * K)
    se = np.stack([u, (u + 1 + rng.integers(0, K - 1, 4 * K)) % K], 1).astype(np.int32)
    se, pos = torch.from_numpy(se).to(dev), torch.from_numpy(rng.uniform(-1, 1, (K, 2)).astype(np.float32)).to(dev)
    alone = bgv.fa2_layout(se, pos.clone(), 30, exact=False)
    wl = dict(graphgen.WORKLOADS["batched_512"], threshold=0, fa2_iters=50)
    c1 = graphgen.hash_coeffs(wl["rows"], 3)
    graphs = []
    for g in range(600):
        n = 200 + g
        a = rng.integers(0, n, 3 * n)
        graphs.append((n, np.stack([a, (a + 1 + rng.integers(0, n - 1, 3 * n)) % n], 1).astype(np.int32)))
    edges, noff, eoff, noff_h, _ = bgv.pack_graphs(graphs, dev)
    bpos = torch.zeros((int(noff_h[-1]), 2), device=dev)
    torch.cuda.synchronize()
    other, own = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(other):
        kept = bgv.batched(edges, noff, eoff, int(noff_h[-1]), wl, c1, c1, bpos)
    with torch.cuda.stream(own):
        beside = [bgv.fa2_layout(se, pos.clone(), 30, exact=False) for _ in range(3)]
    torch.cuda.synchronize()
    del kept
    for run in beside:
        for a, b in zip(alone, run):
            assert torch.equal(a, b)

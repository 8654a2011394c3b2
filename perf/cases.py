"""The work that a user of this library has it do, as cases that can be timed: community
detection, the sketch supergraph, the ForceAtlas2 layout of a supergraph, the layout's
energy with its gradient, and the whole path for one graph or for many.

A case is a dict of plain values; "do" names the kind of work.  The graphs are drawn on
the GPU with the recipes of graphgen (planted partitions and LFR-style power-law graphs
with planted communities), in whole numbers wherever an order of summation could matter,
so a seed gives the same graph every time.  A case fixes the degrees, the communities and
the stream, and with them how many supernodes and superedges come out; the seed draws the
nodes' names, the hash coefficients, the positions and the weights.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2108_00529_amd as bgv

DEV = "cuda"
ROWS_MAX_CELLS = 8192  # the batched form keeps a graph's sketch on chip
SHAPE = 7  # seed of what a case fixes


def listed():
    return [
        # The smallest whole call: a 2,000-node planted graph from edges to a finished
        # exact layout (the bench's small graph).  Some 800 short launches.
        dict(name="pipeline_2k", do="pipeline", n=2000, blocks=8, p_in=0.04, p_out=0.0005, threshold=16, passes=1,
             chunk=256, rows=4, cols=1024, iters=200),
        # Many small graphs at once (the bench's batch of 512 uneven planted graphs), laid
        # out with its tuned launch shape.
        dict(name="batched_512", do="batched", graphs=512, median=2000, sigma=0.9, nmax=20000, threshold=16, passes=1,
             chunk=256, rows=4, cols=1024, iters=300, wg_threads=1024, big_k=32),
        # Communities of a small power-law graph with the default id check: an ordinary
        # interactive call, where launches and latency count.
        dict(name="community_20k", do="community", n=20000, m=200000, gamma=2.3, mu=0.2, threshold=32, passes=3,
             chunk=1 << 15, method=0, tie=0, rule=0, check=True),
        # The largest single graph (the bench's): 34M edges, three passes, chunks of 2^22.
        dict(name="community_3m", do="community", n=3_200_000, m=34_000_000, gamma=2.1, mu=0.3, threshold=128,
             passes=3, chunk=1 << 22, method=0, tie=0, rule=0, check=False),
        # The exact sequential rule (chunk 1) on a 10M-edge stream.
        dict(name="sequential_1m", do="community", n=1_000_000, m=10_000_000, gamma=2.3, mu=0.2, threshold=64,
             passes=3, chunk=1, method=0, tie=0, rule=0, check=False),
        # SCoDA's community-volume rule on the same kind of stream.
        dict(name="volume_1m", do="community", n=1_000_000, m=10_000_000, gamma=2.3, mu=0.2, threshold=64, passes=3,
             chunk=1 << 20, method=0, tie=0, rule=1, check=False),
        # The supergraph of a small graph with a small sketch and the default id check.
        dict(name="supergraph_20k", do="supergraph", n=20000, m=200000, gamma=2.3, mu=0.2, threshold=32, passes=3,
             chunk=1 << 15, rows=4, cols=1024, exact_counts=False, check=True),
        # The supergraph of the largest graph with its 5 x 2^22 sketch.
        dict(name="supergraph_3m", do="supergraph", n=3_200_000, m=34_000_000, gamma=2.1, mu=0.3, threshold=128,
             passes=3, chunk=1 << 22, rows=5, cols=1 << 22, exact_counts=False, check=False),
        # A viewer's step: two exact iterations that continue a layout of 4,001 supernodes
        # with weighted superedges and given masses.
        dict(name="layout_exact_4k", do="layout", supernodes=4001, superedges=60000, gamma=2.3, exact=True, iters=2,
             weighted=True, masses=True, fresh=False),
        # The Barnes-Hut layout of the supergraph of a 10M-edge graph.
        dict(name="layout_17k", do="layout", supernodes=17724, superedges=1_300_000, gamma=2.3, exact=False, iters=500,
             weighted=False, masses=False, fresh=True),
        # The same for the largest graph's supergraph.
        dict(name="layout_172k", do="layout", supernodes=171_724, superedges=12_184_115, gamma=2.1, exact=False,
             iters=200, weighted=False, masses=False, fresh=True),
        # One step of a gradient-based layout of 50,000 supernodes with sketch weights:
        # the energy forward and its gradient backward.
        dict(name="grad_50k", do="grad", supernodes=50_000, superedges=1_000_000, gamma=3.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["pipeline", "batched", "community", "community", "sequential", "volume", "supergraph",
                     "supergraph", "layout", "layout", "grad"])
    if do == "pipeline":
        n = _log(rng, 500, 5000)
        return dict(do=do, n=n, blocks=rng.randint(4, 16), p_in=80.0 / n, p_out=1.0 / n,
                    threshold=rng.choice([8, 16, 32]), passes=rng.randint(1, 3), chunk=_log(rng, 64, 4096),
                    rows=rng.randint(1, 5), cols=_log(rng, 200, 4000), iters=rng.randint(100, 300))
    if do == "batched":
        rows = rng.randint(2, 5)
        return dict(do=do, graphs=_log(rng, 8, 400), median=_log(rng, 300, 2000), sigma=rng.uniform(0.3, 0.9),
                    nmax=16000, threshold=rng.choice([8, 16, 32]), passes=rng.randint(1, 2), chunk=_log(rng, 128, 1024),
                    rows=rows, cols=_log(rng, 200, ROWS_MAX_CELLS // rows), iters=rng.randint(50, 300),
                    **rng.choice([dict(wg_threads=1024, big_k=32), dict(wg_threads=0, big_k=0)]))
    if do in ("community", "sequential", "volume", "supergraph"):
        n = _log(rng, 2000, 3_200_000 if do in ("community", "supergraph") else 1_000_000)
        m = int(n * rng.uniform(5.0, 10.6))
        c = dict(do="supergraph" if do == "supergraph" else "community", n=n, m=m, gamma=rng.uniform(2.1, 2.6),
                 mu=rng.uniform(0.1, 0.4), threshold=rng.choice([16, 64, 128, 300]), passes=rng.randint(1, 4),
                 chunk=1 if do == "sequential" else max(1, int(m / rng.uniform(1.0, 12.0))),
                 check=rng.random() < 0.5)
        if do == "supergraph":
            return dict(c, rows=rng.randint(1, 5), cols=_log(rng, 500, 1 << 22), exact_counts=rng.random() < 0.3)
        return dict(c, method=0, tie=0 if do == "volume" else rng.choice([0, 0, 1]), rule=1 if do == "volume" else 0)
    if do == "layout":
        exact = rng.random() < 0.4
        K = _log(rng, 300, 12000 if exact else 171_724)
        return dict(do=do, supernodes=K, superedges=int(K * rng.uniform(2.0, min(70.0, K / 20.0))),
                    gamma=rng.uniform(2.1, 3.0), exact=exact, iters=_log(rng, 1, 100 if exact else 200),
                    weighted=rng.random() < 0.4, masses=rng.random() < 0.4, fresh=rng.random() < 0.5)
    K = _log(rng, 500, 50_000)
    return dict(do=do, supernodes=K, superedges=int(K * rng.uniform(2.0, 20.0)), gamma=rng.uniform(2.3, 3.5))


# --------------------------------------------------------------------- inputs ----
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + salt) % (1 << 62))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _weights(g, n, m, gamma):
    """Expected degrees ~ Pareto(gamma), scaled to sum 2m, capped at sqrt(2m), in 1/1024."""
    w = (1.0 - _rand(g, n)) ** (-1.0 / (gamma - 1.0))
    w *= 2.0 * m / float(w.sum())
    return (w.clamp_(max=math.sqrt(2.0 * m)) * 1024.0).long() + 1


def _cum(w):
    return torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), torch.cumsum(w, 0)])


def _pick(g, cum, lo, hi):
    """Positions drawn in proportion to the weights within [lo, hi) of their running sum."""
    t = lo + (_rand(g, lo.shape[0]) * (hi - lo).double()).long()
    return torch.searchsorted(cum, torch.minimum(t, hi - 1), right=True) - 1


def _stream(g, u, v):
    """Random order and orientation of the edges, int32 (m, 2)."""
    swap = _rand(g, u.shape[0]) < 0.5
    e = torch.stack([torch.where(swap, v, u), torch.where(swap, u, v)], 1).int()
    return e[torch.randperm(u.shape[0], generator=g, device=DEV)].contiguous()


def _named(edges, name):
    """The edges with every node renamed."""
    return name.int()[edges.long()].contiguous()


def _lfr(n, m, gamma, mu, seed):
    """LFR-style stream: Pareto expected degrees, community sizes ~ s^-1.5 on [20, n/100],
    (1 - mu) m edges inside communities, the others anywhere; both ends by weight."""
    g = _gen(SHAPE, 11)
    smin, smax = 20, max(20, n // 100)
    a, b = smin ** -0.5, (smax + 1.0) ** -0.5
    sizes = (a + _rand(g, n // smin + 1) * (b - a)) ** -2.0
    ends = torch.cumsum(sizes.long().clamp_(smin, smax), 0)
    off = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), ends[ends < n], torch.full((1,), n, device=DEV)])
    cum = _cum(_weights(g, n, m, gamma))  # nodes laid out community by community
    zero, top = torch.zeros(m, dtype=torch.int64, device=DEV), cum[-1].expand(m)
    m_in = int(round((1.0 - mu) * m))
    pu = _pick(g, cum, zero, top)
    c = torch.searchsorted(off, pu[:m_in], right=True) - 1
    lo, hi = cum[off[c]], cum[off[c + 1]]
    pv = torch.cat([_pick(g, cum, lo, hi), _pick(g, cum, zero[m_in:], top[m_in:])])
    for _ in range(3):  # redraw ends that met themselves (the few that are left are loops)
        bad = torch.nonzero(pu == pv)[:, 0]
        inside = bad[bad < m_in]
        pv[inside] = _pick(g, cum, lo[inside], hi[inside])
        outside = bad[bad >= m_in]
        pv[outside] = _pick(g, cum, zero[outside], top[outside])
    return _named(_stream(g, pu, pv), torch.randperm(n, generator=_gen(seed, 10), device=DEV))


def _planted(n, blocks, p_in, p_out, seed):
    g = _gen(SHAPE, 12)
    blk = torch.clamp(torch.arange(n, device=DEV) // max(1, n // blocks), max=blocks - 1)
    p = torch.where(blk[:, None] == blk[None, :], p_in, p_out)
    iu = torch.nonzero(torch.triu(_rand(g, n, n) < p, diagonal=1))
    return _named(_stream(g, iu[:, 0], iu[:, 1]), torch.randperm(n, generator=_gen(seed, 10), device=DEV))


def _batch(c, seed):
    """Uneven planted graphs: log-normal node counts, 5 edges per node, 92% of them inside
    blocks of about 250 nodes; concatenated edges with local ids and the two offset lists."""
    rng = np.random.default_rng([SHAPE, 13])
    ns = np.clip(np.round(np.exp(rng.normal(math.log(c["median"]), c["sigma"], c["graphs"]))), 100, c["nmax"])
    ns = torch.from_numpy(ns.astype(np.int64)).to(DEV)
    noff, eoff = _cum(ns), _cum(5 * ns)
    g = _gen(SHAPE, 14)
    G, m = c["graphs"], int(eoff[-1])
    gid = torch.repeat_interleave(torch.arange(G, device=DEV), 5 * ns)
    n_of = ns[gid]
    blocks = torch.clamp(torch.round(ns / 250.0), 2, 80).long()[gid]
    b = (_rand(g, m) * blocks).long()
    lo, hi = b * n_of // blocks, (b + 1) * n_of // blocks
    size = hi - lo
    at = (_rand(g, m) * size).long()
    u = lo + at
    v_in = lo + (at + 1 + (_rand(g, m) * (size - 1)).long()) % size
    v_out = (hi + (_rand(g, m) * (n_of - size)).long()) % n_of
    v = torch.where(_rand(g, m) < 0.92, v_in, v_out)
    # per graph, nodes renamed and edges reordered at random
    node_g = torch.repeat_interleave(torch.arange(G, device=DEV), ns)
    name = torch.argsort(node_g.double() + _rand(_gen(seed, 10), node_g.shape[0]), stable=True) - noff[node_g]
    u, v = name[noff[gid] + u], name[noff[gid] + v]
    swap = _rand(g, m) < 0.5
    e = torch.stack([torch.where(swap, v, u), torch.where(swap, u, v)], 1).int()
    e = e[torch.argsort(gid.double() + _rand(g, m), stable=True)].contiguous()
    order = torch.argsort(ns, descending=True, stable=True).int()
    return e, noff, eoff, order, int(noff[-1])


def _superedges(K, E, gamma, seed):
    """E distinct pairs of K supernodes, ends by power-law weight, sorted as supergraph()
    returns them."""
    g = _gen(seed, 15)
    E = min(E, K * (K - 1) // 4)
    cum = _cum(_weights(g, K, E, gamma))
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    while keys.shape[0] < E:
        n = E - keys.shape[0] + E // 4 + 16
        zero, top = torch.zeros(n, dtype=torch.int64, device=DEV), cum[-1].expand(n)
        a, b = _pick(g, cum, zero, top), _pick(g, cum, zero, top)
        keys = torch.unique(torch.cat([keys, (torch.minimum(a, b) * K + torch.maximum(a, b))[a != b]]))
    keep = torch.randperm(keys.shape[0], generator=g, device=DEV)[:E]
    keys = torch.sort(keys[keep])[0]
    return torch.stack([keys // K, keys % K], 1).int().contiguous()


def _coefs(rows, seed):
    """Random draws of the two sketches' hash families, uint64 (rows, 3) each."""
    rng = np.random.default_rng([int(seed), 16])
    return tuple(rng.integers(0, np.iinfo(np.uint64).max, size=(rows, 3), dtype=np.uint64, endpoint=True)
                 for _ in range(2))


def _workload(c):
    """The workload description that the library's entry points take."""
    return dict(threshold=c["threshold"], passes=c["passes"], growth=2, chunk=c["chunk"], tie=c.get("tie", 0),
                rule=c.get("rule", 0), rows=c.get("rows", 1), cols=c.get("cols", 1), fa2_iters=c.get("iters", 0),
                exact=True, theta=1.2, kr=1.0, kg=1.0, tau=1.0, ks=0.1, ksmax=10.0)


def _positions(g, K, span):
    return ((_rand(g, K, 2) * 2.0 - 1.0) * span).float()


def _layout_inputs(c, seed):
    """Superedges with the optional weights, masses and running state of a layout."""
    K = c["supernodes"]
    s = dict(se=_superedges(K, c["superedges"], c["gamma"], seed))
    g = _gen(seed, 17)
    E = s["se"].shape[0]
    s["w"] = (1.0 - torch.log2(_rand(g, E).clamp_(min=1e-9)).ceil()).float() if c.get("weighted", True) else None
    if c.get("masses"):
        s["mass"] = (1.0 + torch.bincount(s["se"].flatten().long(), minlength=K) + 9.0 * _rand(g, K)).float()
    else:
        s["mass"] = None
    s["pos"] = _positions(g, K, 50.0 if c["do"] == "grad" or not c["fresh"] else 1.0)
    if c["do"] == "layout":
        s["fprev"] = torch.zeros_like(s["pos"]) if c["fresh"] else _positions(g, K, 20.0)
        s["speed"] = torch.full((1,), 1.0 if c["fresh"] else 0.4, device=DEV)
    return s


def prepare(case, seed):
    c = dict(case)
    s = dict(c=c)
    if c["do"] in ("pipeline", "batched", "supergraph"):
        s["c1"], s["c2"] = _coefs(c["rows"], seed)
    if c["do"] == "pipeline":
        s["edges"] = _planted(c["n"], c["blocks"], c["p_in"], c["p_out"], seed)
        s["pos"] = _positions(_gen(seed, 18), c["n"], 1.0)
        s["wl"] = _workload(c)
    elif c["do"] == "batched":
        s["edges"], s["noff"], s["eoff"], s["order"], s["n"] = _batch(c, seed)
        s["pos0"] = _positions(_gen(seed, 18), s["n"], 1.0)
        s["pos"], s["fprev"] = s["pos0"].clone(), torch.zeros_like(s["pos0"])
        s["speed"] = torch.ones(c["graphs"], device=DEV)
        s["rows"] = {}
        for count, off in (("K", s["noff"]), ("E", s["eoff"])):
            gid = torch.repeat_interleave(torch.arange(c["graphs"], device=DEV), off[1:] - off[:-1])
            s["rows"][count] = gid, torch.arange(gid.shape[0], device=DEV) - off[gid]
        s["ws"] = bgv.batched_workspace(c["graphs"], s["n"], s["edges"].shape[0], s["edges"].device)
        s["wl"] = _workload(c)
    elif c["do"] in ("community", "supergraph"):
        s["edges"] = _lfr(c["n"], c["m"], c["gamma"], c["mu"], seed)
        s["wl"] = _workload(c)
        if c["do"] == "supergraph":
            s["labels"], s["degree"], _ = bgv.community(s["edges"], c["n"], c["threshold"], c["passes"], 2, c["chunk"],
                                                        check=False)
            s["ws"] = bgv.api.supergraph_workspace(s["edges"], c["n"], s["wl"])
        else:
            s["ws"] = bgv.api.community_workspace(s["edges"], c["n"], s["wl"])
    else:
        s.update(_layout_inputs(c, seed))
    return s


def run(s):
    c = s["c"]
    if c["do"] == "pipeline":
        o = bgv.pipeline(s["edges"], c["n"], s["wl"], s["c1"], s["c2"], s["pos"])
        sg = o["sg"]
        return dict(labels=o["labels"], degree=o["degree"], super_label=sg["super_label"], super_size=sg["super_size"],
                    node_super=sg["node_super"], superedges=sg["superedges"], se_weight=sg["se_weight"], M1=sg["M1"],
                    M2=sg["M2"], pos=o["pos"], fprev=o["fprev"], speed=o["speed"])
    if c["do"] == "batched":
        s["pos"].copy_(s["pos0"])
        s["fprev"].zero_()
        s["speed"].fill_(1.0)
        o = bgv.batched(s["edges"], s["noff"], s["eoff"], s["n"], s["wl"], s["c1"], s["c2"], s["pos"],
                        order=s["order"], fprev=s["fprev"], speed=s["speed"], wg_threads=c["wg_threads"],
                        big_k=c["big_k"], ws=s["ws"])
        # the supernodes' and superedges' buffers hold each graph's first K or E entries
        for count, keys in (("K", ("super_label", "super_size")), ("E", ("superedges", "se_weight"))):
            gid, at = s["rows"][count]
            used = at < o[count][gid]
            o.update({k: torch.where(used if o[k].dim() == 1 else used[:, None], o[k], 0) for k in keys})
        return o
    if c["do"] == "community":
        labels, degree, volume = bgv.community(s["edges"], c["n"], c["threshold"], c["passes"], 2, c["chunk"],
                                               volume=True, ws=s["ws"], method=c["method"], tie=c["tie"],
                                               rule=c["rule"], check=c["check"])
        return dict(labels=labels, degree=degree, volume=volume)
    if c["do"] == "supergraph":
        o = bgv.supergraph(s["edges"], s["labels"], s["degree"], c["rows"], c["cols"], s["c1"], s["c2"], ws=s["ws"],
                           exact_counts=c["exact_counts"], check=c["check"])
        return {k: v for k, v in o.items() if v is not None}
    if c["do"] == "layout":
        pos, fprev, speed = bgv.fa2_layout(s["se"], s["pos"].clone(), c["iters"], exact=c["exact"], attr_w=s["w"],
                                           mass=s["mass"], fprev=s["fprev"].clone(), speed=s["speed"].clone())
        return dict(pos=pos, fprev=fprev, speed=speed)
    x = s["pos"].detach().requires_grad_(True)
    energy = bgv.FA2Energy.apply(x, s["se"], 1.0, 1.0, s["w"], s["mass"])
    energy.backward()
    return dict(energy=energy.detach(), grad=x.grad)


def work(case):
    """Each input read once, each output written once; 10 operations per pair of bodies
    (20 where a pair is walked from both ends, 50 such pairs per body under Barnes-Hut)
    and 6 per directed superedge and iteration."""
    c = dict(case)
    if c["do"] == "pipeline":
        m, cells = c["n"] * 5.5, c["rows"] * c["cols"]
        K = c["n"] / 12.0
        return dict(bytes=8 * m + 28 * c["n"] + 8 * cells, flops=c["iters"] * (20.0 * K * K + 12 * 16 * K))
    if c["do"] == "batched":
        n = c["graphs"] * c["median"] * math.exp(c["sigma"] ** 2 / 2)
        k2 = c["graphs"] * (c["median"] / 12.0) ** 2 * math.exp(2 * c["sigma"] ** 2)
        return dict(bytes=52 * n + 8 * n * 5, flops=c["iters"] * 20.0 * k2)
    if c["do"] == "community":
        return dict(bytes=8 * c["m"] + 16 * c["n"], flops=0)
    if c["do"] == "supergraph":
        return dict(bytes=8 * c["m"] + 12 * c["n"] + 8 * c["rows"] * c["cols"] + 12 * c["mu"] * c["m"], flops=0)
    K, E = c["supernodes"], c["superedges"]
    if c["do"] == "layout":
        pairs = 20.0 * K * K if c["exact"] else 20.0 * 50.0 * K
        return dict(bytes=(12 if c["weighted"] else 8) * E + (36 if c["masses"] else 32) * K,
                    flops=c["iters"] * (pairs + 12.0 * E))
    return dict(bytes=12 * E + 16 * K, flops=20.0 * K * K + 10.0 * K * K / 2 + 18.0 * E)


# ----------------------------------------------------- the same in 64 bits -------
def _mass64(s, K):
    if s["mass"] is not None:
        return s["mass"].double()
    return 1.0 + torch.bincount(s["se"].flatten().long(), minlength=K).double()


def _forces64(x, s, m):
    """ForceAtlas2 force (kr = kg = 1) and energy of positions x in float64."""
    K = x.shape[0]
    F = torch.empty_like(x)
    energy = torch.zeros((), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 26) // K)
    for a in range(0, K, step):
        d = x[a:a + step, None, :] - x[None, :, :]
        d2 = (d * d).sum(2)
        near = d2 == 0
        F[a:a + step] = m[a:a + step, None] * (torch.where(near, 0.0, m[None, :] / d2)[:, :, None] * d).sum(1)
        logs = torch.where(near, 0.0, torch.log(torch.where(near, 1.0, d2)))
        energy -= 0.25 * (m[a:a + step, None] * m[None, :] * logs).sum()  # half of ln d^2, each pair twice
    i, j = s["se"][:, 0].long(), s["se"][:, 1].long()
    w = s["w"].double() if s["w"] is not None else torch.ones(i.shape[0], dtype=torch.float64, device=DEV)
    d = x[j] - x[i]
    F.index_add_(0, i, w[:, None] * d)
    F.index_add_(0, j, -w[:, None] * d)
    r = x.norm(dim=1)
    F -= torch.where(r > 0, m / r, 0.0)[:, None] * x
    energy += 0.5 * (w * (d * d).sum(1)).sum() + (m * r).sum()
    return F, energy


def exact(case, seed):
    """Whole numbers have no rounding and Barnes-Hut or long layouts no value in 64 bits (an
    iteration carries a rounding-sized difference of its start on about five times as
    large); short exact layouts and the energy with its gradient do."""
    c = dict(case)
    if c["do"] == "grad":
        s = _layout_inputs(c, seed)
        F, energy = _forces64(s["pos"].double(), s, _mass64(s, c["supernodes"]))
        return dict(energy=energy, grad=-F)
    if c["do"] == "layout" and c["exact"] and c["iters"] <= 2:
        s = _layout_inputs(c, seed)
        x, fp, sp, m = s["pos"].double(), s["fprev"].double(), s["speed"].double(), _mass64(s, c["supernodes"])
        for _ in range(c["iters"]):
            F, _ = _forces64(x, s, m)
            swing, traction = (F - fp).norm(dim=1), 0.5 * (F + fp).norm(dim=1)
            S, T = (m * swing).sum(), (m * traction).sum()
            sp = torch.minimum(T / S, 1.5 * sp) if float(S) > 0 else sp
            local = 0.1 * sp / (1.0 + sp * swing.sqrt())
            local = torch.minimum(local, 10.0 / F.norm(dim=1).clamp(min=1e-300))
            x, fp = x + local[:, None] * F, F
        return dict(pos=x, fprev=fp, speed=sp)
    return None

"""Workloads that stand for what programs have this library do, for timing one build against another.

``listed()`` names them, ``draw(rng)`` gives further ones of the same ranges, ``prepare(case, seed)``
makes the inputs a program has in hand before the call (device CSR arrays, a packed batch, host
CSR jobs with an open server), ``run(state)`` makes ONE pass through the package's public entry
points and returns all of its outputs, ``work(case)`` says what a pass cannot do without, and
``exact(case, seed)`` computes the same outputs in plain 64-bit torch where that is quick.

Every graph is random in the seed and built on the device with torch: uniform random graphs,
R-MAT graphs (.57, .19, .19, .05; permuted ids) and road-like nearest-neighbour graphs, in the
canonical symmetric CSR (rows sorted, no self-loops, no duplicates) that the entry points take.
Sizes and degrees depend on the case alone.
"""
import math
import random

import numpy as np
import torch

import paper_1912_01478_amd as ipgc

DEV = "cuda"


def listed():
    return [
        # The smallest calls: a graph of a thousand nodes, as an inner step of a larger program
        # (register or schedule conflicts, one mesh patch).  Launches and waits are all there is.
        {"name": "color_er_n1000_d8", "kind": "color", "graph": "er", "n": 1000, "d": 8},
        # The repository's smallest benchmark workload: a uniform random graph of 10^4 nodes.
        {"name": "color_er_n10000_d8", "kind": "color", "graph": "er", "n": 10000, "d": 8},
        # A hub-heavy graph of medium size through the entry point for loops that may not allocate:
        # about a hundred rounds, most of them small.
        {"name": "noalloc_rmat_n65536_ef16", "kind": "noalloc", "graph": "rmat", "n": 65536, "d": 16},
        # An ordinary uniform graph at an odd size, with the data-driven schedule (the paper's
        # "Plain" version): light rows and a few wide ones.
        {"name": "color_er_n1000003_d16_data", "kind": "color", "graph": "er", "n": 1000003, "d": 16, "mode": "data"},
        # A hub-heavy graph from an untrusted source: full validation (simple, symmetric) before coloring.
        {"name": "color_rmat_n300007_ef8_full", "kind": "color", "graph": "rmat", "n": 300007, "d": 8, "validate": "full"},
        # The benchmark's largest power-law graph: R-MAT scale 22, edge factor 16.
        {"name": "color_rmat_n4194304_ef16", "kind": "color", "graph": "rmat", "n": 4194304, "d": 16},
        # The benchmark's road-like graph: 24 million nodes of average degree 2.4.
        {"name": "color_road_n24000000", "kind": "color", "graph": "road", "n": 24000000, "d": 2},
        # Many small graphs in one call (one per patch, per basic block, per subdomain).
        {"name": "batch_1024_n1000_10000", "kind": "batch", "graphs": 1024, "lo": 1000, "hi": 10000},
        # The benchmark's batch mix (uniform and R-MAT alternating, sizes log-uniform), fewer graphs.
        {"name": "batch_160_n1000_1000000", "kind": "batch", "graphs": 160, "lo": 1000, "hi": 1000000},
        # The same schedule on another worklist algorithm: breadth-first search over a power-law
        # graph from its widest node, and over a sparse uniform graph with many levels.
        {"name": "bfs_rmat_n4194304_ef16", "kind": "bfs", "graph": "rmat", "n": 4194304, "d": 16},
        {"name": "bfs_er_n100003_d4", "kind": "bfs", "graph": "er", "n": 100003, "d": 4},
        # The job server, saturated: host CSR jobs of the serving mix (a tenth of them R-MAT of
        # 2^20 nodes) submitted at once and stepped until every one is done.
        {"name": "serve_20_n1000_1000000", "kind": "serve", "graphs": 20, "lo": 1000, "hi": 1000000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["color", "color", "color", "color", "noalloc", "batch", "batch", "bfs", "bfs", "serve"])
    if kind in ("batch", "serve"):
        hi = _log(rng, 3000, 1000000)
        if kind == "serve":
            return {"kind": "serve", "graphs": rng.randint(4, 20), "lo": 1000, "hi": hi}
        # about the node total of the listed batches at most
        most = max(4, min(1024, 23000000 // (hi // 6)))
        return {"kind": "batch", "graphs": _log(rng, 4, most), "lo": 1000, "hi": hi}
    graph = rng.choice(["er", "rmat", "road"] if kind == "color" else ["er", "rmat"])
    if graph == "road":
        return {"kind": kind, "graph": "road", "n": _log(rng, 1000, 24000000), "d": 2}
    d = rng.randint(4, 32) if graph == "er" else rng.randint(8, 16)
    most = 1000000 if kind == "noalloc" else 4194304 if graph == "rmat" else 4000000
    if kind == "noalloc":
        d = min(d, 15)  # its scratch holds 10^6 nodes with 32 entries each
    case = {"kind": kind, "graph": graph, "n": _log(rng, 1000, most), "d": d}
    if kind == "color":
        case["mode"] = rng.choice(["hybrid", "hybrid", "data", "topology"])
        if case["n"] <= 1000000 and rng.random() < 0.2:
            case["validate"] = "full"
    return case


# ---------------------------------------------------------------- inputs

def _csr(n, src, dst):
    """Canonical CSR of the undirected pairs (self-loops and duplicates dropped), on the device."""
    keep = src != dst
    src, dst = src[keep], dst[keep]
    key = torch.cat([(src << 32) | dst, (dst << 32) | src])
    del src, dst, keep
    key = torch.sort(key).values
    if key.numel():
        first = torch.ones(key.numel(), dtype=torch.bool, device=key.device)
        torch.ne(key[1:], key[:-1], out=first[1:])
        key = key[first]
        del first
    colidx = (key & 0xFFFFFFFF).to(torch.int32)
    deg = torch.bincount(key >> 32, minlength=n)
    del key
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=deg.device)
    torch.cumsum(deg, 0, out=rowptr[1:])
    return rowptr, colidx


def _rmat_unit(count, levels, gen):
    """`count` R-MAT endpoints pairs as fractions of the id range, `levels` quadrant choices each."""
    x = torch.zeros(count, dtype=torch.float64, device=DEV)
    y = torch.zeros(count, dtype=torch.float64, device=DEV)
    for k in range(levels):
        u = torch.rand(count, generator=gen, device=DEV)
        half = 0.5 ** (k + 1)
        x += (u >= 0.76).to(torch.float64) * half
        y += (((u >= 0.57) & (u < 0.76)) | (u >= 0.95)).to(torch.float64) * half
    return x, y


def _graph(graph, n, d, gen):
    """(rowptr int64, colidx int32) of one random graph."""
    if graph == "road":
        return _road(n, gen)
    if graph == "er":
        count = n * d // 2
        src = torch.randint(0, n, (count,), generator=gen, device=DEV)
        dst = torch.randint(0, n, (count,), generator=gen, device=DEV)
        return _csr(n, src, dst)
    x, y = _rmat_unit(n * d, max(1, math.ceil(math.log2(n))), gen)
    perm = torch.randperm(n, generator=gen, device=DEV)
    return _csr(n, perm[(x * n).long().clamp_(max=n - 1)], perm[(y * n).long().clamp_(max=n - 1)])


def _road(n, gen):
    """Road-like graph: n uniform points, each linked to its nearest (and, 4 times in 5, its second
    nearest) neighbour; ids by sqrt(n) horizontal strips, x-sorted inside each strip."""
    xy = torch.rand(2, n, generator=gen, device=DEV, dtype=torch.float64)
    strips = max(1, int(math.sqrt(n)))
    order = torch.argsort((xy[1] * strips).floor() + xy[0])
    xy = xy[:, order].contiguous()
    del order
    two = torch.rand(n, generator=gen, device=DEV) < 0.8
    g = max(1, int(math.sqrt(n / 2)))
    cx, cy = (xy[0] * g).long().clamp_(max=g - 1), (xy[1] * g).long().clamp_(max=g - 1)
    cell = cy * g + cx
    order = torch.argsort(cell)
    start = torch.zeros(g * g + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(cell, minlength=g * g), 0, out=start[1:])
    del cell
    sx, sy = xy[0][order].float(), xy[1][order].float()
    order = order.to(torch.int32)
    px, py = xy[0].float(), xy[1].float()
    me = torch.arange(n, dtype=torch.int32, device=DEV)
    b1, b2 = (torch.full((n,), 9.0, device=DEV) for _ in range(2))
    i1, i2 = (torch.full((n,), -1, dtype=torch.int32, device=DEV) for _ in range(2))
    for row in (-1, 0, 1):
        r = cy + row
        ok = (r >= 0) & (r < g)
        r = r.clamp(0, g - 1) * g
        a, e = start[r + (cx - 1).clamp(min=0)], start[r + (cx + 1).clamp(max=g - 1) + 1]
        e = torch.where(ok, e, a)
        del r, ok
        for k in range(18):
            at = a + k
            has = at < e
            at.clamp_(max=n - 1)
            u = order[at]
            dist = (sx[at] - px).square_() + (sy[at] - py).square_()
            dist = torch.where(has & (u != me), dist, 9.0)
            near1, near2 = dist < b1, dist < b2
            i2 = torch.where(near1, i1, torch.where(near2, u, i2))
            b2 = torch.where(near1, b1, torch.where(near2, dist, b2))
            i1 = torch.where(near1, u, i1)
            b1 = torch.where(near1, dist, b1)
    v = me.long()
    has1, has2 = i1 >= 0, two & (i2 >= 0)
    return _csr(n, torch.cat([v[has1], v[has2]]), torch.cat([i1[has1], i2[has2]]).long())


def _sizes(case):
    """The graphs of a batch or job stream, by the case alone: (n, kind, d) with sizes spread evenly
    over the logarithm of [lo, hi], uniform and R-MAT alternating; a server's stream has an R-MAT
    graph of 16 entries per node and 2^20 nodes (at most `hi` times 1.05) in every ten."""
    rng = random.Random(12345)
    count, lo, hi = case["graphs"], case["lo"], case["hi"]
    ns = [int(round(lo * (hi / lo) ** ((i + 0.5) / count))) for i in range(count)]
    rng.shuffle(ns)
    out = [(n, "er", rng.randint(4, 32)) if i % 2 == 0 else (n, "rmat", rng.randint(8, 16)) for i, n in enumerate(ns)]
    if case["kind"] == "serve":
        for i in range(9, count, 10):
            out[i] = (min(1 << 20, int(hi * 1.05)), "rmat", 16)
    return out


def _pack(sizes, gen):
    """The graphs as one disjoint union: (node_off, edge_off as numpy, rowptr_packed, colidx_packed)."""
    ns = torch.tensor([s[0] for s in sizes], dtype=torch.int64)
    off = torch.zeros(len(sizes) + 1, dtype=torch.int64)
    torch.cumsum(ns, 0, out=off[1:])
    N = int(off[-1])
    src, dst = [], []
    for kind in ("er", "rmat"):
        sel = [i for i, s in enumerate(sizes) if s[1] == kind]
        if not sel:
            continue
        cnt = torch.tensor([sizes[i][0] * sizes[i][2] // (2 if kind == "er" else 1) for i in sel])
        total = int(cnt.sum())
        g = torch.repeat_interleave(torch.tensor(sel), cnt).to(DEV)
        if kind == "er":
            x, y = (torch.rand(total, generator=gen, device=DEV, dtype=torch.float64) for _ in range(2))
        else:
            x, y = _rmat_unit(total, max(1, math.ceil(math.log2(max(sizes[i][0] for i in sel)))), gen)
        ng, og = ns.to(DEV)[g], off.to(DEV)[g]
        src.append(torch.minimum((x * ng).long(), ng - 1) + og)
        dst.append(torch.minimum((y * ng).long(), ng - 1) + og)
        del g, x, y, ng, og
    # a random renaming of the nodes inside each graph
    gi = torch.repeat_interleave(torch.arange(len(sizes)), ns).to(DEV)
    perm = torch.argsort(gi.double() + torch.rand(N, generator=gen, device=DEV, dtype=torch.float64))
    rowptr, colidx = _csr(N, perm[torch.cat(src)], perm[torch.cat(dst)])
    del src, dst, perm
    first = off[:-1].to(DEV)[gi]  # first node of each node's graph
    deg = rowptr[1:] - rowptr[:-1]
    colidx -= torch.repeat_interleave(first.to(torch.int32), deg)
    edge_off = rowptr[off.to(DEV)]
    packed = torch.empty(N + len(sizes), dtype=torch.int32, device=DEV)
    at = torch.arange(N, device=DEV) + gi
    packed[at] = (rowptr[:-1] - edge_off[gi]).to(torch.int32)
    ends = off[1:].to(DEV) + torch.arange(len(sizes), device=DEV)
    packed[ends] = (edge_off[1:] - edge_off[:-1]).to(torch.int32)
    return off.numpy(), edge_off.cpu().numpy(), packed, colidx


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)
    kind = case["kind"]
    if kind in ("color", "noalloc", "bfs"):
        rowptr, colidx = _graph(case["graph"], case["n"], case["d"], gen)
        state = {"kind": kind, "rowptr": rowptr.to(torch.int32), "colidx": colidx, "mode": case.get("mode", "hybrid"),
                 "validate": ipgc.VALIDATE_FULL if case.get("validate") == "full" else ipgc.VALIDATE_DEFAULT}
        if kind == "bfs":
            state["source"] = int(torch.argmax(rowptr[1:] - rowptr[:-1]))
        if kind == "noalloc":
            state["out"] = torch.empty(case["n"], dtype=torch.int32, device=DEV)
        return state
    sizes = _sizes(case)
    node_off, edge_off, rowptr, colidx = _pack(sizes, gen)
    if kind == "batch":
        return {"kind": kind, "rowptr": rowptr, "colidx": colidx, "node_off": node_off, "edge_off": edge_off}
    rp, ci = rowptr.cpu().numpy(), colidx.cpu().numpy()
    jobs = [(rp[node_off[g] + g:node_off[g + 1] + g + 1].copy(), ci[edge_off[g]:edge_off[g + 1]].copy())
            for g in range(len(sizes))]
    server = ipgc.Server(int(node_off[-1]) + 2 * len(sizes), int(edge_off[-1]) + 16, max_jobs=64)
    return {"kind": kind, "jobs": jobs, "server": server}


def run(state):
    kind = state["kind"]
    if kind == "color":
        res = ipgc.color_graph(state["rowptr"], state["colidx"], state["mode"], validate=state["validate"])
        return {"colors": res.colors, "rounds": res.rounds}
    if kind == "noalloc":
        res = ipgc.color_graph_noalloc(state["rowptr"], state["colidx"], out=state["out"])
        return {"colors": res.colors, "rounds": res.rounds}
    if kind == "bfs":
        res = ipgc.bfs(state["rowptr"], state["colidx"], state["source"])
        return {"dist": res.dist, "levels": res.levels}
    if kind == "batch":
        res = ipgc.color_graphs_batched(state["rowptr"], state["colidx"], state["node_off"], state["edge_off"])
        return {"colors": res.colors, "rounds": np.asarray(res.rounds, dtype=np.int32)}
    server = state["server"]
    ids = {server.submit(rp, ci): k for k, (rp, ci) in enumerate(state["jobs"])}
    colors, rounds = [None] * len(ids), [0] * len(ids)
    left = len(ids)
    while left:
        server.step()
        for done in server.poll():
            colors[ids[done.job_id]], rounds[ids[done.job_id]] = done.colors, done.rounds
            left -= 1
    return {"colors": colors, "rounds": np.asarray(rounds, dtype=np.int32)}


# ---------------------------------------------------------------- what a pass cannot do without

def _entries(n, graph, d):
    """About the CSR entries of a graph (duplicates and self-loops gone)."""
    if graph == "road":
        return 2.39 * n
    return float(n * d) if graph == "er" else 2.0 * n * d * (0.95 if n > 100000 else 0.85)


def work(case):
    """The CSR read once and the result written once, and one comparison per entry."""
    if case["kind"] in ("batch", "serve"):
        sizes = _sizes(case)
    else:
        sizes = [(case["n"], case["graph"], case["d"])]
    n = sum(s[0] for s in sizes)
    m = sum(_entries(s[0], s[1], s[2]) for s in sizes)
    return {"bytes": 4.0 * (n + len(sizes)) + 4.0 * m + 4.0 * n, "flops": m}


# ---------------------------------------------------------------- the same outputs in plain torch

def _color_exact(n, src, dst):
    """Synchronous rounds: every uncolored node takes the smallest color >= 1 that no colored neighbour
    holds; of an edge whose ends took the same color, the higher id is uncolored again.  Returns
    (colors, round in which each node got its color)."""
    col = torch.zeros(n, dtype=torch.int64, device=DEV)
    when = torch.zeros(n, dtype=torch.int64, device=DEV)
    tent = torch.ones(n, dtype=torch.int64, device=DEV)
    r = 0
    base = n + 2
    while True:
        active = col == 0
        if not bool(active.any()):
            return col, when
        r += 1
        keep = active[src]
        src, dst = src[keep], dst[keep]
        if r > 1:
            cd = col[dst]
            has = cd > 0
            pair = torch.unique(src[has] * base + cd[has])
            v, c = pair // base, pair % base
            rank = torch.arange(v.numel(), device=DEV) - torch.searchsorted(v, v)
            gap = torch.full((n,), base, dtype=torch.int64, device=DEV)
            gap.scatter_reduce_(0, v, torch.where(c != rank + 1, rank + 1, base), "amin")
            count = torch.bincount(v, minlength=n)
            tent = torch.where(active, torch.minimum(gap, count + 1), tent)
        clash = (dst < src) & active[dst] & (tent[src] == tent[dst])
        lose = torch.zeros(n, dtype=torch.bool, device=DEV)
        lose[src[clash]] = True
        win = active & ~lose
        col = torch.where(win, tent, col)
        when = torch.where(win, torch.full_like(when, r), when)


def _bfs_exact(n, src, dst, source):
    dist = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    dist[source] = 0
    level = 0
    while True:
        new = dst[(dist[src] == level) & (dist[dst] == -1)]
        if new.numel() == 0:
            return dist, level + 1
        level += 1
        dist[new] = level


def exact(case, seed):
    """The outputs of run() in 64 bits; None for the large cases, whose many rounds take too long this way."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)
    kind = case["kind"]
    if kind in ("color", "noalloc", "bfs"):
        if case["n"] * case["d"] > 4000000 and not (kind == "bfs" or case["graph"] == "road" or case["graph"] == "er"):
            return None
        rowptr, colidx = _graph(case["graph"], case["n"], case["d"], gen)
        n, deg = case["n"], rowptr[1:] - rowptr[:-1]
        src = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
        if kind == "bfs":
            dist, levels = _bfs_exact(n, src, colidx.long(), int(torch.argmax(deg)))
            return {"dist": dist.to(torch.int32), "levels": levels}
        col, when = _color_exact(n, src, colidx.long())
        return {"colors": col.to(torch.int32), "rounds": int(when.max())}
    sizes = _sizes(case)
    if sum(s[0] for s in sizes) > 8000000 or kind == "serve":
        return None
    node_off, edge_off, rowptr, colidx = _pack(sizes, gen)
    off = torch.from_numpy(node_off).to(DEV)
    N, G = int(node_off[-1]), len(sizes)
    gi = torch.repeat_interleave(torch.arange(G, device=DEV), off[1:] - off[:-1])
    rp = rowptr.long()
    at = torch.arange(N, device=DEV) + gi
    deg = rp[at + 1] - rp[at]
    src = torch.repeat_interleave(torch.arange(N, device=DEV), deg)
    dst = colidx.long() + off[gi[src]]
    col, when = _color_exact(N, src, dst)
    rounds = torch.zeros(G, dtype=torch.int64, device=DEV).scatter_reduce_(0, gi, when, "amax")
    return {"colors": col.to(torch.int32), "rounds": rounds.to(torch.int32).cpu().numpy()}

"""The last rounds on one workgroup (worklists of at most 1024 nodes): against the oracle at its edges --
worklists of 1023 to 1025 nodes and their matrix words, windows of 128 colors used up and refilled from
the byte maps, colors committed beyond a window, each way that color sets are kept, batches."""
import numpy as np
import pytest

import graphgen as gg
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def cliques(count, k, extra=0):
    """`count` disjoint K_k with interleaved ids (node j of clique i is j * count + i), then `extra` nodes alone."""
    i, j = np.triu_indices(k, 1)
    src = np.concatenate([i * count + c for c in range(count)])
    dst = np.concatenate([j * count + c for c in range(count)])
    return gg.from_pairs(count * k + extra, src, dst, "%dxK%d+%d" % (count, k, extra))


def late_low_colors(k):
    """K_k whose nodes each have their own leaf, with an id below every clique node: leaves commit color 1
    first, and every node's window starts one color later than the clique's order alone would give."""
    i, j = np.triu_indices(k, 1)
    return gg.from_pairs(2 * k, np.concatenate([i + k, np.arange(k)]), np.concatenate([j + k, np.arange(k) + k]), "K%d+leaves" % k)


GRAPHS = [cliques(2, 512), cliques(2, 512, 1), cliques(5, 205), cliques(341, 3, 2), cliques(16, 130), gg.complete(1100),
          gg.crown(600), late_low_colors(700), gg.complete_bipartite(900, 1100), gg.cycle(1025), gg.path(2049),
          gg.rmat(12, 16, gg.key(77, 0)), gg.erdos_renyi(1500, 90.0, gg.key(77, 1)), gg.erdos_renyi(30011, 5.0, gg.key(77, 2))]
OPTIONS = [dict(), dict(mode="data", light="push"), dict(light="pull", hub_min_degree=40),
           dict(light_max_degree=2, hub_min_degree=64, workgroups=9)]


@pytest.mark.parametrize("kw", OPTIONS, ids=lambda k: "-".join("%s=%s" % x for x in k.items()) or "default")
@pytest.mark.parametrize("g", GRAPHS, ids=lambda g: g.name)
def test_last_rounds_match_the_oracle(g, kw):
    import paper_1912_01478_amd as ip
    ref = oracle.color_graph(g.rowptr, g.colidx)
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    print("[gpu] core %s n=%d m=%d %s" % (g.name, g.n, g.m, kw), flush=True)
    for trace in (True, False):
        res = ip.color_graph(rp, ci, trace=trace, **kw)
        assert res.rounds == ref.rounds
        assert np.array_equal(res.colors.cpu().numpy(), ref.colors)
        if trace:
            assert list(res.wl_sizes) == list(ref.wl_sizes)
            assert list(res.wl_degrees) == list(ref.wl_degree_sums)


@pytest.mark.parametrize("per_graph", [False, True])
def test_last_rounds_of_a_batch(per_graph):
    """Graphs that end in different rounds, their last nodes in one core; every graph's own rounds and colors."""
    import paper_1912_01478_amd as ip
    graphs = GRAPHS[:5] + [gg.complete(300), gg.rmat(11, 16, gg.key(78, 0)), gg.empty(5), gg.erdos_renyi(4000, 9.0, gg.key(78, 1))]
    refs = [oracle.color_graph(g.rowptr, g.colidx) for g in graphs]
    node_off, edge_off, rp, ci = ip.pack_graphs([(g.rowptr, g.colidx) for g in graphs])
    rp, ci = torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda()
    print("[gpu] core batch of %d graphs, per_graph=%s" % (len(graphs), per_graph), flush=True)
    for trace in (True, False):
        res = ip.color_graphs_batched(rp, ci, node_off, edge_off, per_graph=per_graph, trace=trace)
        for k, (g, ref) in enumerate(zip(graphs, refs)):
            assert np.array_equal(res.graph(k).cpu().numpy(), ref.colors), g.name
            assert res.rounds[k] == ref.rounds, g.name
        if trace:
            sizes = np.zeros(len(res.wl_sizes), dtype=np.int64)
            for ref in refs:
                sizes[:len(ref.wl_sizes)] += np.asarray(ref.wl_sizes)
            assert list(res.wl_sizes) == sizes.tolist()


def stars_on_a_path(stars, n):
    """A path of n nodes with `stars` centers of degree 33 to 35 spread over it: wide nodes, the others of class L."""
    gap = n // stars
    c = np.repeat(np.arange(stars) * gap + gap // 2, 33)
    leaf = (c + 2 + np.tile(np.arange(33), stars) * 7) % n
    return gg.from_pairs(n, np.concatenate([np.arange(n - 1), c]), np.concatenate([np.arange(1, n), leaf]), "%d stars" % stars)


# Pushes of class L by tags or by masks: the rule's line is a 64th of the nodes being wide.
@pytest.mark.parametrize("g", [stars_on_a_path(200, 12800), stars_on_a_path(201, 12800), stars_on_a_path(1, 20011),
                               gg.erdos_renyi(20011, 20.0, gg.key(75, 0)), gg.erdos_renyi(20011, 26.0, gg.key(75, 1))],
                         ids=lambda g: "%s_%d" % (g.name, g.m))
def test_light_pushes(g):
    import paper_1912_01478_amd as ip
    ref = oracle.color_graph(g.rowptr, g.colidx)
    print("[gpu] light pushes %s n=%d m=%d" % (g.name, g.n, g.m), flush=True)
    for rowptr, colidx in ((g.rowptr, g.colidx), gg.shuffle_rows(g, 3)):
        rp, ci = torch.from_numpy(np.ascontiguousarray(rowptr)).cuda(), torch.from_numpy(np.ascontiguousarray(colidx)).cuda()
        for kw in (dict(), dict(mode="data"), dict(mode="topology"), dict(mode="rebuild"), dict(light="push", workgroups=70)):
            res = ip.color_graph(rp, ci, **kw)
            assert res.rounds == ref.rounds and np.array_equal(res.colors.cpu().numpy(), ref.colors), kw
        out = torch.empty(g.n, dtype=torch.int32, device="cuda")
        res = ip.color_graph_noalloc(rp, ci, out=out)
        assert res.rounds == ref.rounds and np.array_equal(out.cpu().numpy(), ref.colors)


@pytest.mark.parametrize("graphs", [63, 64, 80])
def test_unions_of_many_graphs(graphs):
    """From 64 graphs on, with a grid of 64 workgroups or more in eighths, each part of a union stays on one XCD."""
    import paper_1912_01478_amd as ip
    gs = [gg.erdos_renyi(1200 + 37 * k, 6.0 + k % 9, gg.key(76, k)) if k % 3 else gg.rmat(10, 10, gg.key(76, k)) for k in range(graphs)]
    gs[5], gs[graphs - 1] = gg.empty(0), gg.star(3000, 0)
    refs = [oracle.color_graph(g.rowptr, g.colidx) for g in gs]
    node_off, edge_off, rp, ci = ip.pack_graphs([(g.rowptr, g.colidx) for g in gs])
    rp, ci = torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda()
    print("[gpu] union of %d graphs" % graphs, flush=True)
    for kw in (dict(workgroups=64), dict(workgroups=72, mode="data"), dict(workgroups=64, mode="topology"), dict(workgroups=64, mode="rebuild"),
               dict(workgroups=64, trace=True), dict(workgroups=68), dict(workgroups=64, per_graph=True), dict(workgroups=64, light="push")):
        res = ip.color_graphs_batched(rp, ci, node_off, edge_off, **kw)
        for k, (g, ref) in enumerate(zip(gs, refs)):
            assert np.array_equal(res.graph(k).cpu().numpy(), ref.colors), (g.name, kw)
            assert res.rounds[k] == ref.rounds, (g.name, kw)


# The W/M cut-off chosen by size, full validation's entry search, and long rows left to the wavefront: rows at and past
# 512, 2048 and 64 entries, empty rows between them, sorted or not.
@pytest.mark.parametrize("g", [gg.star(2048, 1), gg.star(2049, 1), gg.star(13000, 6000), gg.rmat(15, 24, gg.key(74, 0), n=20011),
                               gg.complete_bipartite(200, 10500), gg.empty(20000)], ids=lambda g: g.name)
def test_long_rows_with_full_validation(g):
    import paper_1912_01478_amd as ip
    ref = oracle.color_graph(g.rowptr, g.colidx)
    print("[gpu] long rows %s n=%d m=%d" % (g.name, g.n, g.m), flush=True)
    for rowptr, colidx in ((g.rowptr, g.colidx), gg.shuffle_rows(g, 3)):
        rp, ci = torch.from_numpy(np.ascontiguousarray(rowptr)).cuda(), torch.from_numpy(np.ascontiguousarray(colidx)).cuda()
        for kw in (dict(), dict(validate=ip.VALIDATE_FULL), dict(validate=ip.VALIDATE_FULL, hub_min_degree=512)):
            res = ip.color_graph(rp, ci, **kw)
            assert res.rounds == ref.rounds and np.array_equal(res.colors.cpu().numpy(), ref.colors), kw
    if g.m:  # one entry changed: no longer symmetric, or no longer in range
        bad = ci.clone()
        v = int(torch.argmax(rp[1:] - rp[:-1]))
        bad[int(rp[v]) + 1] = bad[int(rp[v])]
        with pytest.raises(ip.IpgcError) as e:
            ip.color_graph(rp, bad, validate=ip.VALIDATE_FULL)
        assert e.value.code == ip.EBADCSR


def one_way(n, d, kind, seed):
    """CSR whose rows, of at most `d` ids each and sorted, need not be named back."""
    rng = np.random.default_rng(seed)
    rows = []
    for v in range(n):
        lo, hi = {"any": (0, n), "below": (0, v), "above": (v + 1, n), "band": (max(0, v - d), v)}[kind]
        ids = np.arange(lo, hi) if kind == "band" else np.unique(rng.integers(lo, hi, d)) if hi > lo else np.arange(0)
        rows.append(ids[ids != v])
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum([len(r) for r in rows])
    return rp, np.concatenate(rows).astype(np.int32)


# Graphs of class L alone read their own rows in every round, the last ones too: the oracle's colors, named back or not.
@pytest.mark.parametrize("kind, n, d", [("any", 10241, 3), ("any", 20011, 8), ("any", 30011, 32), ("below", 15000, 4), ("below", 20011, 30),
                                        ("above", 20011, 20), ("band", 10500, 20)])
def test_one_way_rows_of_light_nodes(kind, n, d):
    import paper_1912_01478_amd as ip
    rowptr, colidx = one_way(n, d, kind, n + d)
    ref = oracle.color_graph(rowptr, colidx)
    rng = np.random.default_rng(4)
    shuffled = colidx[np.lexsort((rng.random(colidx.size), np.repeat(np.arange(n), np.diff(rowptr))))]
    print("[gpu] one-way %s n=%d m=%d rounds=%d" % (kind, n, colidx.size, ref.rounds), flush=True)
    rp = torch.from_numpy(rowptr).cuda()
    for ids in (colidx, shuffled):
        ci = torch.from_numpy(ids).cuda()
        for kw in (dict(), dict(mode="data", trace=True), dict(mode="topology"), dict(mode="rebuild"), dict(light="pull", workgroups=70)):
            res = ip.color_graph(rp, ci, **kw)
            assert res.rounds == ref.rounds and np.array_equal(res.colors.cpu().numpy(), ref.colors), kw
        out = torch.empty(n, dtype=torch.int32, device="cuda")
        res = ip.color_graph_noalloc(rp, ci, out=out)
        assert res.rounds == ref.rounds and np.array_equal(out.cpu().numpy(), ref.colors)
    small = gg.erdos_renyi(2000, 6.0, gg.key(73, 0))  # every graph of the union of class L
    node_off, edge_off, prp, pci = ip.pack_graphs([(small.rowptr, small.colidx), (rowptr, colidx)])
    for kw in (dict(), dict(trace=True), dict(per_graph=True)):
        res = ip.color_graphs_batched(torch.from_numpy(prp).cuda(), torch.from_numpy(pci).cuda(), node_off, edge_off, **kw)
        assert res.rounds[1] == ref.rounds and np.array_equal(res.graph(1).cpu().numpy(), ref.colors), kw


@pytest.mark.parametrize("H", [1, 500, 1023, 1024, 1025])
@pytest.mark.parametrize("g", [gg.complete(1100), cliques(5, 205), gg.rmat(14, 12, gg.key(72, 0))], ids=lambda g: g.name)
def test_last_rounds_wait_for_a_callers_threshold(g, H):
    """A caller's H leaves the last rounds to one workgroup from min(H, 1024) nodes on."""
    import paper_1912_01478_amd as ip
    ref = oracle.color_graph(g.rowptr, g.colidx, H)
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    print("[gpu] core %s n=%d m=%d H=%d" % (g.name, g.n, g.m, H), flush=True)
    for mode in ("hybrid", "data"):
        res = ip.color_graph(rp, ci, mode=mode, threshold=H, trace=True)
        assert res.rounds == ref.rounds and np.array_equal(res.colors.cpu().numpy(), ref.colors)
        assert list(res.wl_sizes) == list(ref.wl_sizes) and list(res.wl_degrees) == list(ref.wl_degree_sums)
        assert res.topology == (list(ref.topology) if mode == "hybrid" else [0] * ref.rounds)


@pytest.mark.parametrize("kind, n, d", [("any", 20011, 40), ("below", 12000, 70), ("above", 12000, 70)])
def test_one_way_rows_with_wide_nodes_end(kind, n, d):
    """Nodes above class L learn from pushes, so rows that are not named back get no definite colors; the call ends."""
    import paper_1912_01478_amd as ip
    rowptr, colidx = one_way(n, d, kind, n + d)
    rp, ci = torch.from_numpy(rowptr).cuda(), torch.from_numpy(colidx).cuda()
    print("[gpu] one-way wide %s n=%d m=%d" % (kind, n, colidx.size), flush=True)
    for kw in (dict(), dict(mode="data", workgroups=9), dict(mode="topology")):
        res = ip.color_graph(rp, ci, **kw)
        assert 1 <= res.rounds <= n and int(res.colors.min()) >= 1
    with pytest.raises(ip.IpgcError) as e:
        ip.color_graph(rp, ci, validate=ip.VALIDATE_FULL)
    assert e.value.code == ip.EBADCSR

"""Graphs that one workgroup colors (at most 10 240 nodes, default kernel options): against the oracle at the
edges of its lists, matrix and masks, with unsorted rows, in batches with larger graphs, and its verdicts."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from tests.test_gpu_core import cliques, one_way

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def dev(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in arrays]


def check(g, rowptr=None, colidx=None, noalloc=False, **kw):
    import paper_1912_01478_amd as ip
    ref = oracle.color_graph(g.rowptr, g.colidx)
    rp, ci = dev(g.rowptr if rowptr is None else rowptr, g.colidx if colidx is None else colidx)
    print("[gpu] small %s n=%d m=%d %s" % (g.name, g.n, g.m, kw), flush=True)
    for trace in (False, True):
        if noalloc:
            out = torch.empty(g.n, dtype=torch.int32, device="cuda")
            res = ip.color_graph_noalloc(rp, ci, out=out, trace=trace, **kw)
        else:
            res = ip.color_graph(rp, ci, trace=trace, **kw)
        assert res.rounds == ref.rounds
        bad = np.nonzero(res.colors.cpu().numpy() != ref.colors)[0]
        assert bad.size == 0, "node %d" % bad[0]
        if trace:
            assert list(res.wl_sizes) == list(ref.wl_sizes)
            assert list(res.wl_degrees) == list(ref.wl_degree_sums)


# Node counts at the edges of a wavefront, the core and the lists; row lengths at 32 and 33; more than 64 colors
# while the worklist is still in the lists (14 cliques of 150: 77 rounds before the core takes over).
SIZES = [gg.erdos_renyi(n, d, gg.key(80, n + int(d)), name="er%d_%d" % (n, d))
         for n, d in ((1, 0), (2, 1), (63, 5), (64, 5), (65, 60), (1023, 9), (1024, 30), (1025, 32), (2048, 33), (5003, 20),
                      (10239, 7), (10240, 40), (10241, 7))]
SHAPES = [gg.rmat(10, 16, gg.key(81, 0)), gg.rmat(13, 16, gg.key(81, 1)), gg.rmat(14, 12, gg.key(81, 2), n=10007), cliques(14, 150),
          cliques(3, 341), cliques(60, 33, 100), cliques(60, 34, 100), gg.complete(1024), gg.complete(1025), gg.star(10239, 0),
          gg.star(10239, 10239), gg.star(5000, 2500), gg.path(10240), gg.crown(700), gg.empty(1), gg.empty(10240),
          gg.complete_bipartite(3, 9000), gg.road_knn(9001, gg.key(81, 3))]


@pytest.mark.parametrize("g", SIZES + SHAPES, ids=lambda g: g.name)
def test_small_graphs(g):
    check(g)
    check(g, mode="data", noalloc=True)


@pytest.mark.parametrize("g", SIZES[5:9] + SHAPES[:6], ids=lambda g: g.name)
def test_small_graphs_with_unsorted_rows(g):
    rp, ci = gg.shuffle_rows(g, 5)
    check(g, rp, ci)
    check(g, rp, ci, validate=1)


# Row rounds: at and past their nodes (4096), entries (40 960: 10 cliques of 64 have 40 320) and row length (63), from
# the first round and after list rounds.
ROWS = [cliques(10, 64), cliques(11, 64), cliques(9, 65), cliques(60, 64), gg.path(4096), gg.path(4097), gg.cycle(4095),
        gg.erdos_renyi(4096, 4.0, gg.key(85, 0)), gg.erdos_renyi(4097, 4.0, gg.key(85, 1)), gg.erdos_renyi(9000, 20.0, gg.key(85, 2)),
        gg.star(64, 0), gg.star(63, 63), gg.star(62, 30), gg.crown(64), gg.complete(64), gg.complete(65)]


@pytest.mark.parametrize("g", ROWS, ids=lambda g: "%s_%d" % (g.name, g.n))
def test_row_rounds(g):
    check(g)
    check(g, *gg.shuffle_rows(g, 7), noalloc=True)


def test_small_graphs_with_self_loops_and_repeated_entries():
    g = gg.rmat(12, 8, gg.key(82, 0))
    deg = g.degrees()
    rp = np.zeros(g.n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(2 * deg + 1)
    ci = np.concatenate([np.concatenate([np.repeat(g.colidx[g.rowptr[v]:g.rowptr[v + 1]], 2), [v]]) for v in range(g.n)]).astype(np.int32)
    ref = oracle.color_graph(g.rowptr, g.colidx)
    import paper_1912_01478_amd as ip
    res = ip.color_graph(*dev(rp, ci))
    assert res.rounds == ref.rounds and np.array_equal(res.colors.cpu().numpy(), ref.colors)


def test_batches_of_small_and_larger_graphs():
    """Small graphs apart from the union, alone, and none of them; every graph's own colors and rounds."""
    import paper_1912_01478_amd as ip
    large = [gg.rmat(14, 8, gg.key(83, 0)), gg.erdos_renyi(30011, 6.0, gg.key(83, 1)), gg.erdos_renyi(10241, 40.0, gg.key(83, 2))]
    small = SIZES[:9] + SHAPES[:3] + [gg.empty(0), gg.empty(7), cliques(14, 150), gg.complete(300)]
    for graphs in (small, [small[3], large[0], small[9], gg.empty(0), large[1], large[2], small[11]], large, [gg.empty(0)] * 3 + [small[2]]):
        refs = [oracle.color_graph(g.rowptr, g.colidx) for g in graphs]
        node_off, edge_off, rp, ci = ip.pack_graphs([(g.rowptr, g.colidx) for g in graphs])
        rp, ci = dev(rp, ci)
        print("[gpu] small batch of %d graphs" % len(graphs), flush=True)
        for kw in (dict(), dict(mode="data"), dict(mode="topology"), dict(mode="rebuild"), dict(trace=True), dict(workgroups=5)):
            out = torch.full((int(node_off[-1]),), -7, dtype=torch.int32, device="cuda")
            res = ip.color_graphs_batched(rp, ci, node_off, edge_off, out=out, **kw)
            for k, (g, ref) in enumerate(zip(graphs, refs)):
                assert np.array_equal(res.graph(k).cpu().numpy(), ref.colors), (g.name, kw)
                assert res.rounds[k] == ref.rounds, (g.name, kw)


def test_verdicts():
    """The errors of the general path, alone and in a batch; the next call is right."""
    import paper_1912_01478_amd as ip
    g, h = gg.erdos_renyi(3000, 8.0, gg.key(84, 0)), gg.erdos_renyi(20000, 8.0, gg.key(84, 1))
    rp, ci = dev(g.rowptr, g.colidx)
    changes = [("ci", 0, -1), ("ci", g.m - 1, g.n), ("ci", g.m // 2, 2**31 - 1), ("rp", 0, 1), ("rp", g.n, g.m - 1),
               ("rp", g.n // 2, -1), ("rp", g.n // 2, g.m + 5), ("rp", 7, int(g.rowptr[8]) + 1)]
    for which, at, value in changes:
        a, b = rp.clone(), ci.clone()
        (a if which == "rp" else b)[at] = value
        out = torch.empty(g.n, dtype=torch.int32, device="cuda")
        for call in (lambda: ip.color_graph(a, b), lambda: ip.color_graph_noalloc(a, b, out=out)):
            with pytest.raises(ip.IpgcError) as e:
                call()
            assert e.value.code == ip.EBADCSR, (which, at, value)
        for other in ([], [(h.rowptr, h.colidx)]):
            bad = [(a.cpu().numpy(), b.cpu().numpy())]
            node_off, edge_off, prp, pci = ip.pack_graphs([(g.rowptr, g.colidx)] + bad + other)
            with pytest.raises(ip.IpgcError) as e:
                ip.color_graphs_batched(*dev(prp, pci), node_off, edge_off)
            assert e.value.code == ip.EBADCSR, (which, at, value)
    check(g)


# Rows of over 63 entries, so that the lists hand over to the core, or of 33 to 63, to the row rounds: a color per node that its row's nodes of the same
# round do not share is all that such input gets, but the rounds end, the same way every time, and nobody else's colors
# change.
@pytest.mark.parametrize("kind, n, d", [("any", 3000, 100), ("any", 10240, 30), ("below", 3000, 70), ("above", 3000, 80), ("band", 1300, 70),
                                        ("any", 6000, 63), ("below", 3000, 63), ("band", 1500, 63), ("above", 5000, 40)])
def test_long_one_way_rows_end(kind, n, d):
    import paper_1912_01478_amd as ip
    rowptr, colidx = one_way(n, d, kind, n + d)
    if kind == "any" and d == 30:  # one long row
        colidx = np.concatenate([np.arange(1, 101, dtype=np.int32), colidx[rowptr[1]:]])
        rowptr[1:] += 100 - rowptr[1]
    rp, ci = dev(rowptr, colidx)
    print("[gpu] one-way %s n=%d m=%d" % (kind, n, ci.numel()), flush=True)
    first = ip.color_graph(rp, ci)
    col = first.colors.cpu().numpy()
    assert 1 <= first.rounds <= n and col.min() >= 1 and col.max() <= first.rounds
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    for res in (ip.color_graph(rp, ci, mode="data", trace=True), ip.color_graph_noalloc(rp, ci, out=out)):
        assert res.rounds == first.rounds and np.array_equal(res.colors.cpu().numpy(), col)
    others = [SIZES[8], SHAPES[1], gg.erdos_renyi(20011, 9.0, gg.key(86, 0))]
    for k in (2, 3):  # without and with a larger graph
        graphs = [(g.rowptr, g.colidx) for g in others[:k]]
        node_off, edge_off, prp, pci = ip.pack_graphs(graphs[:1] + [(rowptr, colidx)] + graphs[1:])
        res = ip.color_graphs_batched(*dev(prp, pci), node_off, edge_off)
        assert res.rounds[1] == first.rounds and np.array_equal(res.graph(1).cpu().numpy(), col)
        for q, g in zip([0] + list(range(2, k + 1)), others):
            ref = oracle.color_graph(g.rowptr, g.colidx)
            assert res.rounds[q] == ref.rounds and np.array_equal(res.graph(q).cpu().numpy(), ref.colors)


# Rows of at most 32 entries after list rounds, of at most 63 from the first round on in the row rounds or the core: such
# graphs read their own rows, so the oracle's colors hold whether rows are named back or not.
@pytest.mark.parametrize("kind, n, d", [("any", 500, 5), ("any", 4096, 9), ("any", 4097, 4), ("any", 10240, 8), ("any", 10240, 32), ("any", 1000, 63),
                                        ("below", 4000, 4), ("below", 10000, 4), ("below", 4200, 32), ("above", 10000, 20),
                                        ("band", 700, 40), ("band", 4600, 8), ("band", 4200, 32)])
def test_short_one_way_rows_match_the_oracle(kind, n, d):
    import paper_1912_01478_amd as ip
    rowptr, colidx = one_way(n, d, kind, n + d)
    ref = oracle.color_graph(rowptr, colidx)
    rng = np.random.default_rng(4)
    for name, ids in (("sorted", colidx), ("unsorted", colidx[np.lexsort((rng.random(colidx.size), np.repeat(np.arange(n), np.diff(rowptr))))])):
        rp, ci = dev(rowptr, ids)
        print("[gpu] one-way %s n=%d m=%d %s" % (kind, n, ci.numel(), name), flush=True)
        out = torch.empty(n, dtype=torch.int32, device="cuda")
        node_off, edge_off, prp, pci = ip.pack_graphs([(SIZES[3].rowptr, SIZES[3].colidx), (rowptr, ids)])
        batch = ip.color_graphs_batched(*dev(prp, pci), node_off, edge_off)
        for rounds, col in [(r.rounds, r.colors) for r in (ip.color_graph(rp, ci), ip.color_graph(rp, ci, trace=True, mode="data"),
                                                         ip.color_graph_noalloc(rp, ci, out=out))] + [(batch.rounds[1], batch.graph(1))]:
            assert rounds == ref.rounds and np.array_equal(col.cpu().numpy(), ref.colors)


@pytest.mark.parametrize("entries", [1, (3 << 17) + 1])
def test_entries_of_a_graph_without_nodes(entries):
    """A graph of no nodes cannot hold entries, however many; beside small graphs, and beside a larger one."""
    import paper_1912_01478_amd as ip
    g, h = gg.erdos_renyi(3000, 8.0, gg.key(87, 0)), gg.erdos_renyi(20000, 8.0, gg.key(87, 1))
    for others in ([g], [g, h]):
        node_off = np.cumsum([0, 0] + [x.n for x in others])
        edge_off = np.cumsum([0, entries] + [x.m for x in others])
        for only in (0, entries):  # what the graph's one row pointer says
            rp = np.concatenate([[only]] + [x.rowptr for x in others]).astype(np.int32)
            ci = np.concatenate([np.zeros(entries)] + [x.colidx for x in others]).astype(np.int32)
            for kw in (dict(), dict(mode="topology"), dict(trace=True)):
                with pytest.raises(ip.IpgcError) as e:
                    ip.color_graphs_batched(*dev(rp, ci), node_off, edge_off, **kw)
                assert e.value.code == ip.EBADCSR, (entries, only, kw)

"""GPU BFS under the keep-the-worklist hybrid schedule against the BFS oracle: hop distances and
the per-level frontier sizes match exactly for every schedule."""
import numpy as np
import pytest

import graphgen as gg
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MODES = ("topology", "data", "hybrid")


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def run(g, source, mode, **kw):
    import paper_1912_01478_amd as ip
    print("[gpu] bfs %s n=%d m=%d source=%d mode=%s %s" % (g.name, g.n, g.m, source, mode, kw), flush=True)
    res = ip.bfs(torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda(), source, mode, trace=True, **kw)
    torch.cuda.synchronize()
    return res


def check(g, source, mode, **kw):
    ref = oracle.bfs(g.rowptr, g.colidx, source)
    res = run(g, source, mode, **kw)
    dist = res.dist.cpu().numpy()
    bad = np.nonzero(dist != ref.dist)[0]
    assert bad.size == 0, "node %d: gpu %d oracle %d" % (bad[0], dist[bad[0]], ref.dist[bad[0]])
    assert res.levels == ref.levels
    assert list(res.frontier_sizes) == list(ref.frontier_sizes)
    return res


GRAPHS = [gg.path(1), gg.path(50), gg.cycle(51), gg.star(3000, 0), gg.complete(300), gg.crown(40),
          gg.empty(100), gg.complete_bipartite(40, 1500),
          gg.erdos_renyi(20_000, 3.0, gg.key(910, 0), name="er20k_d3"),
          gg.config_graph(2, scale_down=8), gg.config_graph(2, scale_down=6), gg.config_graph(3, scale_down=5)]


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("g", GRAPHS, ids=lambda g: g.name)
def test_bfs_matches_oracle(g, mode):
    for source in sorted({0, g.n // 2, g.n - 1}):
        check(g, source, mode)


@pytest.mark.parametrize("H", [1, 50, 10**9])
def test_bfs_threshold_and_workgroups_never_change_the_result(H):
    g = gg.config_graph(2, scale_down=6)
    hub = int(np.argmax(np.diff(g.rowptr)))
    res = check(g, hub, "hybrid", threshold=H, workgroups=7)
    assert res.topology == [int(s > H) for s in res.frontier_sizes]


def test_bfs_overflow_segments():
    """One workgroup discovers far more nodes than its segment holds (a star's centre on a grid of
    one workgroup's share): the overflow list must carry them."""
    g = gg.star(200_000, 0)
    check(g, 0, "data", workgroups=64)
    check(g, 5, "hybrid", workgroups=64)


def test_bfs_errors():
    import paper_1912_01478_amd as ip
    g = gg.path(6)
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    with pytest.raises(ip.IpgcError) as e:
        ip.bfs(rp, ci, 6)
    assert e.value.code == -1
    with pytest.raises(ip.IpgcError) as e:
        ip.bfs(rp, ci, 0, "rebuild")
    assert e.value.code == -1
    bad = ci.clone()
    bad[2] = 77
    with pytest.raises(ip.IpgcError) as e:
        ip.bfs(rp, bad, 0)
    assert e.value.code == -3
    check(g, 2, "hybrid")


# Rows of more than 2048 entries are expanded by the whole grid in chunks of 256 entries, up to 1024
# such rows staged at a time: row lengths around both edges, and a level with 1100 of them.
@pytest.mark.parametrize("g", [gg.star(2048, 0), gg.star(2049, 0), gg.star(2304, 7), gg.star(2305, 2305),
                               gg.complete_bipartite(1100, 2100)], ids=lambda g: g.name)
def test_bfs_rows_spread_over_the_grid(g):
    for source in sorted({0, g.n // 2, g.n - 1}):
        for mode in MODES:
            check(g, source, mode, workgroups=3)


def two_levels(mids, leaves):
    """A source next to `mids` nodes, each next to `leaves` nodes of its own."""
    src = np.concatenate([np.zeros(mids, dtype=np.int64), np.repeat(np.arange(1, mids + 1), leaves)])
    return gg.from_pairs(1 + mids + mids * leaves, src, np.arange(1, 1 + mids + mids * leaves), "%dx%d" % (mids, leaves))


# One wavefront's frontier nodes reach more nodes than the workgroup's segment holds (n / 64 + 1024): thread rows
# at the edges of 16 entries and of the 32 of a thread, wavefront rows, and several levels on two workgroups.
@pytest.mark.parametrize("g", [two_levels(64, 31), two_levels(64, 30), two_levels(63, 32), two_levels(33, 2047), two_levels(64, 17),
                               two_levels(64, 16), two_levels(64, 15)], ids=lambda g: g.name)
def test_bfs_overflow_from_one_wavefront(g):
    for mode in MODES:
        check(g, 0, mode, workgroups=64)
        check(g, g.n - 1, mode)


# One workgroup: at and past its nodes (32 768) and entries (196 608), rows at the edges of a thread's (32), a
# wavefront's (1024) and those for all threads, frontiers of more than 1024 nodes, many levels, unreached nodes.
@pytest.mark.parametrize("g", [gg.empty(1), gg.path(2), gg.path(3000), gg.star(32767, 0), gg.star(32767, 32767), gg.star(32768, 32768),
                               gg.path(32768), gg.complete_bipartite(96, 1024), gg.complete_bipartite(95, 1025), gg.complete(443),
                               gg.complete(444), two_levels(1000, 32), two_levels(990, 33), two_levels(31, 1024), two_levels(31, 1023),
                               gg.erdos_renyi(32768, 3.0, gg.key(912, 0)), gg.erdos_renyi(32769, 3.0, gg.key(912, 1)),
                               gg.rmat(13, 12, gg.key(912, 2)), gg.rmat(15, 3, gg.key(912, 3))], ids=lambda g: "%s_%d" % (g.name, g.n))
def test_bfs_on_one_workgroup(g):
    for source in sorted({0, g.n // 2, g.n - 1}):
        check(g, source, "hybrid")
        check(g, source, "data")


def test_bfs_checks_come_before_any_row_is_read():
    """Bad row pointers and ids anywhere in the entry array, also in entries past the last full stride."""
    import paper_1912_01478_amd as ip
    g = gg.erdos_renyi(5003, 7.0, gg.key(911, 0))
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    for at, value in ((0, -1), (g.m // 2, g.n), (g.m - 1, 2**31 - 1)):
        bad = ci.clone()
        bad[at] = value
        with pytest.raises(ip.IpgcError) as e:
            ip.bfs(rp, bad, 0)
        assert e.value.code == -3
    for at, value in ((0, 1), (g.n, g.m - 1), (g.n // 2, -4), (g.n // 2, g.m + 1)):
        bad = rp.clone()
        bad[at] = value
        with pytest.raises(ip.IpgcError) as e:
            ip.bfs(bad, ci, 0)
        assert e.value.code == -3
    check(g, 0, "hybrid")


@pytest.mark.parametrize("H", [1, 50, 19999, 20000])
def test_small_graphs_sweep_below_a_callers_threshold(H):
    """An H below the node count asks for sweeps over the grid; from there on no level is one."""
    g = GRAPHS[8]
    for source in (0, g.n - 1):
        res = check(g, source, "hybrid", threshold=H)
        assert res.topology == [int(s > H) for s in res.frontier_sizes]
        check(g, source, "data", threshold=H)

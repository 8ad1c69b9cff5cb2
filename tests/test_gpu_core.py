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

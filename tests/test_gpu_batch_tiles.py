"""The batched count's tiles: pieces and rows that cross a tile's 512 entries,
rows longer than several pieces, runs of empty rows longer than the row starts
a tile keeps, graphs on both sides of the exact-filter bound, lists that end
at the last column, and the counting kernel without forward records.  T, |H|
and levels of every graph equal the oracle's, element by element (integers:
no tolerance)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _pad(g, n):
    """g with isolated vertices up to n, its own vertices spread evenly."""
    at = (np.arange(g.n, dtype=np.int64) * n) // g.n
    return graphgen.Graph(n, at[g.src].astype(np.int32), at[g.dst].astype(np.int32))


def _cases():
    hub = graphgen.wheel(5000)  # one row of 4999 entries at id 0
    hub_last = graphgen.Graph(5000, (4999 - hub.src).astype(np.int32), (4999 - hub.dst).astype(np.int32))
    one = [("rmat%d" % s, graphgen.rmat(s, 16, seed=3)) for s in (6, 9, 12)]
    return one + [
        ("hub first", hub), ("hub last", hub_last),
        ("K513", graphgen.complete(513)), ("K3", graphgen.complete(3)), ("edge", graphgen.path(2)),
        ("sparse rows", _pad(graphgen.rmat(7, 16, seed=5), 60000)),
        ("exact bound 64 rows", graphgen.relabel(graphgen.barabasi_albert(1024, 8, 2), 9)),
        ("past the exact bound", graphgen.relabel(graphgen.barabasi_albert(1025, 8, 2), 9)),
        ("er 65536", graphgen.erdos_renyi(65536, 24.0 / 65535, 4)),
        ("ba 30011", graphgen.barabasi_albert(30011, 13, 6)),
    ]


def _expect(g):
    c = oracle.from_graph(g)
    lv = oracle.bfs_levels(c)
    return oracle.count(c, lv.levels).triangles, len(oracle.cover_edges(c, lv.levels)[0]), lv.levels


@pytest.fixture(scope="module")
def cases():
    got = [(name, g, _expect(g)) for name, g in _cases()]
    return got


@pytest.mark.parametrize("tuning", [None, dict(batch_block=64), dict(batch_block=512), dict(batch_piece=1024),
                                    dict(batch_piece=1500, batch_block=512, batch_blocks_per_cu=1),
                                    dict(batch_piece=100000, batch_block=64)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_tiles_against_oracle(cases, tuning, noalloc):
    import paper_2210_00389_amd as tc
    graphs = [g for _, g, _ in cases]
    # 70 graphs of isolated vertices: 4.6 M vertices, so that the static array has no room for the records
    empty = graphgen.Graph(65536, np.zeros(0, np.int32), np.zeros(0, np.int32))
    for pick in ([graphs + [empty] * 70] if noalloc else [graphs, graphs[4:8]]):
        b = tc.Batch.from_graphs(pick)
        print(f"case: {b.num_graphs} graphs, {tuning}, noalloc {noalloc}", flush=True)
        r = tc.count_batch(b, tuning, return_levels=True, noalloc=noalloc)
        T, H, lev = r.triangles.cpu().numpy(), r.h_count.cpu().numpy(), r.levels.cpu().numpy()
        at = 0
        want = {id(g): e for _, g, e in cases}
        for i, g in enumerate(pick):
            t, h, lv = want.get(id(g), (0, 0, np.zeros(65536, np.int32)))
            assert (T[i], H[i]) == (t, h), i
            assert np.array_equal(lev[at:at + g.n], lv), i
            at += g.n


@pytest.mark.parametrize("i", range(13))
def test_one_graph_against_oracle(cases, i):
    import paper_2210_00389_amd as tc
    name, g, (t, h, lv) = cases[i]
    print(f"case: one graph, {name}", flush=True)
    G = tc.from_host_pairs(g.n, g.src, g.dst)
    r = tc.count(G, return_levels=True, tuning=dict(small_max_nnz=1 << 22))
    assert (r.T, r.h) == (t, h)
    assert np.array_equal(r.levels.cpu().numpy(), lv)
    st = tc.read_stats()
    assert (st["n"], st["nnz"], st["h"]) == (g.n, G.nnz, h)


def _levels_cases():
    rng = np.random.RandomState(3)
    small = graphgen.disjoint_union([graphgen.path(int(k)) for k in rng.randint(1, 9, 900)])
    big = graphgen.disjoint_union([graphgen.path(int(k)) for k in rng.randint(2, 9, 3000)])
    return [
        ("small components", graphgen.relabel(graphgen.disjoint_union([graphgen.rmat(11, 8, seed=1), small]), 2)),
        ("more of them than listed", graphgen.relabel(graphgen.disjoint_union([graphgen.rmat(10, 8, seed=1), big]), 4)),
        ("two halves", graphgen.relabel(graphgen.disjoint_union([graphgen.erdos_renyi(9000, 6 / 9000, 5),
                                                                 graphgen.erdos_renyi(8000, 6 / 8000, 6)]), 7)),
        ("isolated and a path", graphgen.relabel(_pad(graphgen.path(2500), 60000), 8)),
        ("chung-lu", graphgen.chung_lu(8001, mean_degree=6, seed=9)),
        ("long tail", graphgen.relabel(graphgen.disjoint_union([graphgen.complete(60), graphgen.path(6144)]), 1)),
        ("longer tail", graphgen.relabel(graphgen.disjoint_union([graphgen.complete(60), graphgen.path(6145)]), 1)),
    ]


@pytest.mark.parametrize("i", range(7))
def test_levels_of_other_components(i):
    import paper_2210_00389_amd as tc
    name, g = _levels_cases()[i]
    for root in (-1, g.n // 2):
        print(f"case: {name}, root {root}", flush=True)
        c = oracle.from_graph(g)
        lv = oracle.bfs_levels(c, root)
        G = tc.from_host_pairs(g.n, g.src, g.dst)
        r = tc.count(G, root=root, return_levels=True)
        assert np.array_equal(r.levels.cpu().numpy(), lv.levels)
        assert (r.T, r.h) == (oracle.count(c, lv.levels).triangles, len(oracle.cover_edges(c, lv.levels)[0]))
    # beside other graphs, in a batch of its own launch sequence
    b = tc.Batch.from_graphs([g] * 130)
    lv = oracle.bfs_levels(c).levels
    r = tc.count_batch(b, return_levels=True)
    assert np.array_equal(r.levels.cpu().numpy(), np.tile(lv, 130))

"""Tiles of the forward entries of whole rows: batches of rows whose forward
parts fill a tile exactly, overfill it or are empty, long stretches of empty
rows, rows cut by tiles and pieces with more entries beyond than the tile
holds, and more hits than the queue takes.  T and |H| equal the oracle's, in a
batch and (with more vertices) counted alone (integers: no tolerance)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _g(n, s, d):
    return graphgen.Graph(n, np.asarray(s, np.int32), np.asarray(d, np.int32))


def _hub(n, degree, at, seed):
    """Vertex `at` joined to `degree` others above it, these joined at random."""
    r = np.random.default_rng(seed)
    leaf = at + 1 + np.arange(degree)
    s = np.concatenate([np.full(degree, at), r.choice(leaf, 3 * degree), np.zeros(20, int)])
    d = np.concatenate([leaf, r.choice(leaf, 3 * degree), leaf[:20]])
    return _g(n, s, d)


def _shift(g, n, by):
    return _g(n, g.src.astype(np.int64) + by, g.dst.astype(np.int64) + by)


def _both(n):
    r = np.random.default_rng(1)
    ends = np.concatenate([np.arange(40), n - 40 + np.arange(40)])
    s, d = np.triu_indices(80, 1)
    star = _g(n, np.arange(20000), np.full(20000, n - 1))
    return {
        "leaves below their hub": star,
        "leaves above their hub": _g(n, np.zeros(20000, int), 1 + np.arange(20000)),
        "path": _g(n, np.arange(20000), 1 + np.arange(20000)),
        "two ends": _g(n, ends[s], ends[d]),
        "triangles apart": _g(n, np.repeat(np.arange(0, n - 900, 700), 3) + np.tile([0, 0, 300], len(range(0, n - 900, 700))),
                              np.repeat(np.arange(0, n - 900, 700), 3) + np.tile([300, 601, 601], len(range(0, n - 900, 700)))),
        "hub 600": _hub(n, 600, 1, 2), "hub 1100": _hub(n, 1100, 3, 3), "hub 1600": _hub(n, 1600, 1, 4),
        "hub 9000": _hub(n, 9000, 2, 5),
        "clique 90": _shift(graphgen.complete(90), n, 7), "clique 700": _shift(graphgen.complete(700), n, 3000),
        "rows of 256": _g(n, np.repeat(np.arange(2000), 256), 2000 + r.integers(0, 3000, 2000 * 256)),
    }


NAMES = list(_both(2 ** 16))


def _want(g):
    c = oracle.from_graph(g)
    lv = oracle.bfs_levels(c).levels
    return c, oracle.count(c, lv).triangles, len(oracle.cover_edges(c, lv)[0])


@pytest.mark.parametrize("name", NAMES)
def test_one_of_more_vertices(name):
    import paper_2210_00389_amd as tc
    for n in (70001, 400000):
        print(f"case: {name}, n {n}", flush=True)
        c, t, h = _want(_both(n)[name])
        r = tc.count(tc.from_host_csr(c.n, c.row_offsets, c.cols))
        assert (r.T, r.h) == (t, h)


@pytest.mark.parametrize("tuning", [None, dict(batch_block=64), dict(batch_block=512), dict(batch_piece=1024),
                                    dict(batch_piece=1 << 20)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_in_a_batch(tuning, noalloc):
    import paper_2210_00389_amd as tc
    graphs = list(_both(2 ** 16).values()) + list(_both(20011).values())
    want = [_want(g)[1:] for g in graphs]
    if noalloc:  # more vertices than the static array has room for records of
        graphs += [graphgen.Graph(65536, np.zeros(0, np.int32), np.zeros(0, np.int32))] * 70
        want += [(0, 0)] * 70
    print(f"case: {len(graphs)} graphs, {tuning}, noalloc {noalloc}", flush=True)
    for pick in ([range(len(graphs))] + ([] if noalloc else [[i] for i in range(len(graphs))])):
        r = tc.count_batch(tc.Batch.from_graphs([graphs[i] for i in pick]), tuning, noalloc=noalloc)
        got = list(zip(r.triangles.tolist(), r.h_count.tolist()))
        assert got == [want[i] for i in pick], [NAMES[i % len(NAMES)] for i in pick]


@pytest.mark.parametrize("tuning", [None, dict(batch_piece=1024), dict(batch_piece=1024, batch_block=64),
                                    dict(batch_piece=1500, batch_block=512)])
def test_pieces_below_a_large_batchs_default(tuning):
    """34 M entries: the default piece is longer than the smallest to ask for, and the workspace serves both."""
    import paper_2210_00389_amd as tc
    g = graphgen.erdos_renyi(65536, 12.0 / 65535, 8)
    other = graphgen.barabasi_albert(30011, 9, 3)
    pick = [g, other] * 27
    want = [_want(g)[1:], _want(other)[1:]] * 27
    b = tc.Batch.from_graphs(pick)
    assert b.cols.numel() > 1 << 25
    print(f"case: 54 graphs, {b.cols.numel()} entries, {tuning}", flush=True)
    r = tc.count_batch(b, tuning, ws=tc.Workspace())
    assert list(zip(r.triangles.tolist(), r.h_count.tolist())) == want

"""Levels of small graphs searched by one workgroup, where a row's length
decides who expands it: stars, wheels and cliques as the searched component and
beside it, around the bounds of a remainder that is levelled at once.  T, |H|
and levels equal the oracle's, alone and in a batch (integers: no tolerance);
times are compared with those of the same search without the long row."""
import statistics

import numpy as np
import pytest
import torch

import graphgen
import oracle

pytestmark = pytest.mark.gpu

U = graphgen.disjoint_union


def _rev(g):
    return graphgen.Graph(g.n, (g.n - 1 - g.src).astype(np.int32), (g.n - 1 - g.dst).astype(np.int32))


def _rest(h):
    """h beside a larger star, in both orders of the ids."""
    g = U([graphgen.star(8000), h])
    return [g, _rev(g)]


REST = {
    **{f"star {k}": (lambda k=k: _rest(graphgen.star(k))) for k in (2, 64, 65, 66, 67, 1000, 6143, 6144, 6145)},
    **{f"clique {k}": (lambda k=k: _rest(graphgen.complete(k))) for k in (64, 65, 66, 67, 256, 257, 400)},
    "wheels": lambda: _rest(U([graphgen.wheel(k) for k in (5, 64, 66, 80, 700)])),
    "stars and paths": lambda: _rest(graphgen.relabel(U([graphgen.star(k) for k in (3, 70, 2, 500, 66)] +
                                                        [graphgen.path(k) for k in (40, 1, 9)]), 4)),
    "many stars": lambda: _rest(U([graphgen.star(70)] * 60)),
}


def _gap(g, n):
    """g's ids spread over n, the last one on the last."""
    at = (np.arange(g.n, dtype=np.int64) * (n - 1)) // max(g.n - 1, 1)
    return graphgen.Graph(n, at[g.src].astype(np.int32), at[g.dst].astype(np.int32))


# more components than are searched one by one, in all orders of ids
MANY = {
    "3072 edges": lambda: U([graphgen.path(2)] * 3072), "3080 edges": lambda: U([graphgen.path(2)] * 3080),
    "32768 edges": lambda: U([graphgen.path(2)] * 32768),
    "edges apart": lambda: _gap(U([graphgen.path(2)] * 9000), 65536),
    "stars of 70": lambda: U([graphgen.star(70)] * 900), "wheels of 67": lambda: U([graphgen.wheel(67)] * 400),
    "stars of 3000": lambda: U([graphgen.star(3000)] * 20),
    "paths": lambda: U([graphgen.path(1 + i % 40) for i in range(3000)]),
    "long paths": lambda: U([graphgen.path(900)] * 70),
    "cliques": lambda: U([graphgen.complete(12)] * 1500), "dense": lambda: U([graphgen.complete(130)] * 60),
    "sparse random": lambda: graphgen.erdos_renyi(60000, 1.0 / 60000, 3),
    "a large one last": lambda: U([graphgen.path(3)] * 5000 + [graphgen.erdos_renyi(30000, 6.0 / 30000, 4)]),
}


@pytest.mark.parametrize("name", list(MANY))
def test_many_components(name):
    print(f"case: {name}", flush=True)
    g = MANY[name]()
    _check([g, _rev(g), graphgen.relabel(g, 11)])


def _check(graphs):
    import paper_2210_00389_amd as tc
    want = []
    for g in graphs:
        c = oracle.from_graph(g)
        lv = oracle.bfs_levels(c)
        want.append((oracle.count(c, lv.levels).triangles, len(oracle.cover_edges(c, lv.levels)[0]), lv.levels))
        r = tc.count(tc.from_host_csr(c.n, c.row_offsets, c.cols), return_levels=True)
        assert np.array_equal(r.levels.cpu().numpy(), lv.levels)
        assert (r.T, r.h) == want[-1][:2]
    r = tc.count_batch(tc.Batch.from_graphs(graphs), return_levels=True)
    assert r.triangles.cpu().tolist() == [w[0] for w in want] and r.h_count.cpu().tolist() == [w[1] for w in want]
    assert np.array_equal(r.levels.cpu().numpy(), np.concatenate([w[2] for w in want]))


@pytest.mark.parametrize("name", list(REST))
def test_rows_of_a_remainder(name):
    print(f"case: {name}", flush=True)
    _check(REST[name]())


def _tree(hubs, leaves, n=65536):
    """Vertex 0 joined to hubs of as many leaves as listed, isolated vertices up to n."""
    s = [np.zeros(hubs, np.int64), np.repeat(np.arange(1, hubs + 1), leaves)]
    d = [np.arange(1, hubs + 1), hubs + 1 + np.arange(int(np.sum(leaves)))]
    return graphgen.Graph(n, np.concatenate(s).astype(np.int32), np.concatenate(d).astype(np.int32))


@pytest.mark.parametrize("hubs", [1, 2, 3, 4, 5, 8, 9, 16, 17, 40, 200])
@pytest.mark.parametrize("leaves", [15, 63, 127, 128, 129, 300])
def test_long_rows_of_a_frontier(hubs, leaves):
    import paper_2210_00389_amd as tc
    print(f"case: {hubs} hubs of {leaves} leaves", flush=True)
    size = np.full(hubs, leaves)
    size[hubs // 2] += 1700  # one far longer
    for n in (65536, int(size.sum()) + hubs + 1):
        g = _tree(hubs, size, n)
        c = oracle.from_graph(g)
        for root in (0, 1 + hubs // 2, c.n - 1):
            lv = oracle.bfs_levels(c, root)
            r = tc.count(tc.from_host_csr(c.n, c.row_offsets, c.cols), root=root, return_levels=True)
            assert np.array_equal(r.levels.cpu().numpy(), lv.levels), (n, root)
            assert (r.T, r.h) == (0, 0)


def _us(g, root=-1):
    import paper_2210_00389_amd as tc
    G = tc.from_host_pairs(g.n, g.src, g.dst)
    tc.count(G, root=root)
    t = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        tc.count(G, root=root)
        b.record()
        b.synchronize()
        t.append(a.elapsed_time(b) * 1e3)
    return statistics.median(t)


@pytest.mark.parametrize("rev", [False, True])
def test_time_of_a_star_in_the_remainder(rev):
    print(f"case: stars of 60 and 6000 beside an edge that is searched first, ids reversed {rev}", flush=True)

    def us(k):
        g = U([graphgen.path(2), graphgen.star(k)])
        return _us(_rev(g), g.n - 1) if rev else _us(g, 0)

    few, many = us(60), us(6000)
    assert many < 5 * few, (few, many)


def _search_us(g, root):
    """The search alone: the first stage of the call (the second counts the triangles)."""
    import paper_2210_00389_amd as tc
    G = tc.from_host_pairs(g.n, g.src, g.dst)
    tc.profile_enable(True)
    try:
        t = []
        for _ in range(8):
            tc.count(G, root=root)
            t.append(dict(tc.profile_read())["batch_bfs"] * 1e3)
    finally:
        tc.profile_enable(False)
    return statistics.median(t[1:])


def test_time_of_one_long_row():
    print("case: 64000 leaves of one hub and of 64", flush=True)
    one, many = _search_us(_tree(1, [64000]), 0), _search_us(_tree(64, [1000] * 64), 0)
    assert one < 1.5 * many, (one, many)


def test_time_of_many_components():
    print("case: 2000 and 20000 disjoint edges", flush=True)
    few, many = _us(U([graphgen.path(2)] * 2000)), _us(U([graphgen.path(2)] * 20000))
    assert many < 50 * few, (few, many)

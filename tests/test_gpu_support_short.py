"""tc_edge_support on lists short against the graph, around the bounds below
which triangles are added one by one or to both orientations: triangles of the
graph in runs and in any order, random triples, and a pair of vertices in every
triangle.  Supports equal a count over the list (integers: no tolerance); the
time of a short list is compared with that on a smaller graph."""
import statistics

import numpy as np
import pytest
import torch

import graphgen
import oracle

pytestmark = pytest.mark.gpu

A, B = 129998, 129999  # the edge of many triangles


def _want(c, tri):
    n = c.n
    key = np.repeat(np.arange(n), np.diff(c.row_offsets)) * n + c.cols
    sup = np.zeros(len(key), np.int64)
    t = tri.astype(np.int64)
    for x, y in ((0, 1), (0, 2), (1, 2)):
        for p, q in ((x, y), (y, x)):
            k = t[:, p] * n + t[:, q]
            at = np.searchsorted(key, k)
            ok = at < len(key)
            ok[ok] = key[at[ok]] == k[ok]
            sup += np.bincount(at[ok], minlength=len(key))
    return sup


@pytest.fixture(scope="module")
def graph():
    g = graphgen.rmat(16, 16, seed=3)
    r = np.arange(60000)  # two more vertices share 60000 triangles with as many others
    g = graphgen.Graph(130000, np.concatenate([g.src, [A], 0 * r + A, 0 * r + B]).astype(np.int32),
                       np.concatenate([g.dst, [B], r + 65536, r + 65536]).astype(np.int32))
    c = oracle.from_graph(g)
    tri = np.asarray(oracle.list_triangles(c, oracle.bfs_levels(c).levels), dtype=np.int64).reshape(-1, 3)
    return c, tri


@pytest.mark.parametrize("form", ["runs", "any order", "random", "one edge"])
@pytest.mark.parametrize("count", [1, 63, 64, 65, 255, 256, 257, 20000, 131071, 131072, 131073, 150000, 300000, "fifth",
                                   "fifth + 1", 500000])
def test_short_lists(graph, form, count):
    import paper_2210_00389_amd as tc
    c, tri = graph
    fifth = len(c.cols) // 5
    assert 300000 < fifth < 500000
    k = {"fifth": fifth, "fifth + 1": fifth + 1}.get(count, count)
    rng = np.random.RandomState(k)
    if form == "one edge":
        t = np.stack([np.full(k, A), 65536 + np.arange(k) % 60000, np.full(k, B)], axis=1)
    elif form == "random":
        t = rng.randint(0, c.n, (k, 3))
    else:
        t = tri[np.arange(k) % len(tri)]
        if form == "any order":
            t = t[rng.permutation(k)]
    t = np.take_along_axis(t, rng.rand(k, 3).argsort(axis=1), axis=1).astype(np.int32)
    print(f"case: {form}, {k} triples, {len(c.cols)} entries", flush=True)
    sup = tc.edge_support(tc.from_host_csr(c.n, c.row_offsets, c.cols), torch.from_numpy(t).cuda())
    assert np.array_equal(sup.cpu().numpy(), _want(c, t))


def test_time_of_a_short_list():
    import paper_2210_00389_amd as tc

    def us(n):
        r = np.random.default_rng(n)
        G = tc.from_host_pairs(n, r.integers(0, n, 8 * n), r.integers(0, n, 8 * n))
        tri = torch.from_numpy(r.integers(0, n, (100, 3)).astype(np.int32)).cuda()
        tc.edge_support(G, tri)
        t = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            tc.edge_support(G, tri)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b) * 1e3)
        return statistics.median(t)

    print("case: 100 triples on 160 thousand and on 16 million entries", flush=True)
    small, large = us(10007), us(1000003)
    assert large < 5 * small, (small, large)


def test_time_of_a_list_of_a_seventh_of_the_entries():
    import paper_2210_00389_amd as tc
    g = graphgen.rmat(18, 16, seed=1)
    G = tc.from_host_pairs(g.n, g.src, g.dst)
    tri = tc.list_triangles(G).tri

    def us(k):
        tc.edge_support(G, tri[:k])
        t = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            tc.edge_support(G, tri[:k])
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b) * 1e3)
        return statistics.median(t)

    print("case: a seventh and a quarter of the entries as triangles", flush=True)
    short, long = us(G.nnz // 7), us(G.nnz // 4)
    assert short < 0.75 * long, (short, long)

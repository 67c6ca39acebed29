"""Counts of a graph with one hub around the largest degree that is counted on
the caller's CSR: the hub's forward list, but for one entry its whole row, is
streamed from the edge (0, hub), and the triangles there lie at the list's
first and last entries.  T, |H| and levels equal the oracle's (integers: no
tolerance); the statistics say which path the graph took."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

N, DEG, HUB = 1_000_003, 16, 1


@pytest.fixture(scope="module")
def pairs():
    r = np.random.default_rng(5)
    m = N * DEG // 2
    s, d = r.integers(2, N, m), r.integers(2, N, m)
    return s, d, 2 + r.permutation(N - 2)


@pytest.mark.parametrize("degree,direct", [(65527, True), (65528, True), (65529, False), (65535, False), (65536, False)])
def test_hub_at_the_bound(pairs, degree, direct):
    import paper_2210_00389_amd as tc
    s, d, perm = pairs
    leaves = np.sort(perm[:degree - 1])
    ends = np.concatenate([leaves[:9], leaves[-9:]])  # joined to vertex 0 as well
    g = graphgen.Graph(N, np.concatenate([s, np.full(degree - 1, HUB), [0], np.zeros(18, np.int64)]).astype(np.int32),
                       np.concatenate([d, leaves, [HUB], ends]).astype(np.int32))
    c = oracle.from_graph(g)
    assert int(np.diff(c.row_offsets).max()) == degree
    print(f"case: hub of degree {degree}", flush=True)
    lv = oracle.bfs_levels(c)
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    r = tc.count(G, return_levels=True)
    st = tc.read_stats()
    assert (r.T, r.h) == (oracle.count(c, lv.levels).triangles, len(oracle.cover_edges(c, lv.levels)[0]))
    assert np.array_equal(r.levels.cpu().numpy(), lv.levels)
    assert (st["descriptors"] == 0) == direct

"""Counts of graphs beyond the one-graph path whose degrees are even enough to
be counted without the relabelling, over the forms that rule accepts: uniform
and power-law graphs, more than 65536 vertices, rows longer than a tile, many
empty rows, other components, given roots.  T, |H| and levels equal the
oracle's and those of the relabelled path (integers: no tolerance); the
statistics say which path a graph took."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _spread(g, n):
    at = (np.arange(g.n, dtype=np.int64) * n) // g.n
    return graphgen.Graph(n, at[g.src].astype(np.int32), at[g.dst].astype(np.int32))


CASES = {
    "er 65537": (lambda: graphgen.erdos_renyi(65537, 16.0 / 65536, 3), True),
    "er 300007": (lambda: graphgen.erdos_renyi(300007, 9.0 / 300006, 4), True),
    "ba 70001": (lambda: graphgen.relabel(graphgen.barabasi_albert(70001, 9, 5), 6), True),
    "chung-lu 100003": (lambda: graphgen.chung_lu(100003, mean_degree=12, seed=7), True),
    "rmat 14": (lambda: graphgen.rmat(14, 16, seed=8), True),
    "sparse rows": (lambda: _spread(graphgen.erdos_renyi(20000, 30.0 / 19999, 9), 3_000_001), True),
    "wheels": (lambda: graphgen.relabel(graphgen.disjoint_union([graphgen.wheel(4000)] * 40), 10), False),
    "long rows": (lambda: graphgen.relabel(graphgen.disjoint_union([graphgen.wheel(1500)] * 110), 11), True),
    "triangles": (lambda: graphgen.relabel(graphgen.disjoint_union([graphgen.complete(3)] * 90000), 12), True),
    "cliques": (lambda: graphgen.relabel(graphgen.disjoint_union([graphgen.complete(120)] * 40), 13), True),
    "rmat 17": (lambda: graphgen.rmat(17, 16, seed=14), False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_direct_equals_oracle_and_relabelled(name):
    import paper_2210_00389_amd as tc
    make, direct = CASES[name]
    g = make()
    c = oracle.from_graph(g)
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    assert not (c.n <= 65536 and G.nnz <= 1 << 18)
    for root in (-1, c.n // 3):
        print(f"case: {name}, root {root}", flush=True)
        lv = oracle.bfs_levels(c, root)
        T = oracle.count(c, lv.levels).triangles
        h = len(oracle.cover_edges(c, lv.levels)[0])
        r = tc.count(G, root=root, return_levels=True)
        st = tc.read_stats()
        assert (r.T, r.h) == (T, h)
        assert np.array_equal(r.levels.cpu().numpy(), lv.levels)
        assert (st["n"], st["nnz"], st["h"], st["num_levels"]) == (c.n, G.nnz, h, lv.num_levels)
        assert (st["descriptors"] == 0) == direct
        s = tc.count(G, root=root, tuning=dict(small_max_n=-1))
        assert (s.T, s.h) == (T, h)
        assert tc.read_stats()["descriptors"] > 0

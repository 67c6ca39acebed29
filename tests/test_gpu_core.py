"""Counts whose lists are streamed as 16-bit core offsets (graphs of at least
2^22 entries): levels smaller and larger than the core, anchors with few, many
and only entries outside it, chunks whose records outside the core do and do
not fit beside the others, two and four degree groups, several components.  T
and |H| equal the oracle's and the per-vertex counts (which stream whole
32-bit lists) sum to 3 T (integers: no tolerance)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

U = graphgen.disjoint_union
GRAPHS = {
    "rmat 18": lambda: graphgen.rmat(18, 16, seed=5),
    "er 200003": lambda: graphgen.erdos_renyi(200003, 26.0 / 200002, 6),
    "chung-lu 250007": lambda: graphgen.chung_lu(250007, mean_degree=24, seed=7),
    "two components": lambda: graphgen.relabel(U([graphgen.rmat(17, 16, seed=8),
                                                  graphgen.erdos_renyi(150001, 18.0 / 150000, 9)]), 10),
}
TUNINGS = [{}, dict(bin0_max_desc=1), dict(bin0_max_desc=1, light_max=1, dn_light=1, degree_groups=4),
           dict(bin0_max_desc=1, up_anchor_min=32, item_log2=12), dict(bitmap_desc_words=1, bitmap_member_words=1)]


@pytest.fixture(scope="module", params=list(GRAPHS))
def graph(request):
    c = oracle.from_graph(GRAPHS[request.param]())
    assert len(c.cols) >= 1 << 22
    lv = oracle.bfs_levels(c)
    return request.param, c, oracle.count(c, lv.levels).triangles, len(oracle.cover_edges(c, lv.levels)[0])


@pytest.mark.parametrize("tuning", TUNINGS)
def test_core_streams_equal_oracle(graph, tuning):
    import paper_2210_00389_amd as tc
    name, c, T, h = graph
    print(f"case: {name}, {tuning}", flush=True)
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    r = tc.count(G, tuning=dict(tuning, small_max_n=-1))
    st = tc.read_stats()
    assert (r.T, r.h) == (T, h)
    if "bin0_max_desc" in tuning:  # every heavy anchor streams core parts
        assert st["heavy_elems"] > sum(st["bin_elems"])
    p = tc.count(G, per_vertex=True, tuning=dict(tuning, small_max_n=-1))
    assert (p.T, p.h) == (T, h)
    assert int(p.per_vertex.sum().item()) == 3 * T


def test_root_in_a_small_component():
    import paper_2210_00389_amd as tc
    g = U([graphgen.rmat(18, 16, seed=11), graphgen.wheel(300)])
    c = oracle.from_graph(g)
    root = c.n - 150
    lv = oracle.bfs_levels(c, root)
    print("case: root in the wheel beside rmat 18", flush=True)
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    r = tc.count(G, root=root, return_levels=True, tuning=dict(small_max_n=-1))
    assert (r.T, r.h) == (oracle.count(c, lv.levels).triangles, len(oracle.cover_edges(c, lv.levels)[0]))
    assert np.array_equal(r.levels.cpu().numpy(), lv.levels)

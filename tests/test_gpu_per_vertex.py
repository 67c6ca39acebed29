"""Per-vertex counts of the heavy bins: probe sets far larger and far smaller
than the slots kept for apexes, streams of many chunks (their counts are added
once a batch), several items an anchor, and every table kind.  Each vertex's
count equals the oracle's (integers: no tolerance)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

U = graphgen.disjoint_union
GRAPHS = {
    "clique 90": lambda: graphgen.complete(90), "clique 900": lambda: graphgen.complete(900),
    "wheel": lambda: graphgen.wheel(6001),
    "rmat 13": lambda: graphgen.rmat(13, 16, seed=4),
    "chung-lu": lambda: graphgen.chung_lu(40011, mean_degree=24, seed=5),
    "cliques apart": lambda: graphgen.relabel(U([graphgen.complete(k) for k in (33, 40, 200, 513, 600)]), 6),
}
TUNINGS = [{}, dict(light_max=1, dn_light=1), dict(light_max=1, dn_light=1, bitmap_desc_words=1, bitmap_member_words=1),
           dict(bin0_max_desc=1, item_log2=12), dict(bins_mode=2, up_anchor_min=32)]


@pytest.fixture(scope="module", params=list(GRAPHS))
def graph(request):
    c = oracle.from_graph(GRAPHS[request.param]())
    tri = oracle.list_triangles(c, oracle.bfs_levels(c).levels)
    return request.param, c, np.bincount(tri.ravel(), minlength=c.n)


@pytest.mark.parametrize("tuning", TUNINGS)
def test_per_vertex_equals_oracle(graph, tuning):
    import paper_2210_00389_amd as tc
    name, c, want = graph
    print(f"case: {name}, {tuning}", flush=True)
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    r = tc.count(G, per_vertex=True, tuning=dict(tuning, small_max_n=-1))
    assert np.array_equal(r.per_vertex.cpu().numpy(), want)
    assert 3 * r.T == want.sum()

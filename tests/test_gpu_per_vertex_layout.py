"""Per-vertex counts, vertex by vertex, where the numbering and the layout
change hands: rows at the bounds of the short, wave, block and segmented
categories, and vertex counts at the edges of the numbering's tiles.  Each
vertex's count equals the oracle's (integers: no tolerance)."""
import numpy as np
import pytest

import graphgen
import oracle
from test_gpu_layout import _hubs, _strip

pytestmark = pytest.mark.gpu


def _check(g):
    import paper_2210_00389_amd as tc
    c = oracle.from_graph(g)
    want = np.bincount(oracle.list_triangles(c, oracle.bfs_levels(c).levels).ravel(), minlength=c.n)
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    for t in (None, dict(degree_groups=4)):
        got = tc.count(G, per_vertex=True, tuning=t)
        assert np.array_equal(got.per_vertex.cpu().numpy(), want) and 3 * got.T == want.sum()


@pytest.mark.parametrize("degrees", [[32, 33], [512, 513, 33], [4096, 4097, 512], [6144, 6145, 2048, 4096],
                                     [9000] * 40 + [600] * 300 + [40] * 300, [31]])
def test_row_categories(degrees):
    print(f"case: hubs {degrees[:4]}...", flush=True)
    _check(graphgen.relabel(_hubs(degrees, 20011, len(degrees)), 7))


@pytest.mark.parametrize("n", [1023, 1024, 1025, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 20) + 4097])
def test_tile_edges(n):
    print(f"case: n {n}", flush=True)
    k = min(n - 40, 900)
    _check(graphgen.relabel(graphgen.disjoint_union([graphgen.complete(40), _strip(k, n - 40 - k)]), 5))


def test_uneven_graph_of_many_tiles():
    print("case: preferential graph on 2^20 + 30000 ids", flush=True)
    g = graphgen.barabasi_albert(300000, 4, 3)
    at = np.sort(np.random.default_rng(2).choice((1 << 20) + 30000, g.n, replace=False))
    _check(graphgen.relabel(graphgen.Graph((1 << 20) + 30000, at[g.src].astype(np.int32), at[g.dst].astype(np.int32)), 8))

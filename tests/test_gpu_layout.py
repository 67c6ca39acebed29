"""The level-class layout where its kernels change hands: rows at the bounds of
the short, wave, block and segmented categories, vertex counts at the edges of
the numbering's tiles, and graphs whose groups just fit, just miss or far
exceed the one-pass numbering.  T, |H|, per-vertex counts and the cover-edge
list equal the oracle's (integers: no tolerance)."""
import numpy as np
import pytest
import torch

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _hubs(degrees, n, seed):
    """Hubs of exact degrees, their neighbours (the same for all) joined at random."""
    h = len(degrees)
    s = [np.full(d, i, np.int64) for i, d in enumerate(degrees)]
    d = [h + np.arange(k, dtype=np.int64) for k in degrees]
    r = np.random.default_rng(seed)
    a, b = h + r.integers(0, n - h, 3 * n), h + r.integers(0, n - h, 3 * n)
    return graphgen.Graph(n, np.concatenate(s + [a]).astype(np.int32), np.concatenate(d + [b]).astype(np.int32))


def _strip(k, pad=0):
    """A strip of triangles, one level per two vertices from its end."""
    i = np.arange(k)
    return graphgen.Graph(k + pad, np.concatenate([i[:-1], i[:-2]]).astype(np.int32),
                          np.concatenate([i[1:], i[2:]]).astype(np.int32))


def _check(g, root, tunings):
    import paper_2210_00389_amd as tc
    c = oracle.from_graph(g)
    lv = oracle.bfs_levels(c, root)
    want = oracle.count(c, lv.levels)
    hu, hv = oracle.cover_edges(c, lv.levels)
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    for t in tunings:
        r = tc.count(G, root=root, tuning=dict(t, small_max_n=-1))
        assert (r.T, r.h) == (want.triangles, len(hu)), t
    p = tc.count(G, root=root, per_vertex=True, tuning=dict(small_max_n=-1))
    assert int(p.per_vertex.sum().item()) == 3 * want.triangles
    assert int(tc.count_edge_baseline(G).item()) == want.triangles
    gu, gv = tc.cover_edges(G, torch.from_numpy(lv.levels).cuda())
    assert np.array_equal(gu.cpu().numpy(), hu) and np.array_equal(gv.cpu().numpy(), hv)


@pytest.mark.parametrize("degrees", [[32, 33], [512, 513, 33], [4096, 4097, 512], [6144, 6145, 2048, 4096],
                                     [9000] * 40 + [600] * 300 + [40] * 300, [31]])
def test_row_categories(degrees):
    print(f"case: hubs {degrees[:4]}...", flush=True)
    _check(_hubs(degrees, 20011, len(degrees)), -1, [{}, dict(degree_groups=4)])


@pytest.mark.parametrize("n", [1023, 1024, 1025, (1 << 20) - 1, 1 << 20, (1 << 20) + 1])
def test_tile_edges(n):
    print(f"case: n {n}", flush=True)
    k = min(n - 40, 900)
    _check(graphgen.relabel(graphgen.disjoint_union([graphgen.complete(40), _strip(k, n - 40 - k)]), 5), -1,
           [{}, dict(degree_groups=4)])


@pytest.mark.parametrize("k", [118, 120, 122, 124, 126, 128, 244, 246, 248, 250, 252, 254, 256, 258, 3000])
def test_deep_graphs(k):
    print(f"case: strip of {k}", flush=True)
    _check(_strip(k), 0, [dict(degree_groups=2), dict(degree_groups=4)])

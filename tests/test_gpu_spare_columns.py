"""Graphs whose column buffer is longer than their rows (row_offsets[n] below
the entry count that the call is given): the entries past the rows belong to no
row and change nothing, whatever ids they hold.  Every result equals the
oracle's (integers: no tolerance)."""
import numpy as np
import pytest
import torch

import graphgen
import oracle

pytestmark = pytest.mark.gpu

GRAPHS = {
    "edge": lambda: graphgen.path(2), "rmat 11": lambda: graphgen.rmat(11, 16, seed=2),
    "rmat 15": lambda: graphgen.relabel(graphgen.disjoint_union([graphgen.rmat(15, 16, seed=3), graphgen.path(50)]), 4),
    "er 70001": lambda: graphgen.erdos_renyi(70001, 9.0 / 70000, 5),
    "empty rows": lambda: graphgen.Graph(40000, np.array([0, 0, 1], np.int32), np.array([1, 2, 2], np.int32)),
}


def _keys(tri, n):
    t = np.sort(np.asarray(tri, dtype=np.int64).reshape(-1, 3), axis=1)
    return np.sort((t[:, 0] * n + t[:, 1]) * n + t[:, 2])


@pytest.mark.parametrize("spare", [1, 2047, 2048, 2049, 100000])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_spare_columns(name, spare):
    import paper_2210_00389_amd as tc
    c = oracle.from_graph(GRAPHS[name]())
    lv = oracle.bfs_levels(c)
    hu, hv = oracle.cover_edges(c, lv.levels)
    tri = oracle.list_triangles(c, lv.levels)
    print(f"case: {name}, {spare} spare columns", flush=True)
    junk = np.random.default_rng(spare).integers(0, c.n, spare).astype(np.int32)
    G = tc.Graph(c.n, torch.from_numpy(c.row_offsets).cuda(), torch.from_numpy(np.concatenate([c.cols, junk])).cuda())
    lev, num = tc.bfs_levels(G)
    assert num == lv.num_levels and np.array_equal(lev.cpu().numpy(), lv.levels)
    gu, gv = tc.cover_edges(G, lev)
    assert np.array_equal(gu.cpu().numpy(), hu) and np.array_equal(gv.cpu().numpy(), hv)
    for t in (None, dict(small_max_n=-1)):
        r = tc.count(G, tuning=t, return_levels=True)
        assert (r.T, r.h) == (len(tri), len(hu)) and np.array_equal(r.levels.cpu().numpy(), lv.levels)
    pv = tc.count(G, per_vertex=True).per_vertex.cpu().numpy()
    assert np.array_equal(pv, np.bincount(tri.ravel(), minlength=c.n))
    assert int(tc.count_edge_baseline(G).item()) == len(tri)
    got = tc.list_triangles(G)
    assert np.array_equal(_keys(got.tri.cpu().numpy(), c.n), _keys(tri, c.n))
    sup = tc.edge_support(G, got.tri).cpu().numpy()
    assert not sup[len(c.cols):].any() and sup.sum() == 6 * len(tri)
    exact = tc.edge_support(tc.from_host_csr(c.n, c.row_offsets, c.cols), got.tri).cpu().numpy()
    assert np.array_equal(sup[:len(c.cols)], exact)


@pytest.mark.parametrize("lead", [1, 2047, 2048, 5000])
def test_offsets_that_begin_later(lead):
    import paper_2210_00389_amd as tc
    c = oracle.from_graph(graphgen.rmat(11, 16, seed=6))
    lv = oracle.bfs_levels(c).levels
    hu, hv = oracle.cover_edges(c, lv)
    print(f"case: rows from entry {lead}", flush=True)
    junk = np.random.default_rng(lead).integers(0, c.n, lead + 10).astype(np.int32)
    G = tc.Graph(c.n, torch.from_numpy(c.row_offsets + lead).cuda(),
                 torch.from_numpy(np.concatenate([junk[:lead], c.cols, junk[lead:]])).cuda())
    gu, gv = tc.cover_edges(G, torch.from_numpy(lv).cuda())
    assert np.array_equal(gu.cpu().numpy(), hu) and np.array_equal(gv.cpu().numpy(), hv)

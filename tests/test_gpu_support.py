"""tc_edge_support on lists of any form: vertices in any order, repeated
triples, a vertex shared by whole waves or by none, triples with ids out of
range, with a repeated vertex or with pairs that are no edges, and list
lengths around a wave's and a block's share.  Supports equal a count over the
list (integers: no tolerance)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _want(c, tri):
    n = c.n
    row = np.repeat(np.arange(n), np.diff(c.row_offsets))
    key = row * n + c.cols
    sup = np.zeros(len(key), np.int64)
    t = tri[((tri >= 0) & (tri < n)).all(axis=1)].astype(np.int64)
    for x, y in ((0, 1), (0, 2), (1, 2)):
        for p, q in ((x, y), (y, x)):
            k = t[:, p] * n + t[:, q]
            at = np.searchsorted(key, k)
            ok = at < len(key)
            ok[ok] = key[at[ok]] == k[ok]
            sup += np.bincount(at[ok], minlength=len(key))
    return sup


@pytest.mark.parametrize("count", [0, 1, 63, 64, 65, 2047, 2048, 2049, 50000])
@pytest.mark.parametrize("form", ["random", "hub", "listed"])
def test_support_of_any_list(count, form):
    import torch
    import paper_2210_00389_amd as tc
    g = graphgen.rmat(11, 16, seed=3)
    c = oracle.from_graph(g)
    rng = np.random.RandomState(count + len(form))
    if form == "listed":
        tri = np.asarray(oracle.list_triangles(c, oracle.bfs_levels(c).levels), dtype=np.int64).reshape(-1, 3)
        tri = tri[np.arange(count) % len(tri)]
    else:
        tri = rng.randint(0, c.n, (count, 3))
        if form == "hub":
            tri[:, 0] = np.diff(c.row_offsets).argmax()
            nb = c.cols[c.row_offsets[tri[0, 0]]:c.row_offsets[tri[0, 0] + 1]] if count else c.cols
            tri[:, 1] = nb[rng.randint(0, len(nb), count)]
        bad = rng.rand(count) < 0.1
        tri[bad, rng.randint(0, 3, int(bad.sum()))] = rng.choice([-1, c.n, 2**31 - 1, -2**31, 5], int(bad.sum()))
    tri = np.take_along_axis(tri, rng.rand(count, 3).argsort(axis=1), axis=1).astype(np.int32)
    print(f"case: {form}, {count} triples", flush=True)
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    sup = tc.edge_support(G, torch.from_numpy(tri).cuda())
    assert np.array_equal(sup.cpu().numpy(), _want(c, tri))

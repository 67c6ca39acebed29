"""The cover-edge list as a compaction of the entries: tiles of 2048 entries
and their remainders, rows over many tiles, tiles of many and of nearly only
empty rows, levels that bytes tell apart and levels that they do not.  The
list equals the oracle's, element by element (integers: no tolerance)."""
import numpy as np
import pytest
import torch

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _pad(g, n):
    """g's vertices first and last, isolated ones between."""
    k = g.n // 2
    at = np.where(np.arange(g.n) < k, np.arange(g.n), n - g.n + np.arange(g.n))
    return graphgen.Graph(n, at[g.src].astype(np.int32), at[g.dst].astype(np.int32))


def _edges(m):
    """m edges: a path."""
    return graphgen.path(m + 1)


GRAPHS = {
    "edge": lambda: graphgen.path(2), "1023 edges": lambda: _edges(1023), "1024 edges": lambda: _edges(1024),
    "1025 edges": lambda: _edges(1025), "rmat 12": lambda: graphgen.rmat(12, 16, seed=2),
    "star": lambda: graphgen.star(9000), "wheel": lambda: graphgen.wheel(7001),
    "clique 300": lambda: graphgen.complete(300),
    "gap below the bound": lambda: _pad(graphgen.complete(70), 16384 + 40),
    "gap past the bound": lambda: _pad(graphgen.complete(70), 16384 + 140),
    "long gap": lambda: _pad(graphgen.rmat(9, 8, seed=3), 3000001),
    "no edges": lambda: graphgen.Graph(50, np.zeros(0, np.int32), np.zeros(0, np.int32)),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_list_equals_oracle(name):
    import paper_2210_00389_amd as tc
    c = oracle.from_graph(GRAPHS[name]())
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    r = np.random.default_rng(c.n)
    bfs = oracle.bfs_levels(c).levels
    for what, lv in [("bfs", bfs), ("zero", np.zeros(c.n, np.int32)), ("bytes", r.integers(0, 3, c.n)),
                     ("up to 255", r.choice([0, 255], c.n)), ("256", r.choice([0, 256], c.n)),
                     ("signed", r.choice([-256, -1, 0, 255, 511], c.n)),
                     ("one wide", np.where(np.arange(c.n) == c.n - 1, 256, 0)),
                     ("extremes", r.choice([np.iinfo(np.int32).min, np.iinfo(np.int32).max, 0], c.n))]:
        print(f"case: {name}, levels {what}", flush=True)
        lv = lv.astype(np.int32)
        hu, hv = oracle.cover_edges(c, lv)
        gu, gv = tc.cover_edges(G, torch.from_numpy(lv).cuda())
        assert np.array_equal(gu.cpu().numpy(), hu) and np.array_equal(gv.cpu().numpy(), hv), what

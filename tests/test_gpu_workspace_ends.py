"""No entry point writes past the workspace it asks for: every call gets a
buffer of exactly tc_workspace_bytes, inside a larger one whose rest has to keep
its contents.  Shapes where one size is far from the others: many vertices and
few pairs, many empty rows, hubs, many components, many and few small graphs."""
import numpy as np
import pytest
import torch

import graphgen

pytestmark = pytest.mark.gpu

PAD = 16 << 20
U = graphgen.disjoint_union


def _guard():
    import paper_2210_00389_amd as tc

    class Guard(tc.Workspace):
        def get(self, nbytes):
            self.all = torch.full((max(nbytes, 256) + PAD,), 0x5A, dtype=torch.uint8, device=self.device)
            self.buf = self.all[:max(nbytes, 256)]
            return self.buf

        def check(self, what):
            assert bool((self.all[self.buf.numel():] == 0x5A).all()), what

    return Guard()


def _wide(n, m):
    r = np.random.default_rng(m)
    return graphgen.Graph(n, r.integers(0, n, m).astype(np.int32), r.integers(0, n, m).astype(np.int32))


GRAPHS = {
    "one edge": lambda: graphgen.path(2), "no edges": lambda: graphgen.Graph(70000, np.zeros(0, np.int32), np.zeros(0, np.int32)),
    "5 M vertices, 3 pairs": lambda: _wide(5_000_000, 3), "5 M vertices, 5000 pairs": lambda: _wide(5_000_000, 5000),
    "rmat 10": lambda: graphgen.rmat(10, 16, seed=1), "rmat 16": lambda: graphgen.rmat(16, 16, seed=2),
    "star": lambda: graphgen.star(200000), "clique": lambda: graphgen.complete(1200),
    "components": lambda: graphgen.relabel(U([graphgen.complete(k % 40 + 2) for k in range(3000)]), 3),
    "two halves": lambda: U([graphgen.rmat(15, 16, seed=3), graphgen.path(9000)]),
    "er 100003": lambda: graphgen.erdos_renyi(100003, 12.0 / 100002, 4), "deep": lambda: graphgen.path(3000),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_graph_calls(name):
    import paper_2210_00389_amd as tc
    g = GRAPHS[name]()
    ws = _guard()
    calls = {"build": lambda: tc.from_host_pairs(g.n, g.src, g.dst, ws=ws)}
    G = calls["build"]()
    ws.check("build")
    lev, _ = tc.bfs_levels(G, ws=ws)
    ws.check("bfs")
    for what, call in {
            "validate": lambda: tc.validate(G, ws=ws), "cover": lambda: tc.cover_edges(G, lev, ws=ws),
            "count": lambda: tc.count(G, ws=ws), "relabelled": lambda: tc.count(G, ws=ws, tuning=dict(small_max_n=-1)),
            "four groups": lambda: tc.count(G, ws=ws, tuning=dict(small_max_n=-1, degree_groups=4, light_max=1, dn_light=1)),
            "per vertex": lambda: tc.count(G, ws=ws, per_vertex=True), "list": lambda: tc.list_triangles(G, cap=1000, ws=ws),
            "comparator": lambda: tc.count_edge_baseline(G, ws=ws),
            "roots": lambda: tc.select_root(G, num_candidates=2, ws=ws)}.items():
        print(f"case: {name}, {what}", flush=True)
        call()
        ws.check(what)


@pytest.mark.parametrize("tuning", [None, dict(batch_piece=1024), dict(batch_block=64, batch_piece=1024),
                                    dict(batch_piece=65536), dict(batch_block=512)])
def test_batch_calls(tuning):
    import paper_2210_00389_amd as tc
    ws = _guard()
    for what, graphs in {
            "tiny": [graphgen.path(k % 5 + 1) for k in range(3000)], "one large": [graphgen.star(65536)],
            "mixed": [graphgen.rmat(s, 16, seed=s) for s in (6, 13, 9, 15)],
            "empty rows": [_wide(65536, 3) for _ in range(20)],
            "cliques": [graphgen.complete(k) for k in (900, 30, 700)]}.items():
        print(f"case: {what}, {tuning}", flush=True)
        b = tc.Batch.from_graphs(graphs, ws=ws)
        ws.check("build")
        tc.count_batch(b, tuning, ws=ws, return_levels=True)
        ws.check(what)
        tc.count_batch(b, tuning, ws=ws, validate=True)
        ws.check(what)

"""Counts of the deepest graph of the one-workgroup path, a path of 65536
vertices searched from an end: its last level is 65535.  T, |H| and levels
equal the oracle's (integers: no tolerance), also one vertex short of it, from
the vertex beside the end, and where the ids follow the path or not."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

CASES = {
    "path 65536": lambda: graphgen.path(65536),
    "path 65536, ids at random": lambda: graphgen.relabel(graphgen.path(65536), 3),
    "path 65535": lambda: graphgen.path(65535),
    "path 65535 and an isolated vertex": lambda: graphgen.disjoint_union(
        [graphgen.path(65535), graphgen.Graph(1, np.zeros(0, np.int32), np.zeros(0, np.int32))]),
    "path 65534 and an edge": lambda: graphgen.disjoint_union([graphgen.path(65534), graphgen.path(2)]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_levels_from_both_ends(name):
    import paper_2210_00389_amd as tc
    c = oracle.from_graph(CASES[name]())
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    ends = np.flatnonzero(np.diff(c.row_offsets) == 1)
    for root in [int(ends[0]), int(ends[-1]), int(c.cols[c.row_offsets[ends[0]]]), -1]:
        print(f"case: {name}, root {root}", flush=True)
        lv = oracle.bfs_levels(c, root)
        r = tc.count(G, root=root, return_levels=True)
        assert np.array_equal(r.levels.cpu().numpy(), lv.levels), root
        assert (r.T, r.h) == (0, len(oracle.cover_edges(c, lv.levels)[0])), root

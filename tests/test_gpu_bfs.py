"""tc_bfs_levels where its launches change hands: few and many unreached
entries (one block or the grid), long rows listed for the next level and more
of them than the list holds, graphs deeper than the first group of levels,
given roots in small components.  Levels and level counts equal the oracle's
(integers: no tolerance)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _pad(g, extra):
    return graphgen.disjoint_union([g, graphgen.Graph(extra, np.zeros(0, np.int32), np.zeros(0, np.int32))])


def _hubs_chain(hubs, leaves):
    """A path of hubs, each with its own leaves, so that long rows appear one or two per level."""
    s = [i for i in range(hubs - 1)]
    d = [i + 1 for i in range(hubs - 1)]
    for i in range(hubs):
        s += [i] * leaves
        d += list(range(hubs + i * leaves, hubs + (i + 1) * leaves))
    return graphgen.Graph(hubs * (leaves + 1), np.asarray(s, np.int32), np.asarray(d, np.int32))


U = graphgen.disjoint_union
CASES = {
    "rest of a few entries": lambda: U([graphgen.rmat(13, 16, seed=2), graphgen.path(40), graphgen.cycle(9),
                                        graphgen.star(1500)]),
    "rest at the bound": lambda: U([graphgen.complete(400), graphgen.path(32769)]),
    "rest past the bound": lambda: U([graphgen.complete(400), graphgen.path(32770)]),
    "two large components": lambda: graphgen.relabel(U([graphgen.rmat(14, 16, seed=4), graphgen.erdos_renyi(
        20000, 12 / 20000, 5), graphgen.star(3000)]), 6),
    "1500 long rows top-down": lambda: _pad(graphgen.complete_bipartite(1500, 1501), 500000),
    "1024 long rows top-down": lambda: _pad(graphgen.complete_bipartite(1024, 1100), 400000),
    "chain of hubs": lambda: _pad(_hubs_chain(12, 1100), 3_000_000),
    "deep": lambda: graphgen.relabel(U([graphgen.path(5000), graphgen.path(3000), graphgen.grid(60, 70)]), 3),
    "only isolated": lambda: graphgen.Graph(70000, np.zeros(0, np.int32), np.zeros(0, np.int32)),
    "one vertex": lambda: graphgen.Graph(1, np.zeros(0, np.int32), np.zeros(0, np.int32)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_levels_equal_oracle(name):
    import paper_2210_00389_amd as tc
    g = CASES[name]()
    c = oracle.from_graph(g)
    G = tc.from_host_csr(c.n, c.row_offsets, c.cols)
    for root in (-1, 0, c.n - 1, c.n // 2):
        print(f"case: {name}, root {root}", flush=True)
        want = oracle.bfs_levels(c, root)
        lev, num = tc.bfs_levels(G, root=root)
        assert np.array_equal(lev.cpu().numpy(), want.levels), root
        assert num == want.num_levels, root

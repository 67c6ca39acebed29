"""tc_build_csr where its sort and its row offsets can go wrong: pair counts
around the sort's tiles, digit widths of every remainder, runs of empty rows
shorter and longer than one thread fills, rows before the first and after the
last entry, only loops, one pair many times, a hub, and ids out of range.
Offsets and columns equal the oracle's builder (integers: no tolerance)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _random(n, pairs, seed):
    r = np.random.RandomState(seed)
    return graphgen.Graph(n, r.randint(0, n, pairs).astype(np.int32), r.randint(0, n, pairs).astype(np.int32))


def _of(n, s, d):
    return graphgen.Graph(n, np.asarray(s, np.int32), np.asarray(d, np.int32))


CASES = {
    **{"pairs %d" % p: (lambda p=p: _random(3000, p, p)) for p in (1, 63, 64, 2047, 2048, 2049, 4096, 10241)},
    **{"n %d" % n: (lambda n=n: _random(n, 5000, n)) for n in (2, 3, 16, 17, 200, 1025, 2500, 70000, 300000)},
    "gaps of 63 to 66": lambda: _of(400, [0, 64, 129, 195], [399, 399, 399, 399]),
    "long gaps": lambda: _of(2_000_003, [7, 500_000, 1_999_000], [500_000, 1_999_000, 7]),
    "only the first rows": lambda: _of(1_000_001, [0, 0, 1], [1, 2, 2]),
    "only the last rows": lambda: _of(1_000_001, [1_000_000, 999_999], [999_998, 1_000_000]),
    "only loops": lambda: _of(1000, [5, 5, 9], [5, 5, 9]),
    "one pair 9000 times": lambda: _of(50, [3] * 4500 + [4] * 4500, [4] * 4500 + [3] * 4500),
    "hub": lambda: graphgen.star(70001),
    "rmat": lambda: graphgen.rmat(15, 16, seed=8),
    "no pairs": lambda: _of(777, [], []),
}


@pytest.mark.parametrize("name", list(CASES))
def test_build_equals_oracle(name):
    import paper_2210_00389_amd as tc
    g = CASES[name]()
    print(f"case: {name}: n {g.n}, {g.num_pairs} pairs", flush=True)
    want = oracle.from_graph(g)
    for _ in range(2):  # the second call finds the first one's workspace
        G = tc.from_host_pairs(g.n, g.src, g.dst)
        assert np.array_equal(G.row_offsets.cpu().numpy(), want.row_offsets)
        assert np.array_equal(G.cols.cpu().numpy(), want.cols)


@pytest.mark.parametrize("pair", [(-1, 3), (3, -1), (100, 3), (3, 100), (100, 100), (2**31 - 1, 0), (-2**31, 5)])
def test_ids_out_of_range(pair):
    import paper_2210_00389_amd as tc
    s = np.arange(5000, dtype=np.int32) % 100
    d = (s + 7) % 100
    s[4321], d[4321] = pair
    print(f"case: pair {pair}", flush=True)
    with pytest.raises(tc.TcError) as e:
        tc.from_host_pairs(100, s, d)
    assert e.value.status == -7

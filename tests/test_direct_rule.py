"""The rule that sends a count to the tiles of the batched kernel
(csrc/direct_rule.h), compiled for the host: the largest degree it takes, and
that a tile of the longest lists it lets through keeps every chunk in the
packed count.  A graph that passes the rule is counted without any list being
shortened, whatever ids its long lists stand at."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = r"""
#include <stdio.h>
#include <stdlib.h>
#include "direct_rule.h"
int main(int c, char** v) {
  if (c == 1) { printf("%d %d %d %u\n", tc::kTile, tc::kBChunk, tc::kChunkBits, tc::kLongList); return 0; }
  for (int i = 1; i + 3 < c; i += 4)
    printf("%d\n", (int)tc::direct_fits(atoll(v[i]), atoll(v[i + 1]), atoll(v[i + 2]), strtoull(v[i + 3], 0, 10)));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("rule")
    src, exe = str(d / "main.cpp"), str(d / "main")
    open(src, "w").write(MAIN)
    r = subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2210_00389_amd", "csrc"),
                        "-o", exe, src], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return lambda *a: [int(x) for x in subprocess.run([exe, *map(str, a)], capture_output=True, text=True,
                                                      check=True).stdout.split()]


def _hubs(n, deg, hubs, hub_deg):
    """(n, nnz, maxdeg, deg2) of a graph of even degrees with some hubs."""
    return n, n * deg + 2 * hubs * hub_deg, hub_deg, n * deg * deg + hubs * hub_deg * hub_deg


def test_longest_lists_fit_a_tile(rule):
    tile, chunk, bits, longest = rule()
    assert tile * -(-longest // chunk) < 1 << bits
    # one hub, and eleven of them beside 30 M vertices of degree 16: only the largest degree decides
    for hubs, n in ((1, 4_000_037), (11, 30_000_000)):
        for d in range(longest - 2, 65540):
            assert rule(*_hubs(n, 16, hubs, d)) == [int(d <= longest)], (hubs, d)


def test_sizes_of_ids_and_positions(rule):
    assert rule(2**31 - 2, 1000, 3, 3000) == [1] and rule(2**31 - 1, 1000, 3, 3000) == [0]
    assert rule(10**6, 2**31 - 1, 3000, 10**9) == [1] and rule(10**6, 2**31, 3000, 10**9) == [0]


# (n, entries, largest degree, sum of squared degrees, whether the direct count was the faster), timed both ways
TIMED = [
    (300007, 7199792, 51, 179940000, True),       # uniform, degree 24: 701 / 241 us
    (20011, 19517012, 1107, 19056000000, True),   # degree 1000: 2896 / 1882
    (100003, 49876292, 596, 24924000000, True),   # degree 500: 4391 / 3148
    (300007, 11989096, 21611, 2007000000, True),  # preferential, degree 40: 1177 / 760
    (30011, 592634, 732, 71640000, True),         # power law 2.1, degree 20: 290 / 140
    (100003, 1981764, 1380, 374640000, True),     # 354 / 314
    (100003, 3956514, 1942, 1147800000, False),   # degree 40: 467 / 730
    (150001, 4458896, 2042, 1258800000, False),   # degree 30: 567 / 813
    (300007, 1790248, 1348, 249600000, True),     # degree 6: 475 / 387
    (300007, 5958376, 2368, 1710000000, False),   # degree 20: 725 / 1015
    (500009, 5966818, 2389, 1534200000, False),   # degree 12: 777 / 971
    (1000003, 8959056, 2991, 2546400000, False),  # degree 9: 1185 / 1390
    (2000003, 23900808, 4777, 10662000000, False),  # degree 12: 2381 / 2868
    (1000003, 23997626, 4879, 4887000000, True),  # power law 2.5, degree 24: 2331 / 1331
    (16384, 426048, 3620, 156300000, True),       # R-MAT scale 14: 282 / 142
    (32768, 883218, 5979, 444900000, True),       # 15: 357 / 305
    (65536, 1819000, 9584, 1242600000, False),    # 16: 415 / 1024
    (131072, 1942810, 9868, 1089000000, False),   # 17, edge factor 8: 414 / 909
    (262144, 7609464, 25380, 9510000000, False),  # 18: 875 / 4494
    (1000003, 16129894, 65016, 4501200000, True),  # one hub of 65000: 1081 / 758
    (1000003, 17039874, 65028, 34104000000, False),  # eight of them: 1180 / 2003
]


@pytest.mark.parametrize("n,nnz,maxdeg,deg2,faster", TIMED)
def test_faster_path_of_timed_graphs(rule, n, nnz, maxdeg, deg2, faster):
    assert rule(n, nnz, maxdeg, deg2) == [int(faster)]

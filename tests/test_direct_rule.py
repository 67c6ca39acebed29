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

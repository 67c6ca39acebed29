"""Searches whose frontier has more long rows than one part of the list of them
holds, up to and past the list's end, and the time of one far longer row among
them.  Levels are known from the construction (integers: no tolerance); a time
is compared with that of the same search with fewer long rows."""
import statistics

import pytest
import torch

pytestmark = pytest.mark.gpu


def _hubs(hubs, leaves, longest, n):
    """Vertex 0 joined to `hubs` vertices of `leaves` leaves each and one of `longest`; isolated vertices up to n."""
    import paper_2210_00389_amd as tc
    dev = "cuda"
    size = torch.tensor([leaves] * hubs + [longest], device=dev)
    hub = torch.arange(1, hubs + 2, device=dev)
    leaf = hubs + 2 + torch.arange(int(size.sum()), device=dev)
    s = torch.cat([torch.zeros_like(hub), torch.repeat_interleave(hub, size)])
    G = tc.build_csr(n, s.to(torch.int32), torch.cat([hub, leaf]).to(torch.int32))
    want = torch.zeros(n, dtype=torch.int32, device=dev)
    want[hub], want[leaf] = 1, 2
    return G, want


@pytest.mark.parametrize("hubs", [1023, 1024, 1025, 2047, 3000])
def test_parts_of_the_list(hubs):
    import paper_2210_00389_amd as tc
    print(f"case: {hubs} hubs", flush=True)
    G, want = _hubs(hubs, 1030, 5000, 4_000_000)
    lev, num = tc.bfs_levels(G, root=0)
    assert num == 3 and torch.equal(lev, want)


@pytest.mark.parametrize("rows", [65535, 65536, 65537])
def test_end_of_the_list(rows):
    import paper_2210_00389_amd as tc
    print(f"case: {rows} rows of 1100", flush=True)
    n, a = 17_200_000, 1100
    s = torch.arange(rows, device="cuda", dtype=torch.int32).add_(a).repeat_interleave(a)
    d = torch.arange(a, device="cuda", dtype=torch.int32).repeat(rows)
    G = tc.build_csr(n, s, d)
    want = torch.zeros(n, dtype=torch.int32, device="cuda")
    want[1:a], want[a:a + rows] = 2, 1
    lev, num = tc.bfs_levels(G, root=0)
    assert num == 3 and torch.equal(lev, want)


def test_time_of_a_far_longer_row():
    import paper_2210_00389_amd as tc

    def ms(hubs):
        G, _ = _hubs(hubs, 1100, 2_000_000, 4_000_000)
        tc.bfs_levels(G, root=0)
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            tc.bfs_levels(G, root=0)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return statistics.median(t)

    print("case: 900 and 1500 hubs beside one of 2000000 leaves", flush=True)
    few, many = ms(900), ms(1500)
    assert many < 10 * few, (few, many)


def _rest(k, leaves, hub_last):
    """A clique of k vertices, then a star whose hub has its smallest or its largest id."""
    import paper_2210_00389_amd as tc
    i = torch.arange(k, device="cuda")
    s, d = i.repeat_interleave(k), i.repeat(k)
    hub = k + (leaves if hub_last else 0)
    leaf = k + torch.arange(leaves, device="cuda") + (0 if hub_last else 1)
    G = tc.build_csr(k + 1 + leaves, torch.cat([s, torch.full_like(leaf, hub)]).to(torch.int32),
                     torch.cat([d, leaf]).to(torch.int32))
    want = torch.ones(k + 1 + leaves, dtype=torch.int32, device="cuda")
    want[0] = 0
    if hub_last:
        want[k:] = 2
        want[k], want[hub] = 0, 1
    else:
        want[hub] = 0
    return G, want


@pytest.mark.parametrize("leaves", [1, 63, 64, 65, 1023, 1024, 1025, 32768, 32769, 40000])
@pytest.mark.parametrize("hub_last", [False, True])
def test_star_beside_a_component(leaves, hub_last):
    import paper_2210_00389_amd as tc
    print(f"case: {leaves} leaves, hub last {hub_last}", flush=True)
    G, want = _rest(400, leaves, hub_last)
    lev, num = tc.bfs_levels(G, root=0)
    assert num == (3 if hub_last and leaves > 1 else 2) and torch.equal(lev, want)


@pytest.mark.parametrize("hub_last", [False, True])
def test_time_of_a_star_beside_a_component(hub_last):
    import paper_2210_00389_amd as tc

    def ms(leaves):
        G, _ = _rest(2, leaves, hub_last)
        tc.bfs_levels(G, root=0)
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            tc.bfs_levels(G, root=0)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return statistics.median(t)

    print(f"case: stars of 60 and 30000 leaves, hub last {hub_last}", flush=True)
    few, many = ms(60), ms(30000)
    assert many < 10 * few, (few, many)


@pytest.mark.parametrize("pairs", [8191, 8192, 8193, 20000, 32768, 32769])
@pytest.mark.parametrize("tail", [0, 3, 4, 5, 6, 300])
def test_remainders_around_their_bounds(pairs, tail):
    """A clique, disjoint edges, and a path on the last ids, with at most `pairs` edges in all beside the clique."""
    import paper_2210_00389_amd as tc
    print(f"case: {pairs} edges, {tail} of them a path", flush=True)
    k, e = 30, pairs - tail
    i = torch.arange(k, device="cuda")
    a = k + 2 * torch.arange(e, device="cuda")
    p = k + 2 * e + torch.arange(tail, device="cuda")
    n = k + 2 * e + (tail + 1 if tail else 0)
    G = tc.build_csr(n, torch.cat([i.repeat_interleave(k), a, p]).to(torch.int32),
                     torch.cat([i.repeat(k), a + 1, p + 1]).to(torch.int32))
    want = torch.ones(n, dtype=torch.int32, device="cuda")
    want[0], want[a] = 0, 0
    if tail:
        want[p[0]:] = torch.arange(tail + 1, device="cuda", dtype=torch.int32)
    lev, num = tc.bfs_levels(G, root=0)
    assert num == max(2, tail + 1) and torch.equal(lev, want)


def _cliques(sizes):
    """Cliques on consecutive ids: each has its first vertex at level 0, the others at 1."""
    import paper_2210_00389_amd as tc
    size = torch.tensor(sizes, device="cuda")
    first = size.cumsum(0) - size
    i = torch.arange(int(size.sum()), device="cuda")
    own, lo = size.repeat_interleave(size), first.repeat_interleave(size)
    s = i.repeat_interleave(own)
    d = torch.arange(s.numel(), device="cuda") - (own.cumsum(0) - own).repeat_interleave(own) + lo.repeat_interleave(own)
    want = torch.ones(i.numel(), dtype=torch.int32, device="cuda")
    want[first] = 0
    return tc.build_csr(i.numel(), s.to(torch.int32), d.to(torch.int32)), want


@pytest.mark.parametrize("sizes", [[700, 600], [300, 257, 256, 255, 66, 65, 64, 9, 8, 7, 2], [2000, 1999],
                                   [400] + [120] * 200, [200] + [66] * 9000])
def test_dense_remainders(sizes):
    import paper_2210_00389_amd as tc
    print(f"case: cliques of {sizes[:12]} ({len(sizes)})", flush=True)
    G, want = _cliques(sizes)
    lev, num = tc.bfs_levels(G, root=0)
    assert num == 2 and torch.equal(lev, want)


def test_time_of_a_dense_remainder():
    import paper_2210_00389_amd as tc

    def ms(k):
        G, _ = _cliques([700, k])
        tc.bfs_levels(G, root=0)
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            tc.bfs_levels(G, root=0)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return statistics.median(t)

    print("case: cliques of 60 and 600 beside one of 700", flush=True)
    few, many = ms(60), ms(600)
    assert many < 6 * few, (few, many)

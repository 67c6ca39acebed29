"""Workloads whose speed this repository watches, through its public entry points.

Every case is a dict of plain values; `prepare` makes the graph a program
holds before the call (seeded, on the GPU), `run` is one call of the path and
returns its outputs whole, `work` is the traffic that no implementation can
avoid, and `exact` computes the same outputs with plain torch in 64 bits.

Graphs are raw endpoint pairs drawn on the device from the same families as
the benchmark's inputs (R-MAT with quadrants 0.57/0.19/0.19/0.05, Chung-Lu
with exponent 2.1, Erdos-Renyi, Barabasi-Albert), relabelled uniformly, and
turned into CSR by the framework.
"""
import math

import numpy as np
import torch

import paper_2210_00389_amd as tc

DEV = "cuda"
RMAT = (0.57, 0.19, 0.19, 0.05)


def listed():
    return [
        # the smallest count: a latency-bound request on a 1024-vertex graph
        dict(name="count_rmat10", kind="count", family="rmat", scale=10, degree=16),
        # a mid-size power-law request with a ragged vertex count (the small half of a serving pool)
        dict(name="count_cl30k", kind="count", family="chung_lu", n=30011, degree=20),
        # a mid-size skewed graph: short stages, many launches
        dict(name="count_rmat16", kind="count", family="rmat", scale=16, degree=16),
        # a uniform graph: no hubs, few triangles, ragged size
        dict(name="count_er300k", kind="count", family="er", n=300007, degree=24),
        # the ordinary benchmark graph, 16.8 M pairs
        dict(name="count_rmat20", kind="count", family="rmat", scale=20, degree=16),
        # the largest benchmark graph, 268 M pairs
        dict(name="count_rmat24", kind="count", family="rmat", scale=24, degree=16),
        # per-vertex counts and levels (clustering coefficients) of a large power-law graph
        dict(name="vertex_cl500k", kind="vertex", family="chung_lu", n=500009, degree=20),
        # a coalesced batch of a server: some dozens of small graphs
        dict(name="batch_small", kind="batch", graphs=48, n_min=64, n_max=8192),
        # the batched workload: 4096 graphs of 64 to 65536 vertices, half uniform, half preferential
        dict(name="batch_4096", kind="batch", graphs=4096, n_min=64, n_max=65536),
        # triangle finding and the support of every edge (the first step of a k-truss decomposition)
        dict(name="support_rmat16", kind="support", family="rmat", scale=16, degree=16),
        # raw pairs to CSR, what every new graph goes through
        dict(name="build_rmat20", kind="build", family="rmat", scale=20, degree=16),
        # levels and the explicit cover-edge list of a large uniform graph
        dict(name="cover_er1m", kind="cover", family="er", n=1000003, degree=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["count", "count", "count", "vertex", "batch", "support", "build", "cover"])
    if kind == "batch":
        lo = _log_int(rng, 32, 256)
        return dict(kind=kind, graphs=_log_int(rng, 8, 2048), n_min=lo, n_max=_log_int(rng, 16 * lo, 65536))
    family = rng.choice(["rmat", "rmat", "chung_lu", "er"])
    top = {"count": 23, "vertex": 20, "support": 18, "build": 22, "cover": 22}[kind]
    if family == "rmat":
        return dict(kind=kind, family=family, scale=rng.randint(10, top), degree=rng.randint(6, 18))
    return dict(kind=kind, family=family, n=_log_int(rng, 1000, 1 << min(top, 21)) | 1, degree=rng.randint(6, 40))


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)


def _vertices(case):
    return 1 << case["scale"] if case["family"] == "rmat" else case["n"]


def _num_pairs(case):
    # an R-MAT degree is an edge factor (pairs per vertex), the others' a mean degree
    n = _vertices(case)
    return n * case["degree"] if case["family"] == "rmat" else n * case["degree"] // 2


def _chung_lu_cdf(n, degree):
    # w_i ~ (i + i0)^(-1 / 1.1), i0 such that the largest expected degree is sqrt(n * degree)
    idx = torch.arange(n, dtype=torch.float64, device=DEV)
    beta = 1.0 / 1.1
    lo, hi = 1e-3, float(n)
    for _ in range(40):
        mid = math.sqrt(lo * hi)
        top = n * degree * mid ** -beta / float(((idx + mid) ** -beta).sum())
        lo, hi = (mid, hi) if top > math.sqrt(n * degree) else (lo, mid)
    cdf = np.cumsum(((idx + hi) ** -beta).cpu().numpy())  # summed in one order, whatever the device does
    return torch.from_numpy(cdf / cdf[-1]).to(DEV)


def _draw_pairs(case, g, m):
    """m raw int32 pairs before the relabelling (loops, repeats and both orientations may occur)."""
    n = _vertices(case)
    if case["family"] == "rmat":
        a, b, c, _ = RMAT
        s = torch.zeros(m, dtype=torch.int32, device=DEV)
        d = torch.zeros(m, dtype=torch.int32, device=DEV)
        for _ in range(case["scale"]):
            r = torch.rand(m, generator=g, device=DEV)
            s.mul_(2).add_(r >= a + b)
            d.mul_(2).add_(((r >= a) & (r < a + b)) | (r >= a + b + c))
    elif case["family"] == "er":
        s = torch.randint(0, n, (m,), generator=g, device=DEV, dtype=torch.int32)
        d = torch.randint(0, n, (m,), generator=g, device=DEV, dtype=torch.int32)
    else:
        cdf = _chung_lu_cdf(n, case["degree"])
        s, d = (torch.searchsorted(cdf, torch.rand(m, generator=g, device=DEV, dtype=torch.float64)).clamp_(max=n - 1).to(torch.int32)
                for _ in range(2))
    return s, d


def _pairs(case, seed):
    """(n, src, dst): the case's raw pairs.  Where an output has one value per entry (the CSR itself, the
    supports) the graph has exactly _num_pairs edges, some of them listed twice, among a few loops."""
    g, n, m = _gen(seed), _vertices(case), _num_pairs(case)
    s, d = _draw_pairs(case, g, m)
    if case["kind"] in ("build", "support"):
        key = torch.empty(0, dtype=torch.int64, device=DEV)
        while True:
            a, b = torch.minimum(s, d).long(), torch.maximum(s, d).long()
            key = torch.unique(torch.cat([key, (a * n + b)[a < b]]))
            if key.numel() >= m:
                break
            s, d = _draw_pairs(case, g, m)
        key = key[torch.randperm(key.numel(), generator=g, device=DEV)[:m]]
        key = torch.cat([key, key[:m // 16], (key[:m // 64] // n) * (n + 1)])
        s, d = (key // n).to(torch.int32), (key % n).to(torch.int32)
        back = torch.rand(s.numel(), generator=g, device=DEV) < 0.5
        s, d = torch.where(back, d, s), torch.where(back, s, d)
    perm = torch.randperm(n, generator=g, device=DEV, dtype=torch.int32)
    return n, perm[s], perm[d]


def _batch_specs(case):
    """Per graph: vertices, pairs, and the preferential half's pairs per vertex (0: uniform)."""
    G = case["graphs"]
    q = (np.random.RandomState(20 + G).permutation(G) + 0.5) / G  # sizes spread over the logarithm
    n = np.floor(np.exp(np.log(case["n_min"]) + q * np.log(case["n_max"] / case["n_min"]))).astype(np.int64)
    u = (np.random.RandomState(21 + G).permutation(G) + 0.5) / G
    ba = np.arange(G) >= G // 2
    per = np.where(ba, 2 + np.floor(15 * u), 0).astype(np.int64)
    pairs = np.where(ba, n * per, np.minimum((n * (8 + 56 * u) / 2).astype(np.int64), n * (n - 1) // 2))
    return n, pairs, per


def _batch_pairs(case, seed):
    """(vbase, src, dst): the pairs of every graph, ids shifted by its base."""
    g = _gen(seed)
    n, pairs, per = _batch_specs(case)
    vb = np.concatenate([[0], np.cumsum(n)])
    G, half = len(n), len(n) // 2
    out_s, out_d = [], []
    for lo, hi in ((0, half), (half, G)):
        if hi == lo:
            continue
        reps = torch.from_numpy(pairs[lo:hi]).to(DEV)
        rep = lambda x: torch.repeat_interleave(torch.from_numpy(x[lo:hi].copy()).to(DEV), reps)  # noqa: E731
        m = int(pairs[lo:hi].sum())
        base = rep(vb[:-1])
        if lo == 0:  # uniform pairs
            ng = rep(n).to(torch.float64)
            s, d = ((torch.rand(m, generator=g, device=DEV, dtype=torch.float64) * ng).long() for _ in range(2))
        else:  # preferential: pair k of a graph joins vertex k // per to the vertex of a uniform earlier slot
            first = np.concatenate([[0], np.cumsum(pairs[lo:hi])])[:-1]
            start = torch.repeat_interleave(torch.from_numpy(first).to(DEV), reps)
            k = torch.arange(m, device=DEV) - start
            p = rep(per)
            t = (torch.rand(m, generator=g, device=DEV, dtype=torch.float64) * (2 * k + 1)).long()
            while bool((t & 1).any()):  # an odd slot is the far end of an earlier pair
                t = torch.where((t & 1) > 0, t[start + (t >> 1)], t)
            s, d = k // p, (t >> 1) // p
            del k, p, t, start
        out_s.append((s + base).to(torch.int32))
        out_d.append((d + base).to(torch.int32))
        del s, d, base
    return vb, torch.cat(out_s), torch.cat(out_d)


def prepare(case, seed):
    if case["kind"] == "batch":
        vb, s, d = _batch_pairs(case, seed)
        u = tc.build_csr(int(vb[-1]), s, d)
        del s, d
        n = torch.from_numpy(np.diff(vb)).to(DEV)
        vbase = torch.from_numpy(vb).to(DEV)
        base = torch.repeat_interleave(vbase[:-1].to(torch.int32), n)
        cols = u.cols - torch.repeat_interleave(base, u.row_offsets[1:] - u.row_offsets[:-1])
        nnz = np.diff(u.row_offsets[vbase].cpu().numpy())
        return dict(kind="batch", batch=tc.Batch(vbase, u.row_offsets, cols, list(zip(np.diff(vb).tolist(), nnz.tolist()))))
    n, s, d = _pairs(case, seed)
    if case["kind"] == "build":
        return dict(kind="build", n=n, src=s, dst=d)
    g = tc.build_csr(n, s, d)
    state = dict(kind=case["kind"], graph=tc.Graph(n, g.row_offsets, g.cols.clone()))
    if case["kind"] == "cover":  # the program's own edge buffer, as long as the list can get
        state["edges"] = torch.full((2, _num_pairs(case)), -1, dtype=torch.int32, device=DEV)
    return state


def run(state):
    kind = state["kind"]
    if kind == "count":
        r = tc.count(state["graph"])
        return r.triangles, r.h_count
    if kind == "vertex":
        r = tc.count(state["graph"], per_vertex=True, return_levels=True)
        return r.triangles, r.h_count, r.per_vertex, r.levels
    if kind == "batch":
        r = tc.count_batch(state["batch"])
        return r.triangles, r.h_count
    if kind == "support":
        r = tc.list_triangles(state["graph"])
        return r.triangles, r.h_count, tc.edge_support(state["graph"], r.tri)
    if kind == "build":
        g = tc.build_csr(state["n"], state["src"], state["dst"])
        return g.row_offsets, g.cols
    levels, num = tc.bfs_levels(state["graph"])
    hu, hv = tc.cover_edges(state["graph"], levels)
    state["edges"][0, :hu.numel()] = hu
    state["edges"][1, :hv.numel()] = hv
    return levels, num, state["edges"]


def work(case):
    """Input CSR (or pairs) read once and outputs written once; no floating point.
    Entries are taken as twice the pairs, of which repeats take a few per cent (none where the edges are exact)."""
    if case["kind"] == "batch":
        n, pairs, _ = _batch_specs(case)
        return dict(bytes=float(8 * (n.sum() + 1) + 8 * pairs.sum() + 16 * len(n)), flops=0.0)
    n, nnz = _vertices(case), 2 * _num_pairs(case)
    csr = 8 * (n + 1) + 4 * nnz
    extra = dict(count=16, vertex=16 + 12 * n, support=16 + 4 * nnz, build=4 * nnz + nnz // 4, cover=4 * n + 2 * nnz)[case["kind"]]
    return dict(bytes=float(csr + extra), flops=0.0)


# ------------------------------------------------------------------- exact
def _simple(n, s, d):
    """Both orientations of the simple graph, sorted: (u, v) as int64."""
    s, d = s.long(), d.long()
    keep = s != d
    s, d = s[keep], d[keep]
    key = torch.unique(torch.cat([s * n + d, d * n + s]))
    return key // n, key % n


def _levels(n, u, v, vb):
    """Levels from every graph's largest-degree vertex, then its other components from their smallest ids."""
    deg = torch.bincount(u, minlength=n)
    lab = torch.arange(n, device=DEV)
    while True:
        new = lab.scatter_reduce(0, u, lab[v], "amin")
        new = new[new]
        if torch.equal(new, lab):
            break
        lab = new
    first = lab == torch.arange(n, device=DEV)
    for a, b in zip(vb[:-1], vb[1:]):
        if b > a:
            r = int(a) + int((deg[a:b] * (b - a) + torch.arange(b - a, 0, -1, device=DEV) - 1).argmax())
            first[lab[r]] = False
            first[r] = True
    lev = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    lev[first] = 0
    at = 0
    while True:
        hit = (lev[u] == at) & (lev[v] < 0)
        if not bool(hit.any()):
            return lev, at + 1
        at += 1
        lev[v[hit]] = at


def _triangles(n, u, v, each):
    """Calls each(a, b, c) with blocks of triangles, every triangle once (ids ordered by degree)."""
    deg = torch.bincount(u, minlength=n)
    up = (deg[u] < deg[v]) | ((deg[u] == deg[v]) & (u < v))
    a, b = u[up], v[up]
    key = a * n + b
    cnt = torch.bincount(a, minlength=n)
    off = torch.cumsum(cnt, 0) - cnt
    todo = torch.cumsum(cnt[b], 0)
    total, lo, step = int(todo[-1]) if todo.numel() else 0, 0, 1 << 27
    while lo < a.numel():
        before = int(todo[lo - 1]) if lo else 0
        hi = max(lo + 1, int(torch.searchsorted(todo, before + step)))
        c = cnt[b[lo:hi]]
        e = torch.repeat_interleave(torch.arange(lo, hi, device=DEV), c)
        w = b[off[b[e]] + torch.arange(e.numel(), device=DEV) - (todo[e] - cnt[b[e]] - before)]
        want = a[e] * n + w
        pos = torch.searchsorted(key, want).clamp_(max=key.numel() - 1)
        hit = key[pos] == want
        each(a[e[hit]], b[e[hit]], w[hit])
        lo = hi
    return total


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        if _batch_specs(case)[1].sum() > 1 << 25 or case["graphs"] > 512:
            return None
        vb, s, d = _batch_pairs(case, seed)
        n = int(vb[-1])
    else:
        if _num_pairs(case) > (1 << 26 if kind in ("build", "cover") else 1 << 22):
            return None
        n, s, d = _pairs(case, seed)
        vb = np.array([0, n])
    u, v = _simple(n, s, d)
    if kind == "build":
        deg = torch.bincount(u, minlength=n)
        return torch.cat([deg.new_zeros(1), torch.cumsum(deg, 0)]), v.to(torch.int32)
    lev, num = _levels(n, u, v, vb)
    h = (lev[u] == lev[v]) & (u < v)
    if kind == "cover":
        edges = torch.full((2, _num_pairs(case)), -1, dtype=torch.int32, device=DEV)
        edges[0, :int(h.sum())] = u[h].to(torch.int32)
        edges[1, :int(h.sum())] = v[h].to(torch.int32)
        return lev.to(torch.int32), num, edges
    G = len(vb) - 1
    graph_of = torch.repeat_interleave(torch.arange(G, device=DEV), torch.from_numpy(np.diff(vb)).to(DEV))
    hc = torch.bincount(graph_of[u[h]], minlength=G)
    T = torch.zeros(G, dtype=torch.int64, device=DEV)
    pv = torch.zeros(n, dtype=torch.int64, device=DEV)
    sup = torch.zeros(u.numel(), dtype=torch.int64, device=DEV)
    key = u * n + v

    def each(a, b, c):
        T.add_(torch.bincount(graph_of[a], minlength=G))
        if kind == "vertex":
            for x in (a, b, c):
                pv.add_(torch.bincount(x, minlength=n))
        if kind == "support":
            for x, y in ((a, b), (a, c), (b, c)):
                for p, q in ((x, y), (y, x)):
                    sup.add_(torch.bincount(torch.searchsorted(key, p * n + q), minlength=sup.numel()))

    _triangles(n, u, v, each)
    if kind == "vertex":
        return T, hc, pv, lev.to(torch.int32)
    if kind == "support":
        return T, hc, sup.to(torch.int32)
    return T, hc

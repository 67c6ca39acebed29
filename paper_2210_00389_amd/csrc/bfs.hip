// bfs.hip -- BFS levels L(v) of Def. 2 with the root rule of Alg. 1:
// a BFS from r0 (given, or the largest-degree vertex with the smallest id on
// ties), then every component not reached is levelled from its smallest id.
//
// GPU structure (frontiers are bitmaps; three rotate so that the bitmap of
// the level after next is cleared while the current one is read):
//   * one launch per level.  Every block sums the previous level's counts
//     (kSlots partial sums) and decides the direction and the stop for
//     itself; block 0 writes the decision for the next launch;
//   * a top-down step lets every frontier vertex expand its row; a vertex
//     with more than kBig entries was listed when it was found, and listed
//     rows are expanded edge-balanced (flat entry index over the rows, so a
//     hub's row is spread over the whole grid); new vertices are claimed
//     with an atomic OR on the visited bitmap;
//   * a bottom-up step (Beamer et al.'s direction optimisation) lets every
//     unvisited vertex look for a neighbour in the frontier and stop at the
//     first hit; a wave composes its 64 vertices' bits with ballots;
//   * after a group of levels two kernels, which do nothing unless the search
//     has ended, level the isolated vertices and list the other unreached
//     ones, and level those in one block if they are few vertices of few
//     entries; the state goes to the host once per group, usually once in all;
//   * otherwise the remaining components: union-find over the unreached vertices where
//     a root is always hooked under the smaller root, so every component's
//     final root is its smallest id; those roots then start one multi-source
//     BFS (components are disjoint, so the per-component distances are
//     exactly those of separate BFS runs), whose levels after the first group
//     are one block's where all its entries are few.
#include "tc_internal.h"

namespace tc {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ int64_t row_deg(const int64_t* off, int64_t v) { return off[v + 1] - off[v]; }

// frontier rows above this length are expanded edge-balanced over the grid
// (a row below it is expanded by one wave: R-MAT S14's root, 3644 entries,
// took 0.12 ms that way under a bound of 4096, against 5 us listed)
constexpr int kBig = 1024;
// Listed rows per level (more: all expanded by their waves), and how many of
// them a block's prefix of lengths holds at once.  With room for 1024 only, a
// level of 1500 rows of 1100 entries and one of 2 M left the long one to a
// wave: 88 ms for the search, 0.7 ms with all of them listed.
constexpr int kBigCap = 65536;
constexpr int kBigPart = 1024;
constexpr int kRowLoads = 8;       // row entries a bottom-up scan loads at once
constexpr int kSlots = 16;         // partial sums of a level: one atomic per block, spread over them
constexpr int kKeyBlocks = 1024;   // blocks of the first kernel at most (one key each)
// Levels launched before the state is read: six covers a small-world graph
// searched from a hub (R-MAT S10-S20 take 5-6, a uniform graph of 10^6
// vertices 8); after a second group of four, a deeper graph doubles it each
// time (levels past the stop cost a no-op launch each).
constexpr int kFirstLevels = 6;
constexpr int kNextLevels = 4;     // also the first group of the remaining components, usually shallow
constexpr int kMaxLevels = 64;
// Up to kRestNow unreached vertices of at most kRestEntries entries are levelled
// by one block (R-MAT scale 16: a few dozen vertices in components of two and
// three).  With more vertices the grid finds the components and takes their
// first levels, and one block goes on from there.  us, one block from the
// start / so: 4000 disjoint edges 43 / 90, 10000 113 / 60, 30000 392 / 70; a
// path of 20000 vertices 26000 either way, 110000 with a launch a level.
constexpr int64_t kRestNow = 16384;
constexpr int64_t kRestEntries = 65536;
constexpr int kRestThreads = 1024;
// There, rows above this length are expanded by the whole block: with every row
// by a thread of its own, a star of 30000 leaves took 23.6 ms, 55 ms where the
// hub has the largest id.
constexpr int kRestRow = 64;

// State before a level's step.
struct BfsState {
  int64_t unexplored;    // row entries not yet in any frontier
  int32_t bottom_up;     // direction of the step
  int32_t done;          // the frontier is empty
  int32_t num_levels;    // levels so far (final once done)
  int32_t pad;
};

// Device-side bookkeeping of a BFS (BfsWs::st).
struct BfsDev {
  BfsState state[2];                    // of step k at [k & 1]
  unsigned long long acc[3][kSlots][2]; // per level: new vertices and their entries, at [k % 3]
  int32_t nbig[3];                      // rows listed for step k, at [k % 3]
  int32_t rest_n;                       // listed unreached vertices
  int32_t rest_long;                    // a row of theirs is longer than kRestRow
  int64_t maxdeg;
  unsigned long long deg2;              // sum of squared degrees
};

// What the host reads.
struct BfsHost {
  int64_t unexplored, maxdeg;
  unsigned long long deg2;
  int32_t done, num_levels;
  int32_t rest_levels;  // level count of the remaining components (-1: left to the grid)
  int32_t pad;
};

__device__ __forceinline__ uint32_t* bm_at(uint32_t* base, int64_t words, int k, int j) {
  return base + static_cast<int64_t>((k + j) % 3) * words;
}

__device__ __forceinline__ bool goes_up(int64_t cnt, int64_t edg, int64_t unexplored, int64_t n) {
  return edg > unexplored / 14 && cnt > n / 256;  // Beamer's rule, alpha = 14
}

// The state of step k from that of step k - 1 and its counts (any whole wave).
__device__ __forceinline__ BfsState state_of(const BfsDev* d, int k, int64_t n) {
  if (k == 0) return d->state[0];
  BfsState s = d->state[(k - 1) & 1];
  if (s.done) return s;
  const unsigned long long(*a)[2] = d->acc[(k - 1) % 3];
  const int64_t cnt = wave_sum(static_cast<int64_t>(lane() < kSlots ? a[lane()][0] : 0ull));
  const int64_t edg = wave_sum(static_cast<int64_t>(lane() < kSlots ? a[lane()][1] : 0ull));
  if (cnt == 0) {
    s.done = 1;
    s.num_levels = k;
    return s;
  }
  s.num_levels = k + 1;
  s.unexplored -= edg;
  s.bottom_up = !s.bottom_up ? goes_up(cnt, edg, s.unexplored, n) : (cnt >= n / 24);  // beta = 24
  return s;
}

// Adds a block's counts to the level's slots.
__device__ __forceinline__ void add_counts(unsigned long long (*a)[2], int64_t cnt, int64_t edg, int64_t* sh) {
  cnt = block_sum(cnt, sh);
  edg = block_sum(edg, sh);
  if (threadIdx.x == 0 && cnt) {
    atomicAdd(&a[blockIdx.x % kSlots][0], static_cast<unsigned long long>(cnt));
    atomicAdd(&a[blockIdx.x % kSlots][1], static_cast<unsigned long long>(edg));
  }
}

// A found vertex with a long row is listed for the next step (past the
// capacity the list is not used, so nothing more is appended then).
__device__ __forceinline__ void list_big(int32_t* nbig, int32_t* big, int32_t v, int64_t deg) {
  if (deg <= kBig || load_relaxed(nbig) > kBigCap) return;
  const int q = atomicAdd(nbig, 1);
  if (q < kBigCap) big[q] = v;
}

// The long rows a block finds, appended together: one addition to the counter
// a row took 0.17 ms at R-MAT scale 24.
struct BigLds {
  int n, at;
  int32_t row[kBigPart];
};
__device__ __forceinline__ void list_big(BigLds& s, int32_t* nbig, int32_t* big, int32_t v, int64_t deg) {
  if (deg <= kBig) return;
  const int q = atomicAdd(&s.n, 1);
  if (q < kBigPart) s.row[q] = v;
  else list_big(nbig, big, v, deg);
}
// All threads, after a barrier behind the last row.
__device__ __forceinline__ void flush_big(BigLds& s, int32_t* nbig, int32_t* big) {
  const int n = min(s.n, kBigPart);
  if (n == 0) return;  // uniform
  if (threadIdx.x == 0) s.at = atomicAdd(nbig, n);
  __syncthreads();
  for (int i = threadIdx.x; i < n && s.at + i < kBigCap; i += blockDim.x) big[s.at + i] = s.row[i];
}

// Step k of a BFS: level k's frontier finds level k + 1.
__global__ __launch_bounds__(kThreads) void step_kernel(const int64_t* off, const int32_t* cols, int64_t n, int k,
                                                        BfsDev* d, int32_t* L, uint32_t* vis, uint32_t* bms,
                                                        int32_t* bigs) {
  __shared__ int64_t sh[kThreads / kWave + 1];
  __shared__ int32_t s_off[kThreads / kWave][kWave + 1];
  __shared__ int64_t s_beg[kThreads / kWave][kWave];
  __shared__ int64_t s_pre[kBigPart + 1];
  __shared__ BigLds s_found;
  const BfsState st = state_of(d, k, n);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      d->state[k & 1] = st;
      d->nbig[(k + 2) % 3] = 0;
    }
    if (threadIdx.x < 2 * kSlots) (&d->acc[(k + 1) % 3][0][0])[threadIdx.x] = 0ull;
  }
  if (st.done) return;
  if (threadIdx.x == 0) s_found.n = 0;
  __syncthreads();
  const int64_t words = (n + 31) / 32 + 1;
  int64_t cnt = 0, edg = 0;
  const uint32_t* cur = bm_at(bms, words, k, 0);
  uint32_t* nxt = bm_at(bms, words, k, 1);
  uint32_t* old = bm_at(bms, words, k, 2);
  int32_t* nbig = &d->nbig[(k + 1) % 3];
  int32_t* big = bigs + ((k + 1) & 1) * kBigCap;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (int64_t i = t0; i < words; i += stride) old[i] = 0u;  // the bitmap of the level after next
  const int32_t nl = k + 1;
  if (st.bottom_up) {
    // 64 consecutive vertices per wave and round: words 2k, 2k+1 are this wave's
    for (int64_t v0 = (t0 / kWave) * kWave; v0 < n; v0 += stride) {
      const int64_t v = v0 + lane();
      bool take = false;
      if (v < n && !((vis[v >> 5] >> (v & 31)) & 1u)) {
        const int64_t b = off[v], e = off[v + 1];
        for (int64_t j = b; j < e && !take; j += kRowLoads) {  // independent loads in flight
          int32_t w[kRowLoads];
#pragma unroll
          for (int q = 0; q < kRowLoads; ++q) w[q] = j + q < e ? cols[j + q] : -1;
          uint32_t f[kRowLoads];
#pragma unroll
          for (int q = 0; q < kRowLoads; ++q) f[q] = w[q] >= 0 ? cur[w[q] >> 5] >> (w[q] & 31) : 0u;
#pragma unroll
          for (int q = 0; q < kRowLoads; ++q) take |= (f[q] & 1u) != 0u;
        }
        if (take) {
          L[v] = nl;
          ++cnt;
          edg += e - b;
          list_big(s_found, nbig, big, static_cast<int32_t>(v), e - b);
        }
      }
      const uint64_t m = __ballot(take);
      if (m && (lane() & 31) == 0) {
        const uint32_t word = static_cast<uint32_t>(m >> lane());
        if (word) {
          nxt[v >> 5] |= word;
          vis[v >> 5] |= word;
        }
      }
    }
  } else {
    auto claim = [&](int32_t w) {
      const uint32_t bit = 1u << (w & 31);
      if (load_relaxed(&vis[w >> 5]) & bit) return;
      if (atomicOr(&vis[w >> 5], bit) & bit) return;
      atomicOr(&nxt[w >> 5], bit);
      L[w] = nl;
      const int64_t deg = off[w + 1] - off[w];
      ++cnt;
      edg += deg;
      list_big(s_found, nbig, big, w, deg);
    };
    // the listed rows of this frontier, kBigPart at a time, by a flat entry
    // index (each block computes the prefix of their lengths)
    const int nb = d->nbig[k % 3];
    const bool listed = nb <= kBigCap;
    for (int p0 = 0; listed && p0 < nb; p0 += kBigPart) {
      const int32_t* mine = bigs + (k & 1) * kBigCap + p0;
      const int np = min(nb - p0, kBigPart);
      int64_t run = 0;
      for (int b0 = 0; b0 < np; b0 += kThreads) {
        const int i = b0 + threadIdx.x;
        const int64_t dg = i < np ? off[mine[i] + 1] - off[mine[i]] : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan(dg, sh, &tot);
        if (i < np) s_pre[i] = run + ex;
        run += tot;
      }
      if (threadIdx.x == 0) s_pre[np] = run;
      __syncthreads();
      for (int64_t i = t0; i < run; i += stride) {
        int lo = 0, hi = np;  // last row with s_pre <= i
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (s_pre[mid] <= i) lo = mid;
          else hi = mid;
        }
        claim(cols[off[mine[lo]] + (i - s_pre[lo])]);
      }
      __syncthreads();  // the next part's prefix replaces this one's
    }
    // 64 consecutive vertices per wave and round; the rows of the group's
    // frontier vertices are flattened across the lanes
    const int wv = threadIdx.x / kWave;
    for (int64_t v0 = (t0 / kWave) * kWave; v0 < n; v0 += stride) {
      const uint64_t fw = static_cast<uint64_t>(cur[v0 >> 5]) | (static_cast<uint64_t>(cur[(v0 >> 5) + 1]) << 32);
      if (fw == 0) continue;  // uniform per wave
      const int64_t v = v0 + lane();
      int64_t b = 0;
      int dg = 0;
      if (((fw >> lane()) & 1ull) && v < n) {
        b = off[v];
        const int64_t e = off[v + 1];
        if (!(listed && e - b > kBig)) dg = static_cast<int>(e - b);
      }
      const int incl = wave_incl_scan(dg);
      const int total = wave_read(incl, kWave - 1);
      s_off[wv][lane()] = incl - dg;
      s_beg[wv][lane()] = b;
      if (lane() == 0) s_off[wv][kWave] = total;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      for (int i = lane(); i < total; i += kWave) {
        int lo = 0, hi = kWave;  // last j with s_off[j] <= i
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (s_off[wv][mid] <= i) lo = mid;
          else hi = mid;
        }
        claim(cols[s_beg[wv][lo] + (i - s_off[wv][lo])]);
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
  }
  add_counts(d->acc[k % 3], cnt, edg, sh);
  flush_big(s_found, nbig, big);
}

// Clears the state of a BFS in one launch (levels to -1, the visited and
// frontier bitmaps) and takes each block's largest (degree, smallest id) and
// its sum of squared degrees.
__global__ __launch_bounds__(kThreads) void clear_state_kernel(const int64_t* off, int32_t* L, int64_t n,
                                                               uint32_t* vis, int64_t words, uint32_t* bms,
                                                               unsigned long long* keys) {
  __shared__ unsigned long long sh[kThreads / kWave + 1];
  unsigned long long best = 0, d2 = 0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n || i < 3 * words;
       i += (int64_t)gridDim.x * blockDim.x) {
    if (i < n) {
      L[i] = -1;
      const unsigned long long dg = static_cast<unsigned long long>(row_deg(off, i));
      // larger degree first, then smaller id
      const unsigned long long key = (dg << 32) | (0xFFFFFFFFull - static_cast<unsigned long long>(i));
      best = key > best ? key : best;
      d2 += dg * dg;
    }
    if (i < words) vis[i] = 0u;
    if (i < 3 * words) bms[i] = 0u;
  }
  best = wave_max(best);
  if (lane() == 0) sh[threadIdx.x / kWave] = best;
  __syncthreads();
  best = wave_max(lane() < kThreads / kWave ? sh[lane()] : 0ull);
  __syncthreads();
  d2 = block_sum(d2, sh);
  if (threadIdx.x == 0) {
    keys[2 * blockIdx.x] = best;
    keys[2 * blockIdx.x + 1] = d2;
  }
}

// Starts the BFS from one root (the largest key, or a given root).
__global__ __launch_bounds__(kKeyBlocks) void start_kernel(const int64_t* off, int64_t n, int64_t nnz,
                                                           const unsigned long long* keys, int nkeys,
                                                           int64_t given_root, BfsDev* d, int32_t* L, uint32_t* vis,
                                                           uint32_t* bm0, int32_t* bigs) {
  __shared__ unsigned long long sh[kKeyBlocks / kWave + 1];
  const int t = threadIdx.x;
  unsigned long long best = t < nkeys ? keys[2 * t] : 0ull, d2 = t < nkeys ? keys[2 * t + 1] : 0ull;
  best = wave_max(best);
  if (lane() == 0) sh[t / kWave] = best;
  __syncthreads();
  best = wave_max(lane() < kKeyBlocks / kWave ? sh[lane()] : 0ull);
  __syncthreads();
  d2 = block_sum(d2, sh);
  if (t < 3 * kSlots * 2) (&d->acc[0][0][0])[t] = 0ull;
  if (t != 0) return;
  const int64_t r = given_root < 0 ? static_cast<int64_t>(0xFFFFFFFFull - (best & 0xFFFFFFFFull)) : given_root;
  const int64_t dg = row_deg(off, r);
  L[r] = 0;
  vis[r >> 5] = 1u << (r & 31);
  bm0[r >> 5] = 1u << (r & 31);
  d->nbig[0] = dg > kBig;
  d->nbig[1] = d->nbig[2] = 0;
  if (dg > kBig) bigs[0] = static_cast<int32_t>(r);
  d->rest_n = d->rest_long = 0;
  d->maxdeg = static_cast<int64_t>(best >> 32);
  d->deg2 = d2;
  d->state[0] = BfsState{nnz - dg, goes_up(1, dg, nnz - dg, n), 0, 1, 0};
}

// ------------------------------------------------- remaining components
// Once the search from r0 has ended (else nothing is done): its component is
// kept for the relabelling (comp0, nullable), an isolated vertex's own
// one-vertex BFS gives it level 0, and the other unreached vertices, if
// their rows are few entries, are listed for rest_kernel.
__global__ __launch_bounds__(kThreads) void unreached_kernel(const int64_t* off, int64_t n, int k, BfsDev* d,
                                                             const uint32_t* vis, int32_t* L, uint32_t* comp0,
                                                             int64_t words, int32_t* parent, int32_t* list) {
  const BfsState st = state_of(d, k, n);
  if (!st.done) return;
  const bool few = st.unexplored <= kRestEntries;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (comp0)
    for (int64_t i = t0; i < words; i += stride) comp0[i] = vis[i];
  for (int64_t v0 = t0 - lane(); v0 < n; v0 += stride) {  // the whole wave takes part
    const int64_t v = v0 + lane();
    const bool out = v < n && !((vis[v >> 5] >> (v & 31)) & 1u);
    const bool lone = out && (st.unexplored == 0 || row_deg(off, v) == 0);
    if (lone) L[v] = 0;
    const bool take = few && out && !lone;
    const uint64_t m = __ballot(take);
    if (m == 0) continue;  // uniform
    // one addition a wave; past kRestNow they are left to the grid
    int at = 0;
    if (lane() == 0) at = atomicAdd(&d->rest_n, __popcll(m));
    const int q = wave_read(at, 0) + __popcll(m & lanemask_lt());
    if (!take) continue;
    parent[v] = static_cast<int32_t>(v);
    if (q < kRestNow) list[q] = static_cast<int32_t>(v);
  }
}

__device__ __forceinline__ int32_t uf_find(int32_t* parent, int32_t x) {
  for (;;) {
    int32_t p = load_relaxed(&parent[x]);
    if (p == x) return x;
    int32_t gp = load_relaxed(&parent[p]);
    if (gp != p) __hip_atomic_store(&parent[x], gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    x = p;
  }
}

// Hooks the larger root under the smaller, so parent[x] <= x always holds
// and the root of a finished component is its smallest vertex.
__device__ __forceinline__ void uf_union(int32_t* parent, int32_t a, int32_t b) {
  for (;;) {
    a = uf_find(parent, a);
    b = uf_find(parent, b);
    if (a == b) return;
    if (a > b) {
      int32_t t = a;
      a = b;
      b = t;
    }
    int32_t old = atomicCAS(&parent[b], b, a);
    if (old == b) return;
    b = old;  // b was hooked meanwhile: retry from its new parent
  }
}

template <int THREADS>
struct RestLds {
  int len[2], nlong;
  int32_t row[THREADS];  // rows longer than kRestRow
  int64_t pre[THREADS];  // entries of those before
  int64_t sh[THREADS / kWave + 1];
};

// f(v, w) for every entry w of the rows of v = vertex(i), 0 <= i < m (negative:
// none; !kLong: no row is longer than kRestRow), twice for the first of a long
// row: before the block shares it, so that the threads joining its entries find
// its vertex in a tree by then (a clique of 2000 beside a star of 200000 leaves:
// 1.34 ms without that and the look at the parents in uf_hook_kernel, 0.78 so).  All threads of the block; the
// caller has cleared s.nlong and synchronised it, and it is synchronised on
// return.
template <int THREADS, bool kLong, class V, class F>
__device__ __forceinline__ void each_entry(RestLds<THREADS>& s, const int64_t* off, const int32_t* cols, int m,
                                           V vertex, F f) {
  const int tid = threadIdx.x;
  for (int i = tid; i < m; i += THREADS) {
    const int32_t x = vertex(i);
    if (x < 0) continue;
    const int64_t b = off[x], e = off[x + 1];
    if (kLong && e - b > kRestRow) {
      const int q = atomicAdd(&s.nlong, 1);
      if (q < THREADS) {
        s.row[q] = x;
        f(x, cols[b]);
        continue;
      }
    }
    for (int64_t j = b; j < e; ++j) f(x, cols[j]);
  }
  __syncthreads();
  const int nl = kLong ? min(s.nlong, THREADS) : 0;
  if (nl == 0) return;  // uniform
  int64_t total;
  s.pre[tid] = block_excl_scan(tid < nl ? row_deg(off, s.row[tid]) : int64_t(0), s.sh, &total);
  __syncthreads();
  for (int64_t i = tid; i < total; i += THREADS) {
    int lo = 0, hi = nl;  // last row with pre <= i
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s.pre[mid] <= i) lo = mid;
      else hi = mid;
    }
    const int32_t x = s.row[lo];
    f(x, cols[off[x] + (i - s.pre[lo])]);
  }
  __syncthreads();
}

// The levels after `level`, whose s.len[0] vertices are in the first queue (two
// of kRestEntries vertices; a vertex is claimed once), by one block that has
// cleared s.len[1] and s.nlong.  Returns the level count.
template <bool kLong>
__device__ __forceinline__ int finish_levels(RestLds<kRestThreads>& s, const int64_t* off, const int32_t* cols,
                                             int32_t* L, int32_t* queues, int level) {
  int at = 0;
  for (int len = min(s.len[0], static_cast<int>(kRestEntries)); len > 0; at ^= 1) {
    const int32_t* cur = queues + at * kRestEntries;
    int32_t* nxt = queues + (at ^ 1) * kRestEntries;
    int* n = &s.len[at ^ 1];
    ++level;
    each_entry<kRestThreads, kLong>(s, off, cols, len, [&](int i) { return cur[i]; }, [&](int32_t, int32_t w) {
      if (load_relaxed(&L[w]) < 0 && atomicCAS(&L[w], -1, level) == -1) {
        const int q = atomicAdd(n, 1);
        if (q < kRestEntries) nxt[q] = w;
      }
    });
    len = min(*n, static_cast<int>(kRestEntries));
    if (threadIdx.x == 0) s.len[at] = s.nlong = 0;  // the queue just read
    __syncthreads();
  }
  return level;
}

// Levels the listed vertices (one block), and writes the state for the host.
// A neighbour without a level is itself listed.
__global__ __launch_bounds__(kRestThreads) void rest_kernel(const int64_t* off, const int32_t* cols, int64_t n, int k,
                                                            BfsDev* d, int32_t* L, int32_t* parent,
                                                            int32_t* list, BfsHost* out) {
  __shared__ RestLds<kRestThreads> s;
  const BfsState st = state_of(d, k, n);
  const int m = d->rest_n;
  int levels = 0;
  if (st.done && (st.unexplored > kRestEntries || m > kRestNow)) {
    levels = -1;
  } else if (st.done && st.unexplored > 0) {
    if (threadIdx.x == 0) s.len[0] = s.len[1] = s.nlong = 0;
    __syncthreads();
    each_entry<kRestThreads, true>(s, off, cols, m, [&](int i) { return list[i]; }, [&](int32_t v, int32_t w) {
      if (w < v && L[w] < 0) uf_union(parent, v, w);
    });
    const bool lng = s.nlong > 0;
    int32_t* queues = list + kRestEntries;
    for (int i = threadIdx.x; i < m; i += kRestThreads) {
      const int32_t v = list[i];
      if (uf_find(parent, v) != v) continue;
      L[v] = 0;
      queues[atomicAdd(&s.len[0], 1)] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) s.nlong = 0;
    __syncthreads();
    levels = lng ? finish_levels<true>(s, off, cols, L, queues, 0) : finish_levels<false>(s, off, cols, L, queues, 0);
  }
  if (threadIdx.x == 0)
    *out = BfsHost{st.unexplored, d->maxdeg, d->deg2, st.done, st.num_levels, levels, 0};
}

// The rest of the levels of the remaining components after their step k - 1,
// in one block (their rows are at most kRestEntries entries), and the state
// for the host.
__global__ __launch_bounds__(kRestThreads) void rest_tail_kernel(const int64_t* off, const int32_t* cols, int64_t n,
                                                                 int k, const BfsDev* d, int32_t* L,
                                                                 const uint32_t* bms, int32_t* queues, BfsHost* out) {
  __shared__ RestLds<kRestThreads> s;
  const BfsState st = state_of(d, k, n);
  int levels = st.num_levels;
  if (!st.done) {
    const int64_t words = (n + 31) / 32 + 1;
    const uint32_t* cur = bms + static_cast<int64_t>(k % 3) * words;
    if (threadIdx.x == 0) s.len[0] = s.len[1] = s.nlong = 0;
    __syncthreads();
    for (int64_t i = threadIdx.x; i < words; i += kRestThreads)
      for (uint32_t b = cur[i]; b; b &= b - 1) {
        const int q = atomicAdd(&s.len[0], 1);
        if (q < kRestEntries) queues[q] = static_cast<int32_t>(32 * i + __ffs(static_cast<int>(b)) - 1);
      }
    __syncthreads();
    levels = d->rest_long ? finish_levels<true>(s, off, cols, L, queues, k)
                          : finish_levels<false>(s, off, cols, L, queues, k);
  }
  if (threadIdx.x == 0) *out = BfsHost{0, d->maxdeg, d->deg2, 1, levels, 0, 0};
}

__global__ void uf_init_kernel(int32_t* parent, int64_t n) {
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x)
    parent[v] = static_cast<int32_t>(v);
}

// Vertices a block takes at a time (at most kThreads): fewer where the vertices
// are, as a block shares its long rows among its threads only.  With kThreads a
// clique of 600 vertices was three blocks' work: 1.09 ms for the search beside
// one of 700, 0.30 so (524033 vertices and more: kThreads either way).
__host__ __device__ inline int hook_chunk(int64_t n) {
  const int64_t c = (n + 2047) / 2048;
  return c < 8 ? 8 : c < kThreads ? static_cast<int>(c) : kThreads;
}

__global__ __launch_bounds__(kThreads) void uf_hook_kernel(const int64_t* off, const int32_t* cols, int64_t n,
                                                           const uint32_t* vis, int32_t* parent, BfsDev* d) {
  __shared__ RestLds<kThreads> s;
  const int chunk = hook_chunk(n);
  for (int64_t v0 = blockIdx.x * (int64_t)chunk; v0 < n; v0 += (int64_t)gridDim.x * chunk) {
    if (threadIdx.x == 0) s.nlong = 0;
    __syncthreads();
    each_entry<kThreads, true>(
        s, off, cols, chunk,
        [&](int i) {
          const int64_t v = v0 + i;
          return v < n && !((vis[v >> 5] >> (v & 31)) & 1u) ? static_cast<int32_t>(v) : -1;
        },
        [&](int32_t v, int32_t w) {
          if (w < v && load_relaxed(&parent[w]) != load_relaxed(&parent[v])) uf_union(parent, v, w);
        });
    if (threadIdx.x == 0 && s.nlong > 0) d->rest_long = 1;
  }
}

// Roots of the unreached components start the multi-source BFS at level 0
// (bits in the level-0 frontier bitmap); isolated vertices have level 0
// already and need no expansion.  A wave takes 64 consecutive vertices from a
// multiple of 64, i.e. two whole bitmap words that no other wave of this
// kernel touches: its roots are gathered by ballot and one lane updates each
// word, with no atomics.  The counts go to the slots of the step before 0.
__global__ __launch_bounds__(kThreads) void uf_roots_kernel(const int64_t* off, int64_t n, int32_t* parent,
                                                            int32_t* L, uint32_t* vis, uint32_t* bm0, int32_t* bigs,
                                                            BfsDev* d) {
  static_assert(kThreads % kWave == 0, "waves start at multiples of 64 vertices");
  __shared__ int64_t sh[kThreads / kWave + 1];
  int64_t cnt = 0, edg = 0;
  for (int64_t v0 = blockIdx.x * (int64_t)blockDim.x; v0 < n; v0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t v = v0 + threadIdx.x;
    bool root = false, expand = false;
    if (v < n && !((vis[v >> 5] >> (v & 31)) & 1u) && uf_find(parent, static_cast<int32_t>(v)) == v) {
      root = true;
      L[v] = 0;
      const int64_t dg = row_deg(off, v);
      if (dg > 0) {
        expand = true;
        ++cnt;
        edg += dg;
        list_big(&d->nbig[0], bigs, static_cast<int32_t>(v), dg);
      }
    }
    const uint64_t rm = __ballot(root), em = __ballot(expand);
    if (lane() == 0 && rm) {
      const int64_t w = (v - lane()) >> 5;  // the wave's first word
      if (static_cast<uint32_t>(rm)) vis[w] |= static_cast<uint32_t>(rm);
      if (rm >> 32) vis[w + 1] |= static_cast<uint32_t>(rm >> 32);
      if (static_cast<uint32_t>(em)) bm0[w] |= static_cast<uint32_t>(em);
      if (em >> 32) bm0[w + 1] |= static_cast<uint32_t>(em >> 32);
    }
  }
  add_counts(d->acc[2], cnt, edg, sh);
}

// Clears the counters before uf_roots_kernel, and sets step 0's state after
// it.
__global__ void rest_clear_kernel(BfsDev* d) {
  if (threadIdx.x < 3 * kSlots * 2) (&d->acc[0][0][0])[threadIdx.x] = 0ull;
  if (threadIdx.x < 3) d->nbig[threadIdx.x] = 0;
}
__global__ void rest_start_kernel(int64_t n, int64_t rest, BfsDev* d) {
  const int64_t cnt = wave_sum(static_cast<int64_t>(lane() < kSlots ? d->acc[2][lane()][0] : 0ull));
  const int64_t edg = wave_sum(static_cast<int64_t>(lane() < kSlots ? d->acc[2][lane()][1] : 0ull));
  if (lane() != 0) return;
  d->state[0] = BfsState{rest - edg, goes_up(cnt, edg, rest - edg, n), cnt == 0, cnt != 0, 0};
}
// The state for the host after the steps of the remaining components.
__global__ void rest_state_kernel(int64_t n, int k, const BfsDev* d, BfsHost* out) {
  const BfsState st = state_of(d, k, n);
  if (lane() == 0) *out = BfsHost{st.unexplored, d->maxdeg, d->deg2, st.done, st.num_levels, 0, 0};
}

}  // namespace

BfsWs bfs_reserve(Carver& c, int64_t n) {
  BfsWs w;
  const int64_t words = (n + 31) / 32 + 1;
  w.vis = c.take<uint32_t>(words);
  w.bms = c.take<uint32_t>(3 * words);
  w.big = c.take<int32_t>(2 * kBigCap);
  w.parent = c.take<int32_t>(n + 1);
  w.list = c.take<int32_t>(3 * kRestEntries);  // and two queues (the list itself holds up to kRestNow)
  w.keys = c.take<unsigned long long>(2 * kKeyBlocks);
  w.st = c.take<char>(sizeof(BfsDev));
  w.host = c.take<char>(sizeof(BfsHost));
  w.comp0 = nullptr;
  return w;
}

namespace {

// Blocks of the level kernels: one per 256 vertices (each thread then takes
// one vertex or one 64-vertex wave group per level), at most eight per CU,
// so that a small graph's levels launch only the blocks they can use.
unsigned step_grid(int64_t n) {
  const int64_t g = static_cast<int64_t>(num_cus()) * 8, want = (n + kThreads - 1) / kThreads;
  return static_cast<unsigned>(want < 1 ? 1 : (want < g ? want : g));
}

// Pinned host copy of the BFS state, one per host thread (allocated on
// first use, kept until the process ends; null if it cannot be had, and the
// state is then copied from the workspace): the kernels write it themselves,
// where a readback into pageable memory went through a staging copy.
BfsHost* pinned_state() {
  thread_local BfsHost* p = nullptr;
  thread_local bool tried = false;
  if (!tried) {
    tried = true;
    void* q = nullptr;
    if (hipHostMalloc(&q, sizeof(BfsHost), hipHostMallocDefault) == hipSuccess) p = static_cast<BfsHost*>(q);
    else (void)hipGetLastError();  // the fallback needs no error left behind
  }
  return p;
}

// Reads the state that the last kernel wrote to state_target.
BfsHost* state_target(BfsWs& w) {
  BfsHost* pin = pinned_state();
  return pin ? pin : reinterpret_cast<BfsHost*>(w.host);
}
int read_state(BfsWs& w, BfsHost* out, hipStream_t s) {
  const BfsHost* pin = pinned_state();
  if (!pin) TC_HIP(hipMemcpyAsync(out, w.host, sizeof(BfsHost), hipMemcpyDeviceToHost, s));
  TC_HIP(hipStreamSynchronize(s));
  if (pin) *out = *pin;
  return TC_OK;
}

// Steps k .. k + count - 1.
int launch_steps(const tc_csr* g, int32_t* L, BfsWs& w, int k, int count, hipStream_t s) {
  BfsDev* d = reinterpret_cast<BfsDev*>(w.st);
  for (int i = 0; i < count; ++i)
    step_kernel<<<step_grid(g->n), kThreads, 0, s>>>(g->row_offsets, g->cols, g->n, k + i, d, L, w.vis, w.bms, w.big);
  TC_HIP(hipGetLastError());
  return TC_OK;
}

}  // namespace

int bfs_run(const tc_csr* g, int64_t root, int32_t* L, BfsWs& w, hipStream_t s, BfsInfo* info) {
  const int64_t n = g->n;
  *info = BfsInfo{};
  if (n == 0) return TC_OK;
  const int64_t words = (n + 31) / 32 + 1;
  BfsDev* d = reinterpret_cast<BfsDev*>(w.st);
  const int64_t clear = n > 3 * words ? n : 3 * words;
  const unsigned nk = grid_for(clear, kThreads, kKeyBlocks);
  clear_state_kernel<<<nk, kThreads, 0, s>>>(g->row_offsets, L, n, w.vis, words, w.bms, w.keys);
  start_kernel<<<1, kKeyBlocks, 0, s>>>(g->row_offsets, n, g->nnz, w.keys, static_cast<int>(nk), root, d, L, w.vis,
                                        w.bms, w.big);
  TC_HIP(hipGetLastError());
  BfsHost h;
  const unsigned gu = grid_for(n, kThreads, 16384);
  int k = 0;
  for (int group = kFirstLevels;; group = k == kFirstLevels ? kNextLevels : std::min(2 * group, kMaxLevels)) {
    TC_TRY(launch_steps(g, L, w, k, group, s));
    k += group;
    unreached_kernel<<<gu, kThreads, 0, s>>>(g->row_offsets, n, k, d, w.vis, L, w.comp0, words, w.parent, w.list);
    rest_kernel<<<1, kRestThreads, 0, s>>>(g->row_offsets, g->cols, n, k, d, L, w.parent, w.list, state_target(w));
    TC_HIP(hipGetLastError());
    TC_TRY(read_state(w, &h, s));
    if (h.done) break;
  }
  info->first_levels = info->num_levels = h.num_levels;
  info->maxdeg = h.maxdeg;
  info->deg2 = h.deg2;
  if (h.rest_levels >= 0) {
    info->num_levels = std::max(info->num_levels, h.rest_levels);
    return TC_OK;
  }
  // Remaining components (Alg. 1 rescans for unvisited vertices): one
  // union-find pass over the unreached vertices gives each component its
  // smallest id as root.
  const int64_t rest = h.unexplored;
  uf_init_kernel<<<grid_for(n, kThreads, 65536), kThreads, 0, s>>>(w.parent, n);
  uf_hook_kernel<<<grid_for(n, hook_chunk(n), 65536), kThreads, 0, s>>>(g->row_offsets, g->cols, n, w.vis, w.parent, d);
  TC_TRY(fill_i32(reinterpret_cast<int32_t*>(w.bms), 0, 3 * words, s));
  rest_clear_kernel<<<1, 3 * kSlots * 2, 0, s>>>(d);
  uf_roots_kernel<<<step_grid(n), kThreads, 0, s>>>(g->row_offsets, n, w.parent, L, w.vis, w.bms, w.big, d);
  rest_start_kernel<<<1, kWave, 0, s>>>(n, rest, d);
  TC_HIP(hipGetLastError());
  k = 0;
  for (int group = kNextLevels;; group = std::min(2 * group, kMaxLevels)) {
    TC_TRY(launch_steps(g, L, w, k, group, s));
    k += group;
    if (rest <= kRestEntries)
      rest_tail_kernel<<<1, kRestThreads, 0, s>>>(g->row_offsets, g->cols, n, k, d, L, w.bms, w.list, state_target(w));
    else
      rest_state_kernel<<<1, kWave, 0, s>>>(n, k, d, state_target(w));
    TC_HIP(hipGetLastError());
    TC_TRY(read_state(w, &h, s));
    if (h.done) break;
  }
  info->num_levels = std::max(info->num_levels, h.num_levels);
  return TC_OK;
}

}  // namespace tc

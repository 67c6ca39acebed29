// batch.hip -- tc_count_batch: levels, |H| and T of many small graphs (n <=
// 65536 each) in three kernels that issue no host synchronisation and no
// memset, so a caller can capture the whole call in one hipGraph.  The levels
// and |H| are those of Alg. 1; T is summed by edges over forward lists, which
// reads less here than Alg. 1's horizontal edges do.
//
// The level kernel (one block per graph): BFS levels of Alg. 1 with the level array
// resident in LDS as uint16 (128 KB for 65536 vertices).  The first root is
// the highest-degree vertex (smallest id on ties); the root of every other
// component is its smallest id, as in the scan order of Alg. 1, and isolated
// vertices get level 0.  The other components are levelled together where they
// are few vertices, else one after another, and after a few of those together
// again, from labels of all of them.  Each level of a search is one pass over
// the vertices: top-down from the listed frontier (16 lanes a row, longer rows
// a wave or more) or, when the last level was large, bottom-up.
// The block writes the level parity as a bit array (Lemma 1: for adjacent
// vertices L(x) = L(y) iff their parities agree, so the parity is all that
// |H| needs) and the optional int32 levels.
//
// Before it, one grid-wide kernel cuts every graph's CSR entries into work
// pieces and finds, per vertex, where the neighbours above it start
// (the forward list N+(v): a suffix of the sorted row).
//
// The counting kernel gives a block one piece.  |H| is the number of entries
// v > u of equal parity.  T is summed at the smallest edge of each triangle:
// a triangle a < b < c has one or three horizontal edges, so every triangle
// of the graph is one of Alg. 1's (edge, apex) pairs exactly once, and it is
// found once at its edge (a, b) as an element c of N+(b) that lies in N(a).
// The lists streamed are N+(v) instead of N(v): 2.3 times fewer elements on
// G(n, p) graphs (n = 20000, mean degree 36: 4.3 M against 10.2 M for the
// whole lists of the horizontal edges) and on R-MAT scale 10 to 13.
#include "direct_rule.h"
#include "tc_internal.h"

namespace tc {

namespace {

constexpr int kBfsThreads = 1024;
constexpr uint16_t kUnvisited = 0xFFFF;
// Level 65535 is kUnvisited.  Only the last vertex of a path of 65536 searched
// from its other end has it: once level 65534 is reached, all vertices but one
// are, and that one, if it is not isolated, is its neighbour.
constexpr int kLastLevel = TC_BATCH_MAX_N - 2;
constexpr int kFrontCap = 2048;  // frontier vertices of a top-down level (at most n / 32 there)
constexpr int kRowLanes = 16;    // lanes that expand a frontier row together
// A longer frontier row is expanded by a wave or more (bounds of 64 to 384
// alike: 48 small graphs 88 to 92 us, R-MAT scale 10 27 to 28).
constexpr int kLongRow = 128;
constexpr int kRowLoads = 8;     // row entries a thread loads at once in a bottom-up level
constexpr int kRestCap = 6144;   // unreached vertices of other components levelled together (LDS left beside L)
constexpr int kRestEntries = 65536;  // and their row entries
constexpr int kRestRow = 64;     // a longer row of theirs is a wave's, not a thread's
constexpr int kRestLong = kRestEntries / (kRestRow + 1);  // such rows at most
constexpr int kSearches = 4;     // searches of one component each before all are labelled
constexpr int kLabelEntries = 65536;  // entries to label per search so far (each costs about what a search does)
constexpr int kLabelLong = 8192; // long rows among them
constexpr int kPieceMin = 1024;  // smallest piece size a caller may ask for
constexpr int kAutoMin = 16;     // smallest piece size chosen by auto_piece

// Piece slots of graph g start at row_offsets[vbase[g]] / piece + g, parity
// words at vbase[g] / 32 + g: both leave room for ceil(size / unit) entries.
__device__ __forceinline__ int64_t piece_base(int64_t e0, int piece, int g) {
  // a 64-bit division is a hundred instructions: powers of two shift (uniform branch)
  return ((piece & (piece - 1)) == 0 ? e0 >> (31 - __clz(piece)) : e0 / piece) + g;
}
__device__ __forceinline__ int64_t parity_base(int64_t v0, int g) { return v0 / 32 + g; }

__device__ __forceinline__ int64_t block_max_i64(int64_t v, int64_t* sh) {
  v = wave_max(v);
  const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
  if (lane() == 0) sh[w] = v;
  __syncthreads();
  const int64_t r = wave_max(lane() < nw ? sh[lane()] : sh[0]);
  __syncthreads();
  return r;
}

// LDS of a level block.  L is the level array; the rest beside it serves the
// frontier of a top-down level and, at other times, the unreached vertices.
struct LevelLds {
  alignas(4) uint16_t L[TC_BATCH_MAX_N];
  union {
    struct {
      uint16_t all[kFrontCap];
      uint16_t row[kFrontCap];  // of them, those with rows longer than kLongRow
    } front;
    struct {
      uint16_t v[kRestCap];    // an unreached vertex
      uint16_t low[kRestCap];  // the smallest vertex known of its component
      uint16_t row[kRestLong];  // places of those with rows longer than kRestRow
    } rest;
    struct {
      uint32_t out[TC_BATCH_MAX_N / 32];  // bits of the unreached vertices
      uint16_t row[kLabelLong];           // those with rows longer than kRestRow
    } label;
  };
  int64_t sh[kBfsThreads / kWave + 1];
  int cnt, num, nlong;
};

// Level-synchronous BFS from the vertex of level 0 (set by the caller), with
// L resident in LDS; kLong: rows may be longer than kLongRow.  Returns its last
// level.
template <bool kLong>
__device__ int bfs_levels_lds(LevelLds& s, const int64_t* rows, const int32_t* cols, int n) {
  const int tid = threadIdx.x, nt = blockDim.x, ln = lane();
  uint16_t* L = s.L;
  int level = 0;
  int last = 1;  // vertices found at the previous level
  for (;;) {
    bool bottom_up = last > n / 32;
    if (tid == 0) {
      s.cnt = s.num = 0;
      if (kLong) s.nlong = 0;
    }
    __syncthreads();
    int found = 0;
    const uint16_t cur = static_cast<uint16_t>(level), nxt = static_cast<uint16_t>(level + 1);
    // every lanes-th of the row entries [k0, e), where `lanes` lanes share a row
    auto expand = [&](int64_t k0, int64_t e, int lanes) {
      for (; k0 < e; k0 += lanes * 4) {
        int32_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = k0 + u * lanes < e ? cols[k0 + u * lanes] : -1;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (w[u] >= 0 && L[w[u]] == kUnvisited) {
            L[w[u]] = nxt;
            ++found;
          }
      }
    };
    // `found` may count a vertex more than once in the top-down pass (two
    // parents in one level); it only steers the direction and the stop test
    auto add_found = [&]() {
      const int f = wave_sum(found);
      if (ln == 0 && f) atomicAdd(&s.cnt, f);
    };
    if (!bottom_up) {
      // the frontier is listed; with the same level of components searched
      // before it may not fit (an unvisited vertex has no neighbour there).
      // Two levels are read at once: a grid of 100 x 100 443 us one by one, 404 so
      auto list = [&](int i) {
        const int q = atomicAdd(&s.num, 1);
        if (q < kFrontCap) s.front.all[q] = static_cast<uint16_t>(i);
      };
      for (int i = 2 * tid; i < n; i += 2 * nt) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(L + i);
        if ((w & 0xFFFF) == cur) list(i);
        if (w >> 16 == cur && i + 1 < n) list(i + 1);
      }
      __syncthreads();
      bottom_up = s.num > kFrontCap;
    }
    if (bottom_up) {
      // rows are read kRowLoads entries at a time (independent loads in
      // flight together) and left after the group holding the first parent
      for (int i = tid; i < n; i += nt) {
        if (L[i] != kUnvisited) continue;
        const int64_t e = rows[i + 1];
        for (int64_t k = rows[i]; k < e; k += kRowLoads) {
          int32_t w[kRowLoads];
#pragma unroll
          for (int q = 0; q < kRowLoads; ++q) w[q] = k + q < e ? cols[k + q] : -1;
          bool hit = false;
#pragma unroll
          for (int q = 0; q < kRowLoads; ++q) hit |= w[q] >= 0 && L[w[q]] == cur;
          if (hit) {
            L[i] = nxt;
            ++found;
            break;
          }
        }
      }
    } else {
      const int m = s.num;
      for (int q = tid / kRowLanes; q < m; q += nt / kRowLanes) {
        const int i = s.front.all[q];
        const int64_t b = rows[i], e = rows[i + 1];
        if (!kLong || e - b <= kLongRow) expand(b + tid % kRowLanes, e, kRowLanes);
        else if (tid % kRowLanes == 0) s.front.row[atomicAdd(&s.nlong, 1)] = static_cast<uint16_t>(i);
      }
    }
    add_found();
    __syncthreads();
    last = s.cnt;
    const int nl = kLong ? s.nlong : 0;
    if (nl > 0) {  // uniform
      // the long rows share the block, a wave each at least (with 16 lanes for
      // any row a star of 65536 vertices took 750 us, 334 so)
      int sh = __builtin_ctz(kBfsThreads);
      while ((1 << sh) > kWave && (nl << sh) > nt) --sh;
      found = 0;
      for (int q = tid >> sh; q < nl; q += nt >> sh) {
        const int i = s.front.row[q];
        expand(rows[i] + (tid & ((1 << sh) - 1)), rows[i + 1], 1 << sh);
      }
      add_found();
      __syncthreads();
      last = s.cnt;
    }
    __syncthreads();
    if (last == 0 || ++level == kLastLevel) break;
  }
  return level;
}

// The remaining components together, when they hold at most kRestCap vertices
// and, where rows may be longer than kRestRow (may_long), kRestEntries entries:
// L of a listed vertex is its place in the list while the smallest vertex of
// every component spreads through it (each pass also jumps to the label of the
// label), then levels from those vertices.  One search per component instead
// took 0.94 ms on a Chung-Lu graph of 8001 vertices and mean degree 6, whose
// hundreds of small components each cost passes over all vertices.  With every
// row walked by a thread, a star of 6000 vertices beside one of 20000 took 2.8
// ms, 3.5 where its hub has the largest id; the two together now take 0.67.
// Returns false if there are more: a search of their own levels dense
// components sooner.
__device__ bool rest_levels_lds(LevelLds& s, const int64_t* rows, const int32_t* cols, int n, bool may_long) {
  const int tid = threadIdx.x, nt = blockDim.x, wv = tid / kWave, nw = nt / kWave, ln = lane();
  uint16_t* L = s.L;
  if (tid == 0) s.num = s.cnt = s.nlong = 0;
  __syncthreads();
  int entries = 0;
  for (int i = tid; i < n; i += nt)
    if (L[i] == kUnvisited) {
      const int q = atomicAdd(&s.num, 1);
      if (q >= kRestCap) continue;
      s.rest.v[q] = static_cast<uint16_t>(i);
      if (!may_long) continue;  // rows short enough for a thread each, whatever their sum
      const int64_t dg = rows[i + 1] - rows[i];
      entries += static_cast<int>(min(dg, static_cast<int64_t>(kRestEntries + 1)));
      if (dg > kRestRow) {
        const int at = atomicAdd(&s.nlong, 1);
        if (at < kRestLong) s.rest.row[at] = static_cast<uint16_t>(q);
      }
    }
  if (may_long) {
    entries = wave_sum(entries);
    if (ln == 0 && entries) atomicAdd(&s.cnt, entries);
  }
  __syncthreads();
  const int m = s.num, nl = s.nlong;
  if (m > kRestCap || s.cnt > kRestEntries) return false;  // then nl fits as well
  if (m == 0) return true;
  for (int q = tid; q < m; q += nt) {
    s.rest.low[q] = s.rest.v[q];
    L[s.rest.v[q]] = static_cast<uint16_t>(q);
  }
  // a neighbour of an unreached vertex is unreached, so L of it is a place
  // (min: in a list that is not symmetric it may be a level)
  auto place = [&](int v) { return min(static_cast<int>(L[v]), m - 1); };
  auto low_of = [&](int v) { return static_cast<int>(s.rest.low[place(v)]); };
  for (int more = 1; more;) {
    __syncthreads();
    int changed = 0;
    auto take = [&](int q, int low) {
      low = min(low, low_of(low));
      if (low < s.rest.low[q]) {
        s.rest.low[q] = static_cast<uint16_t>(low);
        changed = 1;
      }
    };
    for (int q = tid; q < m; q += nt) {
      const int v = s.rest.v[q];
      const int64_t b = rows[v], e = rows[v + 1];
      if (may_long && e - b > kRestRow) continue;
      int low = s.rest.low[q];
      for (int64_t k = b; k < e; ++k) low = min(low, low_of(cols[k]));
      take(q, low);
    }
    for (int i = wv; i < nl; i += nw) {
      const int q = s.rest.row[i], v = s.rest.v[q];
      int low = s.rest.low[q];
      for (int64_t k = rows[v] + ln, e = rows[v + 1]; k < e; k += kWave) low = min(low, low_of(cols[k]));
      low = kUnvisited - wave_max(kUnvisited - low);
      if (ln == 0) take(q, low);
    }
    more = __syncthreads_or(changed);
  }
  for (int q = tid; q < m; q += nt) {
    const int v = s.rest.v[q];
    L[v] = s.rest.low[q] == v ? 0 : kUnvisited;
  }
  for (int level = 0, more = 1; more; ++level) {
    __syncthreads();
    int found = 0;
    auto reach = [&](int w) {
      if (L[w] != kUnvisited) return;
      L[w] = static_cast<uint16_t>(level + 1);
      found = 1;
    };
    for (int q = tid; q < m; q += nt) {
      const int v = s.rest.v[q];
      if (L[v] != level) continue;
      const int64_t b = rows[v], e = rows[v + 1];
      if (may_long && e - b > kRestRow) continue;
      for (int64_t k = b; k < e; ++k) reach(cols[k]);
    }
    for (int i = wv; i < nl; i += nw) {
      const int v = s.rest.v[s.rest.row[i]];
      if (L[v] != level) continue;
      for (int64_t k = rows[v] + ln, e = rows[v + 1]; k < e; k += kWave) reach(cols[k]);
    }
    more = __syncthreads_or(found);
  }
  return true;
}

// Any number of remaining components, at most `most` entries: L of an unreached
// vertex is the smallest vertex known of its component (as above), and level 0
// or kUnvisited in the end, so that one search levels them all.  One search
// after another took 3.4 s on 30000 disjoint edges.  Returns false if there are
// more entries or long rows.
__device__ bool label_lds(LevelLds& s, const int64_t* rows, const int32_t* cols, int n, int64_t most) {
  const int tid = threadIdx.x, nt = blockDim.x, wv = tid / kWave, nw = nt / kWave, ln = lane();
  uint16_t* L = s.L;
  if (tid == 0) s.nlong = 0;
  __syncthreads();
  int64_t entries = 0;
  for (int i0 = tid - ln; i0 < n; i0 += nt) {
    const int i = i0 + ln;
    const bool out = i < n && L[i] == kUnvisited;
    const uint64_t m = __ballot(out);
    if ((ln & 31) == 0 && i < n) s.label.out[i >> 5] = static_cast<uint32_t>(m >> ln);
    if (!out) continue;
    const int64_t dg = rows[i + 1] - rows[i];
    entries += dg;
    if (dg <= kRestRow) continue;
    const int q = atomicAdd(&s.nlong, 1);
    if (q < kLabelLong) s.label.row[q] = static_cast<uint16_t>(i);
  }
  entries = block_sum(entries, s.sh);
  const int nl = s.nlong;
  if (entries > most || nl > kLabelLong) return false;
  auto out = [&](int i) { return (s.label.out[i >> 5] >> (i & 31)) & 1u; };
  for (int i = tid; i < n; i += nt)
    if (out(i)) L[i] = static_cast<uint16_t>(i);
  for (int more = 1; more;) {
    __syncthreads();
    int changed = 0;
    auto take = [&](int i, int low) {
      low = min(low, static_cast<int>(L[low]));
      if (low < L[i]) {
        L[i] = static_cast<uint16_t>(low);
        changed = 1;
      }
    };
    for (int i = tid; i < n; i += nt) {
      if (!out(i)) continue;
      const int64_t b = rows[i], e = rows[i + 1];
      if (e - b > kRestRow) continue;
      int low = L[i];
      for (int64_t k = b; k < e; ++k) low = min(low, static_cast<int>(L[cols[k]]));
      take(i, low);
    }
    for (int q = wv; q < nl; q += nw) {
      const int i = s.label.row[q];
      int low = L[i];
      for (int64_t k = rows[i] + ln, e = rows[i + 1]; k < e; k += kWave) low = min(low, static_cast<int>(L[cols[k]]));
      low = kUnvisited - wave_max(kUnvisited - low);
      if (ln == 0) take(i, low);
    }
    more = __syncthreads_or(changed);
  }
  for (int i = tid; i < n; i += nt)
    if (out(i)) L[i] = L[i] == i ? 0 : kUnvisited;
  __syncthreads();
  return true;
}

// Levels of graph g (its vertices v0 .. v0 + n - 1), one block.  root0 >= 0
// replaces the default root.  Inlined: as a function it saves registers to
// scratch (120 of them used and 24 bytes, 52 and none inlined), and 10000 graphs
// of 16 vertices took 494 us instead of 467, 3000 without an edge 120 instead
// of 110; a path's level costs 6% more.
__device__ __forceinline__ void graph_levels(LevelLds& s, int g, int64_t v0, int64_t n64,
                                             const int64_t* row_offsets, const int32_t* cols, int32_t* levels,
                                             uint32_t* parity, int64_t* T, int64_t* H, int32_t root0) {
  uint16_t* L = s.L;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t* rows = row_offsets + v0;  // rows[i] = global position of local row i
  // a graph beyond the on-chip level array is skipped and flagged with -1
  // (the host rejects it first when validation is on); it gets no pieces
  const bool too_big = n64 > TC_BATCH_MAX_N;
  if (tid == 0) {
    T[g] = too_big ? -1 : 0;
    if (H) H[g] = too_big ? -1 : 0;
  }
  if (n64 <= 0 || too_big) return;
  const int n = static_cast<int>(n64);
  // root: highest degree, smallest id on ties; isolated vertices get level 0
  int64_t key = -1;
  for (int i = tid; i < n; i += nt) {
    const int64_t d = rows[i + 1] - rows[i];
    L[i] = d == 0 ? 0 : kUnvisited;
    const int64_t k = (d << 32) | static_cast<int64_t>(0xFFFFFFFFu - static_cast<uint32_t>(i));
    key = k > key ? k : key;
  }
  key = block_max_i64(key, s.sh);
  const int root = root0 >= 0 && root0 < n ? root0
                                           : static_cast<int>(0xFFFFFFFFu - static_cast<uint32_t>(key & 0xFFFFFFFF));
  if (tid == 0) L[root] = 0;  // a given root of degree 0 is level 0 already
  __syncthreads();
  const int64_t maxdeg = key >> 32;
  // called at one place (at three the code was 25 KB instead of 14)
  auto search = [&]() {
    return maxdeg > kLongRow ? bfs_levels_lds<true>(s, rows, cols, n) : bfs_levels_lds<false>(s, rows, cols, n);
  };
  // remaining components: together if they are few vertices, else one search
  // from the smallest unvisited id until they are; every id below the last
  // such root is visited, so each scan starts there.  Where the searches have
  // taken about as long as labelling the rest does, one search levels it.
  int from = 0;
  bool labelled = false;
  for (int searches = 1;; ++searches) {
    if (search() == kLastLevel || labelled || rest_levels_lds(s, rows, cols, n, maxdeg > kRestRow)) break;
    if (searches >= kSearches && (searches & (searches - 1)) == 0 &&
        label_lds(s, rows, cols, n, static_cast<int64_t>(searches) * kLabelEntries)) {
      labelled = true;
      continue;
    }
    int64_t cand = -1;  // max of (n - i) over unvisited i = smallest i
    for (int i = from + tid; i < n; i += nt)
      if (L[i] == kUnvisited) {
        cand = n - i;
        break;
      }
    cand = block_max_i64(cand, s.sh);
    from = static_cast<int>(n - cand);
    if (tid == 0) L[from] = 0;
    __syncthreads();
  }
  __syncthreads();
  // outputs: parity bits (a wave's 64 vertices are two words), levels
  uint32_t* par = parity + parity_base(v0, g);
  for (int i0 = tid - lane(); i0 < n; i0 += nt) {
    const int i = i0 + lane();
    const uint64_t odd = __ballot(i < n && (L[i] & 1));
    if ((lane() & 31) == 0 && i < n) par[i >> 5] = static_cast<uint32_t>(odd >> lane());
  }
  if (levels)
    for (int i = tid; i < n; i += nt) levels[v0 + i] = L[i];
}

__global__ __launch_bounds__(kBfsThreads) void batch_bfs_kernel(const int64_t* vbase, const int64_t* row_offsets,
                                                                const int32_t* cols, int32_t* levels, uint32_t* parity,
                                                                int64_t* T, int64_t* H) {
  __shared__ LevelLds s;
  const int g = blockIdx.x;
  graph_levels(s, g, vbase[g], vbase[g + 1] - vbase[g], row_offsets, cols, levels, parity, T, H, -1);
}

__device__ __forceinline__ uint32_t par_bit(const uint32_t* p, int32_t i) { return (p[i >> 5] >> (i & 31)) & 1u; }

// Forward list of a vertex, N+(v) = its neighbours above it: first entry
// (40 bits, absolute) and length (at most TC_BATCH_MAX_N - 1) in 8 bytes.
struct FwdRec {
  uint32_t lo, hi_len;  // hi_len = first >> 32 | length << 8
};
constexpr int64_t kFwdLenMax = TC_BATCH_MAX_N - 1;  // a simple graph's lists are no longer
__device__ __forceinline__ FwdRec pack_fwd(int64_t first, int len) {
  return FwdRec{static_cast<uint32_t>(first),
                static_cast<uint32_t>(static_cast<uint64_t>(first) >> 32) | (static_cast<uint32_t>(len) << 8)};
}

// One launch before the counting kernel: forward records of every vertex
// (kRec), the piece slots (slot -> graph, first row; graph -1: empty), and
// where one graph is counted alone its vertex bases {0, n}, the work
// statistics and, if its levels are given, the outputs' zeros and the parity
// bits.  A wave takes 64 consecutive vertices: one search of the vertex bases
// finds the first one's graph, the lanes step on from there.
struct OneGraph {
  int64_t* vbase;     // written {0, n}; null for a batch
  int64_t* stats;
  int64_t n, nnz;
  const int32_t* L;   // levels already known (null: batch_bfs_kernel writes parity, T and H)
  int64_t num_levels;
  uint32_t* parity;
  int64_t* sums;      // then: kSumStripes of T and |H|, written 0
};

// One graph's T and |H| are added in stripes of a 128-byte line each: the
// additions of thousands of blocks to one place take about 4 ns each (G(300007,
// d 24): 267 -> 223 us with the launch that sums the stripes).
constexpr int kSumStripes = 32, kSumPad = 16;

template <bool kRec>
__device__ void batch_prep(int64_t t0, int64_t stride, const int64_t* vbase, int G, const int64_t* row_offsets,
                           const int32_t* cols, int64_t total_n, int64_t nslots, int piece, FwdRec* rec, int2* pieces,
                           const OneGraph& one) {
  const bool single = one.vbase != nullptr;
  if (single) {
    if (t0 < 2) one.vbase[t0] = t0 ? one.n : 0;
    if (t0 < 24) one.stats[t0] = t0 == 0 ? one.n : (t0 == 1 ? one.nnz : (t0 == 3 ? one.num_levels : 0));
    if (one.L)
      for (int64_t i = t0; i < kSumStripes * kSumPad; i += stride) one.sums[i] = 0;
  }
  const int64_t max_n = one.L ? INT64_MAX : TC_BATCH_MAX_N;
  auto base_of = [&](int g) -> int64_t { return single ? (g ? one.n : 0) : vbase[g]; };
  if (kRec) {
    for (int64_t w0 = t0 - lane(); w0 < total_n; w0 += stride) {
      int g = 0;
      if (!single) {
        int lo = 0, hi = G;  // last g with vbase[g] <= w0
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (vbase[mid] <= w0) lo = mid;
          else hi = mid;
        }
        g = lo;
      }
      const int64_t v = w0 + lane();
      if (one.L) {
        const uint64_t odd = __ballot(v < total_n && (one.L[v] & 1));
        if ((lane() & 31) == 0 && v < total_n) one.parity[v >> 5] = static_cast<uint32_t>(odd >> lane());
      }
      if (v >= total_n) continue;
      while (g + 1 < G && base_of(g + 1) <= v) ++g;
      const int64_t v0 = base_of(g);
      if (base_of(g + 1) - v0 > max_n) continue;  // a skipped graph has no pieces
      const int64_t b = row_offsets[v], e = row_offsets[v + 1];
      const int64_t f = upper_bound_dev(cols, b, e, static_cast<int32_t>(v - v0));
      rec[v] = pack_fwd(f, static_cast<int>(min(e - f, kFwdLenMax)));
    }
  }
  for (int64_t s = t0; s < nslots; s += stride) {
    int g = 0;
    if (!single) {
      int lo = 0, hi = G;  // last g whose first slot is at or before s
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (piece_base(row_offsets[vbase[mid]], piece, mid) <= s) lo = mid;
        else hi = mid;
      }
      g = lo;
    }
    const int64_t v0 = base_of(g);
    const int64_t n = base_of(g + 1) - v0;
    const int64_t* rows = row_offsets + v0;
    const int64_t e0 = rows[0];
    const int64_t p = s - piece_base(e0, piece, g), ps = e0 + p * piece;
    int2 out = make_int2(-1, 0);
    // the piece's first row is the last one starting at or before entry ps
    // (rows[n] > ps, so that row is not empty)
    if (n > 0 && n <= max_n && p >= 0 && ps < rows[n])
      out = make_int2(g, static_cast<int>(upper_bound_dev(rows, 0, n + 1, ps)) - 1);
    pieces[s] = out;
  }
}

template <bool kRec>
__global__ void batch_prep_kernel(const int64_t* vbase, int G, const int64_t* row_offsets, const int32_t* cols,
                                  int64_t total_n, int64_t nslots, int piece, FwdRec* rec, int2* pieces,
                                  OneGraph one) {
  batch_prep<kRec>(blockIdx.x * (int64_t)blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x, vbase, G,
                   row_offsets, cols, total_n, nslots, piece, rec, pieces, one);
}

// Few and small graphs: the levels (blocks 0 .. G - 1) and the rest of the
// preparation (the blocks after them, on CUs the levels leave idle) in one
// launch.
__global__ __launch_bounds__(kBfsThreads) void batch_first_kernel(const int64_t* vbase, int G,
                                                                  const int64_t* row_offsets, const int32_t* cols,
                                                                  int64_t total_n, int64_t nslots, int piece,
                                                                  FwdRec* rec, int2* pieces, OneGraph one,
                                                                  int32_t* levels, uint32_t* parity, int64_t* T,
                                                                  int64_t* H, int32_t root0) {
  __shared__ LevelLds s;
  const int g = blockIdx.x;
  if (g < G) {
    const int64_t v0 = one.vbase ? 0 : vbase[g], v1 = one.vbase ? one.n : vbase[g + 1];
    graph_levels(s, g, v0, v1 - v0, row_offsets, cols, levels, parity, T, H, root0);
  } else {
    batch_prep<true>((blockIdx.x - G) * static_cast<int64_t>(kBfsThreads) + threadIdx.x,
                     (gridDim.x - G) * static_cast<int64_t>(kBfsThreads), vbase, G, row_offsets, cols, total_n, nslots,
                     piece, rec, pieces, one);
  }
}

constexpr int kRows = 2;                 // rows a thread looks at for a tile
constexpr int kCols = 1024;
constexpr int kQueue = 256;              // hits of a tile looked up together
constexpr int kSumTiles = 64;            // tiles added up in 32 bits (fewer than 2^22 chunks of 8 each)
constexpr int kFilterBits = TC_BATCH_MAX_N;
constexpr int kWinTiles = 64;            // 64-chunk groups whose stream starts are marked at once
static_assert(kLongList == TC_BATCH_MAX_N - kBChunk, "a graph of a batch has at most 28 longer lists in a tile");
constexpr int kLongMany = 64;
constexpr uint32_t kRowStep = 40503u;    // odd: rows of a tile start at spread places of the filter

// Slots of an XCD given to consecutive blocks of that XCD (about the blocks
// it holds at once), where there are many more slots than the chip holds:
// without it the 4096 graphs named below take 3 ms more.
constexpr int kXcds = 8, kXcdRun = 256;

// The counting kernel: a block takes one piece (or, where the caller limits
// the grid, every gridDim.x-th), kTile of its forward entries at a time.
//   1. the next rows' forward parts are laid end to end: a scan of their
//      lengths places them in the tile, a mark at each row's first place
//      gives every entry its row;
//   2. an entry v > u counts towards |H| if the parities agree; its forward
//      list N+(v) becomes a stream, and v itself is set in the tile's filter:
//      one bit at (v + offset of u) mod 65536 (the rest of the tile's last
//      row, beyond the tile, is set as well);
//   3. all streams are cut into chunks of kBChunk entries, dealt to the lanes
//      in order; an element w whose bit is set lies in N(u) above v if the
//      rows' ranges of the filter are disjoint (few rows, or one), else the
//      hit is queued and looked up in the row with the others of the window.
// A tile's dependent loads (forward records, entries, their records, streams)
// are taken once for 512 edges.  Measured on 4096 graphs of 64 to 65536
// vertices (1.08 G entries) and one Chung-Lu graph (n = 30011, mean degree
// 20): a wave per vertex with a 65536-bit map of its own took 43.1 ms and
// 0.54 ms; tiles of 512 entries of both directions, hits looked up where they
// were found, 15.3 ms (6.8 of them the tiles' set-up, half of it for entries
// that have no stream) and 94 us (45 of them the look-ups of the few lanes
// with hits, the other lanes waiting); this form 9.6 ms and 52 us.  VALU
// bound, at seven waves per SIMD, which the 22 KB of LDS allow.
// kWide: one graph of any number of vertices (ids of 32 bits in LDS; a bit of
// the filter then also stands for the ids 65536 apart).
template <int THREADS, bool kRec, bool kWide>
__global__ __launch_bounds__(THREADS, THREADS == kWave ? 2 : (kWide ? 6 : 7)) void batch_count_kernel(const int64_t* vbase, const int64_t* row_offsets,
                                                              const int32_t* cols, int64_t total_nnz,
                                                              const uint32_t* parity, const FwdRec* rec,
                                                              const int2* pieces, int64_t nslots, int piece,
                                                              bool by_xcd, int64_t* T, int64_t* H, int64_t* H2) {
  if (kWide) {  // this block's stripe
    T += blockIdx.x % kSumStripes * kSumPad;
    H += blockIdx.x % kSumStripes * kSumPad;
  }
  constexpr int NW = THREADS / kWave;
  constexpr int kPer = kTile / THREADS;  // entries per thread
  static_assert(kPer * THREADS == kTile, "whole entries per thread");
  __shared__ alignas(16) uint32_t s_filt[kFilterBits / 32];
  // streams of the tile: first chunk, entry position of the list (relative to
  // the graph), length | filter offset of the row << 16, the places of the
  // row's entries after the edge's (first | end << 16)
  using Id = typename std::conditional<kWide, int32_t, uint16_t>::type;
  __shared__ uint4 s_st[kTile];
  __shared__ Id s_col[kCols];  // ids of the tile's entries, then of the last row's beyond it as far as they fit
  __shared__ uint16_t s_own[kTile];  // at a row's first entry in the tile: the row (from the tile's first one)
  __shared__ alignas(8) uint32_t s_beg[kTile / 32];  // bits of those entries
  __shared__ uint2 s_q[kQueue];  // list entries with a hit, and their stream's places
  uint32_t* s_src = reinterpret_cast<uint32_t*>(s_q);  // before the hits: a row's first position less its place
  static_assert(sizeof(s_q) >= sizeof(uint32_t) * kTile, "s_src fits");
  __shared__ uint32_t s_M[kWinTiles][2];
  __shared__ int32_t s_tb[kWinTiles];
  __shared__ uint32_t sh[NW + 1];
  __shared__ uint32_t s_sum[2][NW];
  __shared__ uint2 s_cut;
  __shared__ uint32_t s_cur;
  __shared__ int s_long, s_qn, s_next, s_done;
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid / kWave), ln = lane();
  for (int64_t bi = blockIdx.x;; bi += gridDim.x) {
    // consecutive blocks go to different XCDs: by_xcd gives the blocks of one
    // XCD kXcdRun consecutive slots, so the pieces of a graph share one L2
    int64_t sl = bi;
    if (by_xcd) {
      constexpr int64_t kAll = static_cast<int64_t>(kXcds) * kXcdRun;
      const int64_t r = bi / kXcds;
      sl = (r / kXcdRun) * kAll + (bi % kXcds) * kXcdRun + r % kXcdRun;
      if (bi >= (nslots + kAll - 1) / kAll * kAll) break;
      if (sl >= nslots) continue;
    } else if (sl >= nslots) {
      break;
    }
    const int2 pc = pieces[sl];
    if (pc.x < 0) continue;  // empty slot (block-uniform)
    const int g = pc.x;
    const int64_t v0 = vbase[g];
    const int n = static_cast<int>(vbase[g + 1] - v0);
    const int64_t* rows = row_offsets + v0;
    const int64_t e0 = rows[0];
    const uint32_t* par = parity + parity_base(v0, g);
    const int64_t ps = e0 + (sl - piece_base(e0, piece, g)) * piece;
    const int64_t pe = min(ps + piece, rows[n]);
    // every list ends a whole chunk before the columns do
    const bool inside = rows[n] + kBChunk <= total_nnz;
    // the next slot's first row bounds the piece's (the last row of the graph
    // where that slot is empty or another graph's)
    const int2 pn = sl + 1 < nslots ? pieces[sl + 1] : make_int2(-1, 0);
    const int vz = pn.x == g ? pn.y : n - 1;
    uint32_t tc = 0, th = 0;  // of the tiles not yet added up
    int tiles_left = kSumTiles;
    auto add_up = [&]() {
      tc = wave_sum(tc);
      th = wave_sum(th);
      if (ln == 0) {
        s_sum[0][wv] = tc;
        s_sum[1][wv] = th;
      }
      __syncthreads();
      if (tid == 0) {
        int64_t cnt = 0, hc = 0;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
          cnt += s_sum[0][q];
          hc += s_sum[1][q];
        }
        if (cnt) atomicAdd(reinterpret_cast<unsigned long long*>(&T[g]), static_cast<unsigned long long>(cnt));
        if (hc && H) atomicAdd(reinterpret_cast<unsigned long long*>(&H[g]), static_cast<unsigned long long>(hc));
        if (hc && H2) atomicAdd(reinterpret_cast<unsigned long long*>(H2), static_cast<unsigned long long>(hc));
      }
      tc = th = 0;
      tiles_left = kSumTiles;
    };
    // positions are relative to the graph's first entry
    const uint32_t end = static_cast<uint32_t>(pe - e0);
    uint32_t cur = static_cast<uint32_t>(ps - e0);  // the piece's entries before it are done
    int vb = pc.y;
    for (;;) {
      __syncthreads();  // the previous tile is done with the LDS
      // the forward parts of the next rows, as far as the piece has them
      uint32_t fs[kRows], fl[kRows], fe[kRows];
      uint32_t sum = 0;
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        const int r = vb + tid * kRows + k;
        fs[k] = fl[k] = fe[k] = 0;
        if (r > vz) continue;
        if (kRec) {
          const FwdRec q = rec[v0 + r];
          fs[k] = static_cast<uint32_t>((static_cast<int64_t>(q.lo) | (static_cast<int64_t>(q.hi_len & 0xFFu) << 32)) - e0);
          fe[k] = fs[k] + (q.hi_len >> 8);
        } else {
          const int64_t e = rows[r + 1];
          fs[k] = static_cast<uint32_t>(upper_bound_dev(cols, rows[r], e, r) - e0);
          fe[k] = static_cast<uint32_t>(e - e0);
        }
      }
      for (int i = tid; i < kFilterBits / 128; i += THREADS)
        reinterpret_cast<uint4*>(s_filt)[i] = make_uint4(0u, 0u, 0u, 0u);
      if (tid < kTile / 32) s_beg[tid] = 0u;
      if (tid == 0) {
        s_long = s_qn = 0;
        s_next = vb + kRows * THREADS;
        s_cut = make_uint2(0u, 0u);
        s_done = 0;
      }
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        const uint32_t z = min(fe[k], end);
        fs[k] = max(fs[k], cur);
        fl[k] = z > fs[k] ? z - fs[k] : 0u;
        sum += fl[k];
      }
      uint32_t total;
      uint32_t at0 = block_excl_scan(sum, sh, &total);
      const int tn = static_cast<int>(min(total, static_cast<uint32_t>(kTile)));
      // rows mark their first entry of the tile; the row that goes on past it
      // is the next tile's first
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        if (fe[k] >= end && vb + tid * kRows + k <= vz) s_done = 1;  // no later row has entries of the piece
        if (fl[k] && at0 <= kTile) {
          if (at0 < kTile) {
            s_own[at0] = static_cast<uint16_t>(tid * kRows + k);
            s_src[at0] = fs[k] - at0;
            atomicOr(&s_beg[at0 >> 5], 1u << (at0 & 31));
          }
          const uint32_t z = min(fl[k], kTile - at0);
          if (fl[k] > z) {
            s_next = vb + tid * kRows + k;
            s_cur = fs[k] + z;
          }
          if (z > 0 && fe[k] > fs[k] + z) s_cut = make_uint2(fs[k] + z, fe[k]);
        }
        at0 += fl[k];
      }
      __syncthreads();
      const bool last_tile = total <= kTile && s_done;
      if (total == 0) {  // uniform, as all below
        if (last_tile) break;
        int nb = vb + kRows * THREADS;
        if (nb > vz) break;
        // empty rows are skipped together
        const int64_t at = rows[nb];
        if (at == rows[vb]) nb = static_cast<int>(upper_bound_dev(rows, nb, vz + 1, at)) - 1;
        if (at >= pe) break;
        vb = nb;
        continue;
      }
      // an entry's row is that of the last mark at or before it: in its own
      // 64 entries (one wave's), else in the last group before with a mark;
      // the mark's rank places the row in the filter
      const uint64_t marks = ln < kTile / 64 ? reinterpret_cast<const uint64_t*>(s_beg)[ln] : 0ull;
      const uint64_t some = __ballot(marks != 0ull);
      auto last_mark = [&](uint64_t groups) {  // of the highest group in the mask (uniform, not empty)
        const int q = 63 - __clzll(static_cast<long long>(groups));
        return q * kWave + 63 - __clzll(static_cast<long long>(wave_read(marks, q)));
      };
      const int upto = wave_incl_scan(__popcll(marks));
      const int nrows = wave_read(upto, kTile / kWave - 1);
      const uint2 cut = s_cut;  // the last row's entries beyond the tile, of them in s_col up to place held
      const int held = static_cast<int>(min(static_cast<uint32_t>(tn) + (cut.y - cut.x), static_cast<uint32_t>(kCols)));
      // disjoint ranges of the filter per row where they fit: a set bit is then exact
      const bool exact = static_cast<int64_t>(nrows) * n <= kFilterBits;
      const uint32_t step = exact ? static_cast<uint32_t>(n) : kRowStep;
      int u[kPer];
      int32_t v[kPer];
      uint32_t off[kPer], az[kPer];  // the row's place in the filter, the places of its entries after this one
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int e = tid + j * THREADS, q = wv + j * NW;
        u[j] = 0;
        v[j] = -1;
        off[j] = az[j] = 0u;
        if (q * kWave >= tn) continue;  // uniform per wave
        const uint64_t below = some & ((1ull << q) - 1ull);
        const int before = below ? last_mark(below) : 0;
        const uint64_t own = wave_read(marks, q) & ((2ull << ln) - 1ull);
        const int at = own ? q * kWave + 63 - __clzll(static_cast<long long>(own)) : before;
        const uint64_t rest = wave_read(marks, q) & ~((2ull << ln) - 1ull), above = some & ~((2ull << q) - 1ull);
        int after = held;
        if (above) {
          const int qa = __ffsll(static_cast<unsigned long long>(above)) - 1;
          after = qa * kWave + __ffsll(static_cast<unsigned long long>(wave_read(marks, qa))) - 1;
        }
        const int row_end = rest ? q * kWave + __ffsll(static_cast<unsigned long long>(rest)) - 1 : after;
        az[j] = static_cast<uint32_t>(e + 1) | (static_cast<uint32_t>(row_end) << 16);
        const int rank = (q > 0 ? wave_read(upto, q - 1) : 0) + __popcll(own) - 1;
        off[j] = __umul24(rank, step) & (kFilterBits - 1);
        if (e < tn) {
          u[j] = vb + static_cast<int>(s_own[at]);
          v[j] = cols[e0 + (s_src[at] + static_cast<uint32_t>(e))];
        }
      }
      uint32_t beg[kPer], len[kPer];
      // chunks | streams << kChunkBits.  Lists of up to kLongList always fit
      // the chunks' bits.  Longer ones: a graph counted alone (kWide) has none
      // (direct_fits); in a batch their ids are below 8 in a simple graph (n is
      // at most TC_BATCH_MAX_N), so at most 28 entries of a tile have one; in
      // any other batch kLongMany keep their length
      uint32_t mine = 0;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        len[j] = beg[j] = 0;
        if (v[j] < 0) continue;  // past the tile
        if (kRec) {
          const FwdRec r = rec[v0 + v[j]];
          const int64_t f = static_cast<int64_t>(r.lo) | (static_cast<int64_t>(r.hi_len & 0xFFu) << 32);
          beg[j] = static_cast<uint32_t>(f - e0);
          len[j] = r.hi_len >> 8;
        } else {
          const int64_t b = rows[v[j]], e = rows[v[j] + 1];
          const int64_t f = upper_bound_dev(cols, b, e, v[j]);
          beg[j] = static_cast<uint32_t>(f - e0);
          len[j] = static_cast<uint32_t>(min(e - f, kFwdLenMax));
        }
        th += par_bit(par, v[j]) == par_bit(par, u[j]);
        s_col[tid + j * THREADS] = static_cast<Id>(v[j]);
        const uint32_t h = (static_cast<uint32_t>(v[j]) + off[j]) & (kFilterBits - 1);
        atomicOr(&s_filt[h >> 5], 1u << (h & 31));
        if (len[j] > kLongList && atomicAdd(&s_long, 1) >= kLongMany) len[j] = kLongList;
        if (len[j]) mine += (len[j] + kBChunk - 1) / kBChunk + (1u << kChunkBits);
      }
      {
        const uint32_t toff = static_cast<uint32_t>(nrows - 1) * step;
        for (uint32_t k = cut.x + tid; k < cut.y; k += THREADS) {
          const int32_t w = cols[e0 + k];
          const uint32_t h = (static_cast<uint32_t>(w) + toff) & (kFilterBits - 1);
          atomicOr(&s_filt[h >> 5], 1u << (h & 31));
          const uint32_t at = tn + (k - cut.x);
          if (at < kCols) s_col[at] = static_cast<Id>(w);
        }
      }
      const int next = s_next;
      if (total > kTile) cur = s_cur;
      uint32_t tot;
      const uint32_t pre = block_excl_scan(mine, sh, &tot);
      constexpr uint32_t kChunks = (1u << kChunkBits) - 1u;
      const int C = static_cast<int>(tot & kChunks), nst = static_cast<int>(tot >> kChunkBits);
      {
        int slot = static_cast<int>(pre >> kChunkBits), ch = static_cast<int>(pre & kChunks);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          if (!len[j]) continue;
          s_st[slot] = make_uint4(static_cast<uint32_t>(ch), beg[j], len[j] | (off[j] << 16), az[j]);
          ++slot;
          ch += static_cast<int>((len[j] + kBChunk - 1) / kBChunk);
        }
      }
      // whether x is among the places az (first | end << 16) of a row, or,
      // where these are the last row's, in the rest of it past s_col
      auto in_row = [&](int32_t x, uint32_t az) -> uint32_t {
        const int z = static_cast<int>(az >> 16);
        int lo = static_cast<int>(az & 0xFFFFu), hi = z;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (s_col[mid] < x) lo = mid + 1;
          else hi = mid;
        }
        if (lo < z) return s_col[lo] == x;
        if (z != held || cut.x + (held - tn) >= cut.y) return 0u;
        const int64_t q0 = lower_bound_dev(cols, e0 + cut.x + (held - tn), e0 + cut.y, x);
        return q0 < e0 + cut.y && cols[q0] == x;
      };
      for (int w0 = 0; w0 < C; w0 += kWinTiles * kWave) {
        for (int i = tid; i < kWinTiles * 2; i += THREADS) (&s_M[0][0])[i] = 0u;
        __syncthreads();
        for (int i = tid; i < nst; i += THREADS) {
          const int f = static_cast<int>(s_st[i].x) - w0;
          if (f >= 0 && f < kWinTiles * kWave) atomicOr(&s_M[f >> 6][(f >> 5) & 1], 1u << (f & 31));
        }
        __syncthreads();
        if (wv == 0) {
          int lo = 0, hi = w0 > 0 ? nst : 0;  // streams begun before the window
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (static_cast<int>(s_st[mid].x) < w0) lo = mid + 1;
            else hi = mid;
          }
          const int k = __popc(s_M[ln][0]) + __popc(s_M[ln][1]);
          s_tb[ln] = lo + wave_incl_scan(k) - k;
        }
        __syncthreads();
        const int tiles = min(kWinTiles, (C - w0 + kWave - 1) / kWave);
        for (int t = wv; t < tiles; t += NW) {
          const int c = w0 + t * kWave + ln;
          if (c >= C) continue;
          const uint32_t m0 = s_M[t][0], m1 = s_M[t][1];
          const int below = static_cast<int>(__builtin_amdgcn_mbcnt_hi(m1, __builtin_amdgcn_mbcnt_lo(m0, 0u)));
          const int own = static_cast<int>(((ln < 32 ? m0 : m1) >> (ln & 31)) & 1u);
          const int j = s_tb[t] + below + own - 1;
          const uint4 st = s_st[j];
          const int k0 = (c - static_cast<int>(st.x)) * kBChunk;
          const int rem = static_cast<int>(st.z & 0xFFFFu) - k0;
          const uint32_t so = st.z >> 16;
          const uint32_t p0 = st.y + static_cast<uint32_t>(k0);
          uint32_t valid = rem >= kBChunk ? (1u << kBChunk) - 1u : (1u << rem) - 1u;
          int32_t w[kBChunk];
          if (inside) {  // the whole chunk is loaded
#pragma unroll
            for (int q = 0; q < kBChunk; ++q) w[q] = cols[e0 + p0 + q];
          } else if (total_nnz >= kBChunk) {  // moved back where it would pass the columns' end
            const int64_t over = e0 + p0 + kBChunk - total_nnz;
            const int64_t back = over > 0 ? over : 0;
            valid <<= back;
#pragma unroll
            for (int q = 0; q < kBChunk; ++q) w[q] = cols[e0 + p0 - back + q];
          } else {
#pragma unroll
            for (int q = 0; q < kBChunk; ++q) w[q] = q < rem ? cols[e0 + p0 + q] : 0;
          }
          uint32_t hits = 0;
#pragma unroll
          for (int q = 0; q < kBChunk; ++q) {
            const uint32_t h = static_cast<uint32_t>(w[q]) + so;
            hits |= __builtin_amdgcn_ubfe(s_filt[(h & (kFilterBits - 1)) >> 5], h & 31, 1) << q;
          }
          hits &= valid;
          if (exact) {
            tc += __popc(hits);
            continue;
          }
          // hits, real and false ones, are looked up together after the
          // window: one here and there, they would stop a whole wave each
          for (uint64_t any = __ballot(hits != 0u); any; any = __ballot(hits != 0u)) {
            const int first = __ffsll(static_cast<unsigned long long>(any)) - 1;
            int base = 0;
            if (ln == first) base = atomicAdd(&s_qn, __popcll(any));
            base = wave_read(base, first);
            if (hits) {
              int32_t x = w[0];
#pragma unroll
              for (int q = 1; q < kBChunk; ++q)
                if ((hits & ((1u << q) - 1u)) == 0u) x = w[q];
              hits &= hits - 1;
              const int to = base + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                                        static_cast<uint32_t>(any >> 32),
                                        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(any), 0u)));
              if (to < kQueue) s_q[to] = make_uint2(static_cast<uint32_t>(x), st.w);
              else tc += in_row(x, st.w);
            }
          }
        }
        __syncthreads();
        const int nq = min(s_qn, kQueue);
        for (int i = tid; i < nq; i += THREADS) tc += in_row(static_cast<int32_t>(s_q[i].x), s_q[i].y);
        __syncthreads();
        if (tid == 0) s_qn = 0;
      }
      if (last_tile) break;
      vb = next;
      if (vb > vz) break;
      if (--tiles_left == 0) add_up();
    }
    add_up();
  }
}

// Piece size where the caller names none: the entries are spread over about
// kAutoSlots blocks (eight per CU, what their LDS allows), one wave each for
// the smallest graphs, until a piece is one whole tile of forward entries
// (half its entries, on average); where there are kAutoMany of those, two
// tiles a piece waste less of the last one (4096 graphs: 14.3 ms at 1024
// entries, 13.5 at 2048, 14.2 at 4096, 15.1 at 8192; 17.9 at 512).
constexpr int64_t kAutoSlots = 2048, kAutoMany = 16384;
constexpr int kAutoMax = 2048;

int auto_piece(int64_t total_nnz) {  // a power of two, so that the kernels shift instead of dividing
  int piece = kAutoMin;
  while (piece < kAutoMax && 2 * piece * (piece < 2 * kTile ? kAutoSlots : kAutoMany) <= total_nnz) piece *= 2;
  return piece;
}

struct BatchPlan {
  uint32_t* parity;
  int2* pieces;
  FwdRec* rec;  // null: the counting kernel finds the forward lists itself
  size_t bytes;
};

BatchPlan plan_batch(void* base, int64_t total_n, int64_t total_nnz, int32_t G, bool with_rec) {
  BatchPlan p;
  Carver c(base);
  p.parity = c.take<uint32_t>(total_n / 32 + G + 2);
  // the most slots any call of this size has: the default piece may be larger than the smallest to ask for
  p.pieces = c.take<int2>(total_nnz / std::min(auto_piece(total_nnz), kPieceMin) + G + 2);
  p.rec = with_rec ? c.take<FwdRec>(total_n + 1) : nullptr;
  p.bytes = c.used();
  return p;
}

template <int THREADS>
int launch_count(const tc_batch* b, const BatchPlan& p, int64_t nslots, int piece, int blocks_per_cu, int64_t* T,
                 int64_t* H, int64_t* H2, hipStream_t s, bool wide = false) {
  const bool by_xcd = nslots >= 4 * kXcds * kXcdRun;
  int64_t blocks = by_xcd ? (nslots + kXcds * kXcdRun - 1) / (kXcds * kXcdRun) * (kXcds * kXcdRun) : nslots;
  if (blocks_per_cu > 0) blocks = std::min<int64_t>(blocks, 8 * ((static_cast<int64_t>(num_cus()) * blocks_per_cu + 7) / 8));
  blocks = std::min<int64_t>(blocks, int64_t(1) << 23);  // far below 2^32 work-items; a multiple of 8
  if (wide)
    batch_count_kernel<THREADS, true, true><<<static_cast<unsigned>(blocks), THREADS, 0, s>>>(
        b->vbase, b->row_offsets, b->cols, b->total_nnz, p.parity, p.rec, p.pieces, nslots, piece, by_xcd, T, H, H2);
  else if (p.rec)
    batch_count_kernel<THREADS, true, false><<<static_cast<unsigned>(blocks), THREADS, 0, s>>>(
        b->vbase, b->row_offsets, b->cols, b->total_nnz, p.parity, p.rec, p.pieces, nslots, piece, by_xcd, T, H, H2);
  else
    batch_count_kernel<THREADS, false, false><<<static_cast<unsigned>(blocks), THREADS, 0, s>>>(
        b->vbase, b->row_offsets, b->cols, b->total_nnz, p.parity, p.rec, p.pieces, nslots, piece, by_xcd, T, H, H2);
  TC_HIP(hipGetLastError());
  return TC_OK;
}

// The launches of a batch (tuning checked here, validation done by the
// caller); one: the one-graph path's vertex bases and statistics, written
// first, and H2 (nullable) receives |H| of all graphs.
int batch_launch(const tc_batch* b, const tc_tuning* t, int64_t* triangles, int64_t* h_count, int32_t* levels,
                 void* ws, size_t ws_bytes, hipStream_t s, int32_t root0, bool with_rec, OneGraph one, int64_t* H2) {
  const int G = b->num_graphs;
  int piece = auto_piece(b->total_nnz), bpc = 0;
  // one wave per piece while a piece is a handful of edges, else four
  int threads = piece < 128 ? kWave : 256;
  if (t) {
    if (t->batch_piece) {
      piece = t->batch_piece;
      threads = 256;
      if (piece < kPieceMin) return fail(TC_ERR_INVALID_ARG, "tc_count_batch: batch_piece must be >= %d", kPieceMin);
    }
    if (t->batch_block) threads = t->batch_block;
    bpc = t->batch_blocks_per_cu;
  }
  if (threads != kWave && threads != 256 && threads != 512)
    return fail(TC_ERR_INVALID_ARG, "tc_count_batch: batch_block must be 64, 256 or 512 (got %d)", threads);
  BatchPlan p = plan_batch(ws, b->total_vertices, b->total_nnz, G, with_rec);
  if (ws_bytes < p.bytes) return fail(TC_ERR_WORKSPACE, "tc_count_batch: workspace %zu < %zu", ws_bytes, p.bytes);
  const int64_t nslots = b->total_nnz / piece + G + 2;
  prof_stage("batch_bfs");
  const int64_t work = std::max<int64_t>(nslots, with_rec ? b->total_vertices : 0);
  // one launch where the preparation finds CUs beside the levels' blocks
  // (their LDS allows one a CU): R-MAT scale 10 takes 18 us so instead of
  // 12.5 + 5.7 in a row and the gap between
  if (with_rec && (one.vbase || (G <= 128 && work <= 128 * kBfsThreads))) {
    const unsigned blocks = static_cast<unsigned>(G) + grid_for(work, kBfsThreads);
    batch_first_kernel<<<blocks, kBfsThreads, 0, s>>>(b->vbase, G, b->row_offsets, b->cols, b->total_vertices, nslots,
                                                      piece, p.rec, p.pieces, one, levels, p.parity, triangles,
                                                      h_count, root0);
    TC_HIP(hipGetLastError());
  } else {
    const unsigned blocks = grid_for(work, 256, 16384);
    if (with_rec)
      batch_prep_kernel<true><<<blocks, 256, 0, s>>>(b->vbase, G, b->row_offsets, b->cols, b->total_vertices, nslots,
                                                     piece, p.rec, p.pieces, one);
    else
      batch_prep_kernel<false><<<blocks, 256, 0, s>>>(b->vbase, G, b->row_offsets, b->cols, b->total_vertices, nslots,
                                                      piece, p.rec, p.pieces, one);
    TC_HIP(hipGetLastError());
    batch_bfs_kernel<<<static_cast<unsigned>(G), kBfsThreads, 0, s>>>(b->vbase, b->row_offsets, b->cols, levels,
                                                                      p.parity, triangles, h_count);
    TC_HIP(hipGetLastError());
  }
  prof_stage("batch_count");
  if (threads == kWave) return launch_count<kWave>(b, p, nslots, piece, bpc, triangles, h_count, H2, s);
  if (threads == 256) return launch_count<256>(b, p, nslots, piece, bpc, triangles, h_count, H2, s);
  return launch_count<512>(b, p, nslots, piece, bpc, triangles, h_count, H2, s);
}

}  // namespace

size_t batch_ws_bytes(int64_t total_n, int64_t total_nnz, int32_t num_graphs, bool with_rec) {
  return plan_batch(nullptr, total_n, total_nnz, num_graphs, with_rec).bytes;
}

int batch_run(const tc_batch* b, const tc_tuning* t, uint32_t flags, int64_t* triangles, int64_t* h_count,
              int32_t* levels, void* ws, size_t ws_bytes, hipStream_t s, bool with_rec) {
  if (b->num_graphs == 0) return TC_OK;
  if (flags & TC_VALIDATE) TC_TRY(validate_batch_run(b, ws, s));
  return batch_launch(b, t, triangles, h_count, levels, ws, ws_bytes, s, -1, with_rec, OneGraph{}, nullptr);
}

namespace {

struct SmallPlan {
  int64_t* stats;  // the tc_stats mirror, first in the workspace like the count plan's
  int64_t* vbase;  // {0, n}
  char* batch;
  size_t bytes;
};

SmallPlan plan_small(void* base, int64_t n, int64_t nnz) {
  SmallPlan p;
  Carver c(base);
  p.stats = c.take<int64_t>(24);
  p.vbase = c.take<int64_t>(2);
  p.batch = c.take<char>(0);
  p.bytes = c.used() + batch_ws_bytes(n, nnz, 1, true);
  return p;
}

}  // namespace

size_t small_ws_bytes(int64_t n, int64_t nnz) { return plan_small(nullptr, n, nnz).bytes; }

bool small_path_fits(int64_t n, int64_t nnz, int64_t max_n, int64_t max_nnz) {
  return n > 0 && n <= TC_BATCH_MAX_N && n <= max_n && nnz <= max_nnz;
}

int small_count_run(const tc_csr* g, int64_t root, int64_t* triangles, int64_t* h_count, int32_t* levels, void* ws,
                    size_t ws_bytes, hipStream_t s) {
  SmallPlan p = plan_small(ws, g->n, g->nnz);
  if (ws_bytes < p.bytes) return fail(TC_ERR_WORKSPACE, "tc_count: workspace %zu < %zu", ws_bytes, p.bytes);
  prof_stage("small_count");
  tc_batch b;
  b.num_graphs = 1;
  b.total_vertices = g->n;
  b.total_nnz = g->nnz;
  b.vbase = p.vbase;
  b.row_offsets = g->row_offsets;
  b.cols = g->cols;
  b.max_graph_vertices = static_cast<int32_t>(g->n);
  // |H| of the statistics (tc_stats::h) is summed beside the caller's
  return batch_launch(&b, nullptr, triangles, h_count, levels, p.batch, p.bytes - (p.batch - static_cast<char*>(ws)), s,
                      static_cast<int32_t>(root), true, OneGraph{p.vbase, p.stats, g->n, g->nnz}, p.stats + 2);
}

// ------------------------------------------------ one graph, levels known
namespace {

struct DirectPlan {
  int64_t* vbase;
  int64_t* sums;
  BatchPlan batch;
  size_t bytes;
};

DirectPlan plan_direct(void* base, int64_t n, int64_t nnz) {
  DirectPlan p;
  Carver c(base);
  p.vbase = c.take<int64_t>(2);
  p.sums = c.take<int64_t>(kSumStripes * kSumPad);
  char* at = c.take<char>(0);
  p.batch = plan_batch(at, n, nnz, 1, true);
  p.bytes = c.used() + p.batch.bytes;
  return p;
}

__global__ __launch_bounds__(kWave) void direct_sum_kernel(const int64_t* sums, int64_t* T, int64_t* H, int64_t* stats) {
  static_assert(kSumStripes <= kWave, "a lane per stripe");
  const bool one = lane() < kSumStripes;
  const int64_t t = wave_sum(one ? sums[lane() * kSumPad] : int64_t(0));
  const int64_t h = wave_sum(one ? sums[lane() * kSumPad + 1] : int64_t(0));
  if (lane() != 0) return;
  *T = t;
  if (H) *H = h;
  stats[2] = h;
}

}  // namespace

size_t direct_ws_bytes(int64_t n, int64_t nnz) { return plan_direct(nullptr, n, nnz).bytes; }

int direct_count_run(const tc_csr* g, const int32_t* L, const BfsInfo& info, int64_t* stats, int64_t* triangles,
                     int64_t* h_count, void* ws, hipStream_t s) {
  DirectPlan p = plan_direct(ws, g->n, g->nnz);
  tc_batch b;
  b.num_graphs = 1;
  b.total_vertices = g->n;
  b.total_nnz = g->nnz;
  b.vbase = p.vbase;
  b.row_offsets = g->row_offsets;
  b.cols = g->cols;
  b.max_graph_vertices = 0;
  const int piece = auto_piece(g->nnz);
  const int64_t nslots = g->nnz / piece + 1 + 2;
  prof_stage("direct_prep");
  batch_prep_kernel<true><<<grid_for(std::max(nslots, g->n), 256, 16384), 256, 0, s>>>(
      p.vbase, 1, g->row_offsets, g->cols, g->n, nslots, piece, p.batch.rec, p.batch.pieces,
      OneGraph{p.vbase, stats, g->n, g->nnz, L, info.num_levels, p.batch.parity, p.sums});
  TC_HIP(hipGetLastError());
  prof_stage("direct_count");
  TC_TRY(launch_count<256>(&b, p.batch, nslots, piece, 0, p.sums, p.sums + 1, nullptr, s, true));
  direct_sum_kernel<<<1, kWave, 0, s>>>(p.sums, triangles, h_count, stats);
  TC_HIP(hipGetLastError());
  return TC_OK;
}

}  // namespace tc

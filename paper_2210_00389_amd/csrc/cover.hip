// cover.hip -- tc_cover_edges: the horizontal edges of a level function as a
// list.  In the order of the CSR entries they are a stream compaction: entry
// (x, y) is taken if y > x and the levels agree, so the list needs no
// counts per vertex.  A tile of kTile entries is one block's, whatever rows
// it holds: rows are marked at their first entry and every thread takes
// kItems consecutive entries.
//   1. prep: levels as bytes (a million of them stay in one XCD's 4 MB of L2,
//      where int32 levels do not), the first row of every tile;
//   2. mark: a bit per entry, a count per tile;
//   3. scan of the counts, and the list from the bits.
// Bound by the level gathers of the forward entries.  G(1000003, d 16), 16 M
// entries: the list through a full level-class layout (all entries classified
// and moved, a 32-byte record a row, then the runs of equal level copied)
// took 0.31 ms, this takes 0.10 ms (mark 64 us, list 27 us).
#include "tc_internal.h"

namespace tc {

namespace {

constexpr int kThreads = 256;
constexpr int kItems = 8;
constexpr int kTile = kThreads * kItems;
constexpr int kPrepBlocks = 1024;
constexpr int kManyRows = 8 * kTile;  // rows of a tile (nearly all empty) beyond which its entries search theirs

struct CoverWs {
  uint8_t* lev8;      // levels modulo 256
  int32_t* wide;      // [kPrepBlocks]: a level outside 0..255 was seen
  int32_t* tile_row;  // [tiles]: row of a tile's first entry
  int32_t* tile_cnt;  // list entries of a tile
  int64_t* tile_off;  // their scan
  uint8_t* bits;      // a byte for the kItems entries of a thread
  char* scratch;
  size_t bytes;
};

CoverWs plan_cover(void* base, int64_t n, int64_t nnz) {
  CoverWs w;
  Carver c(base);
  const int64_t tiles = (nnz + kTile - 1) / kTile;
  w.lev8 = c.take<uint8_t>(n + 1);
  w.wide = c.take<int32_t>(kPrepBlocks);
  w.tile_row = c.take<int32_t>(tiles + 2);
  w.tile_cnt = c.take<int32_t>(tiles + 1);
  w.tile_off = c.take<int64_t>(tiles + 2);
  w.bits = c.take<uint8_t>(tiles * kThreads + 1);
  w.scratch = c.take<char>(scan_ws_bytes(tiles + 1));
  w.bytes = c.used();
  return w;
}

__global__ __launch_bounds__(kThreads) void cover_prep_kernel(const int64_t* off, const int32_t* L, int64_t n,
                                                              int64_t tiles, uint8_t* lev8, int32_t* wide,
                                                              int32_t* tile_row) {
  int w = 0;
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
    const int32_t l = L[v];
    lev8[v] = static_cast<uint8_t>(l);
    w |= l < 0 || l > 255;
    const int64_t b = off[v], e = off[v + 1];
    const int64_t t1 = min(tiles, (e + kTile - 1) / kTile);
    for (int64_t t = v == 0 ? 0 : (b + kTile - 1) / kTile; t < t1; ++t) tile_row[t] = static_cast<int32_t>(v);
  }
  w = __syncthreads_or(w);
  if (threadIdx.x == 0) wide[blockIdx.x] = w;
}

struct TileLds {
  uint8_t beg[kThreads];  // bits of the entries that begin a row, a byte per thread
  int32_t own[kTile];     // there: the row, from the tile's first one
  int last[kThreads / kWave];
};

// The entries of the block's tile that lie in a row, [from, tn) of its kTile (tn
// = 0: none), and its first and last row.  The offsets may begin after 0 and end
// before nnz (a column buffer with room to spare): the tiles past their end
// have no row, and what tile_row holds there is not used.
struct TileRange {
  int64_t t0;
  int from, tn;
  int32_t r0, r1;
};
__device__ __forceinline__ TileRange tile_range(const int64_t* off, int64_t n, const int32_t* tile_row, int64_t nnz) {
  TileRange r;
  r.t0 = blockIdx.x * static_cast<int64_t>(kTile);
  const int64_t end = min(nnz, off[n]) - r.t0, tile = kTile;
  r.from = static_cast<int>(min(max(off[0] - r.t0, static_cast<int64_t>(0)), tile));
  r.tn = static_cast<int>(min(max(end, static_cast<int64_t>(0)), tile));
  const int32_t a = tile_row[blockIdx.x], z = tile_row[blockIdx.x + 1];
  r.r0 = r.tn > 0 ? a : 0;
  r.r1 = end > tile ? z : static_cast<int32_t>(n - 1);
  return r;
}

// Rows of the thread's entries (tile t0 .. t0 + tn).  Contains __syncthreads.
__device__ __forceinline__ void tile_rows(TileLds& s, const int64_t* off, int32_t r0, int32_t r1, int64_t t0, int tn,
                                          int32_t (&x)[kItems]) {
  const int tid = threadIdx.x, w = tid / kWave, ln = lane();
  if (r1 - r0 > kManyRows) {  // uniform: a long run of empty rows
    int64_t next = 0;
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      const int64_t p = t0 + min(tid * kItems + q, tn - 1);
      x[q] = q ? x[q - 1] : 0;
      if (q == 0 || p >= next) {
        x[q] = max(r0, static_cast<int32_t>(upper_bound_dev(off, static_cast<int64_t>(r0), static_cast<int64_t>(r1) + 1, p)) - 1);
        next = off[x[q] + 1];
      }
    }
    return;
  }
  s.beg[tid] = tid == 0 ? 1 : 0;
  if (tid == 0) s.own[0] = 0;
  __syncthreads();
  for (int32_t r = r0 + 1 + tid; r <= r1; r += kThreads) {
    const int64_t b = off[r] - t0;
    if (b >= tn || off[r + 1] - t0 <= b) continue;
    s.own[b] = r - r0;
    atomicOr(reinterpret_cast<uint32_t*>(s.beg) + b / 32, 1u << (b % 32));
  }
  __syncthreads();
  const uint32_t m = s.beg[tid];
  // the last mark before the thread's entries: in the wave, or in the waves before
  const uint64_t some = __ballot(m != 0u);
  const int mine = m ? tid * kItems + 31 - __clz(m) : 0;
  if (ln == 0) s.last[w] = 0;
  if (m && (some >> ln) == 1ull) s.last[w] = mine;
  __syncthreads();
  int at = 0;
#pragma unroll
  for (int q = 0; q < kThreads / kWave; ++q)
    if (q < w) at = max(at, s.last[q]);
  const uint64_t below = some & lanemask_lt();
  const int from = below ? 63 - __clzll(static_cast<long long>(below)) : 0;
  const int got = __shfl(mine, from, kWave);
  if (below) at = got;
  int32_t cur = r0 + s.own[at];
#pragma unroll
  for (int q = 0; q < kItems; ++q) {
    if ((m >> q) & 1u) cur = r0 + s.own[tid * kItems + q];
    x[q] = cur;
  }
}

__global__ __launch_bounds__(kThreads) void cover_mark_kernel(const int64_t* off, const int32_t* cols, int64_t n,
                                                              const int32_t* L, const uint8_t* lev8,
                                                              const int32_t* wide, int nwide, const int32_t* tile_row,
                                                              int64_t nnz, uint8_t* bits, int32_t* tile_cnt) {
  __shared__ TileLds s;
  __shared__ int32_t sh[kThreads / kWave + 1];
  const int tid = threadIdx.x;
  const int64_t t0 = blockIdx.x * static_cast<int64_t>(kTile);
  int32_t y[kItems], x[kItems];
#pragma unroll
  for (int q = 0; q < kItems; ++q) y[q] = t0 + tid * kItems + q < nnz ? cols[t0 + tid * kItems + q] : -1;
  const TileRange r = tile_range(off, n, tile_row, nnz);
  if (r.tn == 0) {  // uniform
    bits[blockIdx.x * static_cast<int64_t>(kThreads) + tid] = 0;
    if (tid == 0) tile_cnt[blockIdx.x] = 0;
    return;
  }
#pragma unroll
  for (int q = 0; q < kItems; ++q)
    if (tid * kItems + q < r.from || tid * kItems + q >= r.tn) y[q] = -1;
  int wd = 0;
  for (int i = tid; i < nwide; i += kThreads) wd |= wide[i];
  wd = __syncthreads_or(wd);
  tile_rows(s, off, r.r0, r.r1, r.t0, r.tn, x);
  uint32_t take = 0;
  auto mark = [&](const auto* lev) {
    int32_t lx[kItems], ly[kItems];
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      lx[q] = q && x[q] == x[q - 1] ? lx[q - 1] : static_cast<int32_t>(lev[x[q]]);
      ly[q] = y[q] > x[q] ? static_cast<int32_t>(lev[y[q]]) : 0;
    }
#pragma unroll
    for (int q = 0; q < kItems; ++q) take |= static_cast<uint32_t>(y[q] > x[q] && ly[q] == lx[q]) << q;
  };
  if (wd) mark(L);  // bytes do not tell these levels apart
  else mark(lev8);
  bits[blockIdx.x * static_cast<int64_t>(kThreads) + tid] = static_cast<uint8_t>(take);
  const int32_t c = block_sum(static_cast<int32_t>(__popc(take)), sh);
  if (tid == 0) tile_cnt[blockIdx.x] = c;
}

__global__ __launch_bounds__(kThreads) void cover_emit_kernel(const int64_t* off, const int32_t* cols, int64_t n,
                                                              const int32_t* tile_row, int64_t nnz,
                                                              const uint8_t* bits, const int64_t* tile_off,
                                                              int64_t cap, int32_t* h_u, int32_t* h_v,
                                                              int64_t* h_count) {
  __shared__ TileLds s;
  __shared__ int2 s_out[kTile];
  __shared__ int32_t sh[kThreads / kWave + 1];
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && tid == 0) *h_count = tile_off[gridDim.x];
  const TileRange r = tile_range(off, n, tile_row, nnz);
  if (r.tn == 0) return;  // uniform
  const uint32_t take = bits[blockIdx.x * static_cast<int64_t>(kThreads) + tid];
  int32_t y[kItems], x[kItems];
#pragma unroll
  for (int q = 0; q < kItems; ++q) y[q] = (take >> q) & 1u ? cols[r.t0 + tid * kItems + q] : 0;
  tile_rows(s, off, r.r0, r.r1, r.t0, r.tn, x);
  int32_t total;
  int32_t at = block_excl_scan(static_cast<int32_t>(__popc(take)), sh, &total);
#pragma unroll
  for (int q = 0; q < kItems; ++q)
    if ((take >> q) & 1u) s_out[at++] = make_int2(x[q], y[q]);
  __syncthreads();
  const int64_t o = tile_off[blockIdx.x];
  for (int i = tid; i < total && o + i < cap; i += kThreads) {
    h_u[o + i] = s_out[i].x;
    h_v[o + i] = s_out[i].y;
  }
}

}  // namespace

size_t cover_ws_bytes(int64_t n, int64_t nnz) { return plan_cover(nullptr, n, nnz).bytes; }

int cover_run(const tc_csr* g, const int32_t* levels, int32_t* h_u, int32_t* h_v, int64_t cap, int64_t* h_count,
              void* ws, hipStream_t s) {
  const int64_t n = g->n, nnz = g->nnz, tiles = (nnz + kTile - 1) / kTile;
  if (n == 0 || nnz == 0) return fill_i64(h_count, 0, 1, s);
  CoverWs w = plan_cover(ws, n, nnz);
  const unsigned prep = grid_for(n, kThreads, kPrepBlocks);
  cover_prep_kernel<<<prep, kThreads, 0, s>>>(g->row_offsets, levels, n, tiles, w.lev8, w.wide, w.tile_row);
  cover_mark_kernel<<<static_cast<unsigned>(tiles), kThreads, 0, s>>>(g->row_offsets, g->cols, n, levels, w.lev8, w.wide,
                                                                      static_cast<int>(prep), w.tile_row, nnz, w.bits,
                                                                      w.tile_cnt);
  TC_HIP(hipGetLastError());
  {
    Carver sc(w.scratch);
    TC_TRY(scan_exclusive<int32_t>(w.tile_cnt, w.tile_off, tiles, sc, s));
  }
  cover_emit_kernel<<<static_cast<unsigned>(tiles), kThreads, 0, s>>>(g->row_offsets, g->cols, n, w.tile_row, nnz, w.bits,
                                                                      w.tile_off, cap, h_u, h_v, h_count);
  TC_HIP(hipGetLastError());
  return TC_OK;
}

}  // namespace tc

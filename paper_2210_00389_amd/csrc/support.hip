// support.hip -- triangles per edge (the support of k-truss decompositions)
// from a list of triangles: each triangle adds one to its three edges.
//
// The additions go to the entry (u, v), u < v, of an edge; a second pass
// copies every sum to the entry (v, u), one search per edge instead of three
// searches and atomics per triangle (short lists add to both, see kFew).
//
// Atomics to memory bound it (six a triangle, the hubs' edges on the same
// addresses: 3.8 ms for the 15.6 M triangles of R-MAT scale 16).  A triangle
// list comes in runs with a common vertex (tc_list_triangles: an anchor's),
// whose two edges repeat through the run: a wave takes the vertex shared by
// its first and last triangle, and the edges at that vertex are summed by
// their two ids in a table of the block in LDS, so that they are searched and
// added once a block.  The same triangles then take 0.76 ms, 31 G atomics a
// second (0.84 with positions as keys, which every triangle had to search,
// 1.7 without the table, 1.0 with all three edges in it: the third edge rarely
// repeats and takes the slots; a table of 4096 edges 0.99, of 1024 for 1024
// triangles 0.78).
#include "tc_internal.h"

namespace tc {

namespace {

constexpr int kThreads = 256;
constexpr int kTri = 2048;      // consecutive triangles of a block at most
constexpr int kTable = 2048;    // edges summed in LDS (24 KB)
constexpr int kProbes = 4;      // slots an edge may take
// Lists of up to kFew triangles are added one by one, without the table; lists
// of up to a fifth of the entries add to both orientations, since the mirror
// pass over all entries takes longer than their second searches.  us, all
// lists with the mirror pass and shares of kTri / so: 1 triangle on
// G(1000003, d 16) 612 / 28; R-MAT scale 20, 31.4 M entries, 65536 triangles
// 1911 / 77 (122 with the table), 131072 1907 / 92 (118), 0.49 M 1945 / 209, 2.0
// M 2061 / 540.  Near the line a list as it is written gains what one in random
// order loses (mirror pass / both): at an eighth of the entries 2319 / 1163 and
// 3619 / 4123, a fifth 2521 / 1658 and 4775 / 6718, a quarter 2596 / 1975 and
// 5612 / 8477; a wheel of 10^6 vertices at a quarter 191 / 123 and 322 / 357.
constexpr int64_t kFew = 131072, kMirrorRatio = 5;
constexpr unsigned long long kFree = ~0ull;

__device__ __forceinline__ void order2(int32_t& x, int32_t& y) {
  const int32_t t = min(x, y);
  y = max(x, y);
  x = t;
}

// Adds s[q] to the entry (u[q], v[q]) where there is one, and to (v[q], u[q])
// if kBoth, N searches advancing together (s[q] = 0: none).
template <bool kBoth, int N>
__device__ __forceinline__ void add_edges(const int64_t* off, const int32_t* cols, const int32_t (&u)[N],
                                          const int32_t (&v)[N], const int32_t (&s)[N], int32_t* sup) {
  int64_t lo[N], hi[N], end[N];
#pragma unroll
  for (int q = 0; q < N; ++q) lo[q] = s[q] ? off[u[q]] : 0;
#pragma unroll
  for (int q = 0; q < N; ++q) hi[q] = end[q] = s[q] ? off[u[q] + 1] : 0;
  for (;;) {
    int32_t m[N];
    bool any = false;
#pragma unroll
    for (int q = 0; q < N; ++q) m[q] = lo[q] < hi[q] ? cols[lo[q] + ((hi[q] - lo[q]) >> 1)] : 0;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      if (lo[q] >= hi[q]) continue;
      const int64_t mid = lo[q] + ((hi[q] - lo[q]) >> 1);
      if (m[q] < v[q]) lo[q] = mid + 1;
      else hi[q] = mid;
      any |= lo[q] < hi[q];
    }
    if (!any) break;
  }
#pragma unroll
  for (int q = 0; q < N; ++q)
    if (lo[q] < end[q] && cols[lo[q]] == v[q]) atomicAdd(&sup[lo[q]], s[q]);
  if constexpr (kBoth) add_edges<false, N>(off, cols, v, u, s, sup);
}

template <bool kBoth>
__global__ __launch_bounds__(kThreads) void support_kernel(const int64_t* off, const int32_t* cols, int64_t n,
                                                           const int32_t* tri, int64_t ntri, int share, int32_t* sup) {
  __shared__ unsigned long long s_key[kTable];  // u << 32 | v
  __shared__ int32_t s_sum[kTable];
  const bool plain = kBoth && ntri <= kFew;
  auto keep = [&](int32_t u, int32_t v) {
    const unsigned long long key = (static_cast<unsigned long long>(static_cast<uint32_t>(u)) << 32) |
                                   static_cast<uint32_t>(v);
    uint32_t slot = ((static_cast<uint32_t>(u) * 0x85EBCA6Bu + static_cast<uint32_t>(v)) * 0x9E3779B1u) >>
                    (32 - __builtin_ctz(kTable));
    for (int q = 0; q < kProbes; ++q) {
      const unsigned long long was = atomicCAS(&s_key[slot], kFree, key);
      if (was == kFree || was == key) {
        atomicAdd(&s_sum[slot], 1);
        return true;
      }
      slot = (slot + 1) & (kTable - 1);
    }
    return false;
  };
  for (int64_t t0 = blockIdx.x * static_cast<int64_t>(share); t0 < ntri; t0 += static_cast<int64_t>(gridDim.x) * share) {
    for (int i = threadIdx.x; i < (plain ? 0 : kTable); i += kThreads) {
      s_key[i] = kFree;
      s_sum[i] = 0;
    }
    __syncthreads();
    const int64_t t1 = min(t0 + share, ntri);
    for (int64_t w0 = t0 + (threadIdx.x & ~(kWave - 1)); w0 < t1; w0 += kThreads) {  // uniform per wave
      const int64_t i = w0 + lane();
      int32_t a = -1, b = -1, c = -1;
      if (i < t1) {
        a = tri[3 * i];
        b = tri[3 * i + 1];
        c = tri[3 * i + 2];
      }
      // the vertex shared by the wave's first and last triangle (-1: none)
      const int z = static_cast<int>(min(t1 - w0, static_cast<int64_t>(kWave))) - 1;
      const int32_t za = wave_read(a, z), zb = wave_read(b, z), zc = wave_read(c, z);
      int32_t x = -1;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const int32_t f = wave_read(q == 0 ? a : (q == 1 ? b : c), 0);
        if (f == za || f == zb || f == zc) x = f;
      }
      // ids outside [0, n) would index rows that do not exist: such a triple is skipped
      if (a < 0 || b < 0 || c < 0 || a >= n || b >= n || c >= n) continue;
      order2(a, b);
      order2(b, c);
      order2(a, b);
      if (plain || x < 0) {  // uniform
        const int32_t u[3] = {a, a, b}, v[3] = {b, c, c};
        int32_t some[3] = {1, 1, 1};
        if (plain) {  // an edge that all triangles of the wave have is added once
          const uint64_t in = __ballot(true);
          const int first = __ffsll(static_cast<unsigned long long>(in)) - 1;
#pragma unroll
          for (int q = 0; q < 3; ++q)
            if (__ballot(u[q] == wave_read(u[q], first) && v[q] == wave_read(v[q], first)) == in)
              some[q] = lane() == first ? __popcll(in) : 0;
        }
        add_edges<kBoth, 3>(off, cols, u, v, some, sup);
        continue;
      }
      uint32_t left = 7u;  // edges not kept
      if ((a == x || b == x) && keep(a, b)) left &= ~1u;
      if ((a == x || c == x) && keep(a, c)) left &= ~2u;
      if ((b == x || c == x) && keep(b, c)) left &= ~4u;
      while (left) {  // mostly one
        const bool ab = (left & 1u) != 0u, ac = !ab && (left & 2u) != 0u;
        left &= left - 1;
        const int32_t u[1] = {ab || ac ? a : b}, v[1] = {ab ? b : c}, one[1] = {1};
        add_edges<kBoth, 1>(off, cols, u, v, one, sup);
      }
    }
    __syncthreads();
    if (plain) continue;
    constexpr int kAtOnce = 4;
    static_assert(kTable % (kThreads * kAtOnce) == 0, "whole rounds");
    for (int i = threadIdx.x; i < kTable; i += kThreads * kAtOnce) {
      int32_t u[kAtOnce], v[kAtOnce], s[kAtOnce];
#pragma unroll
      for (int q = 0; q < kAtOnce; ++q) {
        const unsigned long long key = s_key[i + q * kThreads];
        s[q] = s_sum[i + q * kThreads];
        u[q] = static_cast<int32_t>(key >> 32);
        v[q] = static_cast<int32_t>(key & 0xFFFFFFFFull);
      }
      add_edges<kBoth, kAtOnce>(off, cols, u, v, s, sup);
    }
    __syncthreads();
  }
}

// The entry (v, u), u < v, takes the sum of (u, v).  A wave takes kMirror
// consecutive entries: their first and last row are found once, and a lane
// looks for its entry's row between them (a hub's row of a wave of its own
// took 0.27 ms at R-MAT scale 16).
constexpr int kMirror = 512;

__global__ __launch_bounds__(kThreads) void mirror_kernel(const int64_t* off, const int32_t* cols, int64_t n,
                                                          int64_t nnz, int32_t* sup) {
  const int64_t nw = (int64_t)gridDim.x * (kThreads / kWave);
  const int64_t wid = blockIdx.x * static_cast<int64_t>(kThreads / kWave) +
                      __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t last = min(nnz, off[n]);
  for (int64_t j0 = wid * kMirror; j0 < last; j0 += nw * kMirror) {
    const int64_t j1 = min(j0 + kMirror, last);
    const int64_t r0 = upper_bound_dev(off, 0, n + 1, j0) - 1;  // the row holding entry j0
    const int64_t r1 = upper_bound_dev(off, r0, n + 1, j1 - 1);
    for (int64_t j = j0 + lane(); j < j1; j += kWave) {
      const int64_t v = upper_bound_dev(off, r0 + 1, r1, j) - 1;
      const int32_t u = cols[j];
      if (u >= v || u < 0) continue;
      const int64_t ue = off[u + 1], p = lower_bound_dev(cols, off[u], ue, static_cast<int32_t>(v));
      if (p < ue && cols[p] == v) sup[j] = sup[p];
    }
  }
}

}  // namespace

int support_run(const tc_csr* g, const int32_t* tri, int64_t ntri, int32_t* support, hipStream_t s) {
  TC_TRY(fill_i32(support, 0, g->nnz, s));
  if (ntri <= 0 || g->n == 0) return TC_OK;
  // short lists in smaller shares, so that they still fill the chip
  const int64_t even = (ntri / (4 * static_cast<int64_t>(num_cus())) + kThreads - 1) / kThreads * kThreads;
  const int share = static_cast<int>(std::min<int64_t>(std::max<int64_t>(even, kThreads), kTri));
  const unsigned blocks = grid_for(ntri, share, 65536);
  if (ntri <= std::max(kFew, g->nnz / kMirrorRatio)) {
    support_kernel<true><<<blocks, kThreads, 0, s>>>(g->row_offsets, g->cols, g->n, tri, ntri, share, support);
  } else {
    support_kernel<false><<<blocks, kThreads, 0, s>>>(g->row_offsets, g->cols, g->n, tri, ntri, share, support);
    mirror_kernel<<<grid_for(g->nnz, kMirror * (kThreads / kWave), 16384), kThreads, 0, s>>>(
        g->row_offsets, g->cols, g->n, g->nnz, support);
  }
  TC_HIP(hipGetLastError());
  return TC_OK;
}

}  // namespace tc

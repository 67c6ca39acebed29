// csr_build.hip -- raw pairs -> simple undirected CSR (the graph input of
// Sec. III, with both orientations and sorted rows).
//
// Every pair (s, d), s != d, becomes two keys (s << B) | d and (d << B) | s
// with B = bits(n - 1); loops become an all-ones sentinel that sorts last.
// An LSD radix sort orders the keys by digits of at most 8 bits (five passes
// of 8 for 2^20 vertices); its first pass takes the keys straight from the
// pairs.  Each pass is a per-tile digit histogram, a device scan of the
// digit-major histogram, and a stable scatter.  Of the sorted keys the first
// of each run of equal ones gives an entry of cols (its low B bits), and the
// first entry of a row its offset.
#include "tc_internal.h"

namespace tc {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kItems = 16;                       // keys per thread
constexpr int kPart = kItems * kWave;            // keys of one wave, consecutive
constexpr int64_t kTile = kThreads * kItems;     // 4096 keys per tile
constexpr int kMaxBits = 8;
constexpr int kRadix = 1 << kMaxBits;
constexpr uint64_t kSentinel = ~0ull;

// Where a pass reads key i, and which key a lane takes in round j of its
// wave's part.  A pass over an array takes 64 consecutive keys a round, in
// order (the sort is stable); the first pass, whose order is free, takes both
// keys of a pair in one lane, so that every pair is loaded once.  A pair with
// an id outside [0, n) sets *bad (where given) and counts as a loop, so that
// nothing after it indexes with it.
struct KeyArray {
  const uint64_t* keys;
  static __device__ __forceinline__ int64_t index(int64_t part, int j) { return part + j * kWave + lane(); }
  __device__ __forceinline__ uint64_t operator()(int64_t i) const { return keys[i]; }
};
struct KeyPairs {
  const int32_t* src;
  const int32_t* dst;
  uint32_t n;
  int B;
  int32_t* bad;
  static __device__ __forceinline__ int64_t index(int64_t part, int j) {
    return part + (j >> 1) * (2 * kWave) + 2 * lane() + (j & 1);
  }
  __device__ __forceinline__ uint64_t operator()(int64_t i) const {
    const uint32_t s = static_cast<uint32_t>(src[i >> 1]), d = static_cast<uint32_t>(dst[i >> 1]);
    if (s >= n || d >= n) {
      if (bad) atomicOr(bad, 1);
      return kSentinel;
    }
    if (s == d) return kSentinel;
    return (i & 1) ? (static_cast<uint64_t>(d) << B) | s : (static_cast<uint64_t>(s) << B) | d;
  }
};

// Digit counts of a tile, digit-major.  Each wave counts in a histogram of
// its own: the digits of a hub's row meet on one address.
template <class Src>
__global__ __launch_bounds__(kThreads) void hist_kernel(Src src, int64_t N, int shift, int bits, int64_t nblocks,
                                                        int32_t* ghist) {
  __shared__ int32_t h[kWaves][kRadix];
  const int w = threadIdx.x / kWave, radix = 1 << bits;
  for (int i = threadIdx.x; i < kWaves * kRadix; i += kThreads) (&h[0][0])[i] = 0;
  __syncthreads();
  const int64_t part = blockIdx.x * kTile + w * kPart;
  uint64_t key[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = Src::index(part, j);
    key[j] = i < N ? src(i) : 0;
  }
#pragma unroll
  for (int j = 0; j < kItems; ++j)
    if (Src::index(part, j) < N) atomicAdd(&h[w][(key[j] >> shift) & (radix - 1)], 1);
  __syncthreads();
  for (int d = threadIdx.x; d < radix; d += kThreads) {
    int32_t c = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) c += h[q][d];
    ghist[d * nblocks + blockIdx.x] = c;
  }
}

// Stable scatter of a tile.  A wave ranks its 1024 consecutive keys round by
// round (the lanes of one digit are the AND of the digit's ballots; counts in
// the wave's own LDS row, so a round needs no barrier), the tile is put in
// digit order in LDS, and the digits' runs (16 keys on average) are written
// whole: with every key stored from its own lane, each store instruction
// touched 64 lines and a pass over 33.5 M keys took 345 us; this one takes
// 170 us (3.2 TB/s), its histogram 68 us (3.9 TB/s).
template <class Src>
__global__ __launch_bounds__(kThreads) void scatter_kernel(Src src, int64_t N, int shift, int bits, int64_t nblocks,
                                                           const int64_t* gpos, uint64_t* out) {
  __shared__ uint64_t s_key[kTile];
  __shared__ int32_t s_cnt[kWaves][kRadix];
  __shared__ int64_t s_to[kRadix];  // output position of a digit's run less its place in the tile
  __shared__ int32_t sh[kWaves + 1];
  const int tid = threadIdx.x, w = tid / kWave, radix = 1 << bits;
  const uint64_t lt = lanemask_lt();
  const int64_t tile0 = blockIdx.x * kTile;
  const int64_t part = tile0 + w * kPart;
  uint64_t key[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = Src::index(part, j);
    key[j] = i < N ? src(i) : 0;
  }
  for (int i = lane(); i < kRadix; i += kWave) s_cnt[w][i] = 0;
  const int64_t run0 = tid < radix ? gpos[tid * nblocks + blockIdx.x] : 0;
  int32_t rank[kItems];
  volatile int32_t* cnt = s_cnt[w];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const bool valid = Src::index(part, j) < N;
    const int dig = static_cast<int>((key[j] >> shift) & (radix - 1));
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (dig >> b) & 1;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    rank[j] = 0;
    if (valid) {
      const int32_t before = cnt[dig];
      rank[j] = before + __popcll(peers & lt);
      if ((peers & lt) == 0) cnt[dig] = before + __popcll(peers);
    }
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  {
    int32_t c[kWaves], sum = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) {
      c[q] = s_cnt[q][tid];
      sum += c[q];
    }
    int32_t tot;
    int32_t at = block_excl_scan(sum, sh, &tot);
    s_to[tid] = run0 - at;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) {
      s_cnt[q][tid] = at;
      at += c[q];
    }
  }
  static_assert(kRadix == kThreads, "one thread per digit");
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j)
    if (Src::index(part, j) < N) s_key[s_cnt[w][(key[j] >> shift) & (radix - 1)] + rank[j]] = key[j];
  __syncthreads();
  const int tn = static_cast<int>(min(kTile, N - tile0));
  for (int i = tid; i < tn; i += kThreads) {
    const uint64_t k = s_key[i];
    out[s_to[(k >> shift) & (radix - 1)] + i] = k;
  }
}

// The first key of a run of equal ones (loops excluded) becomes an entry.
__device__ __forceinline__ bool is_entry(const uint64_t* keys, int64_t i, int64_t N, uint64_t& k, uint64_t& prev) {
  k = i < N ? keys[i] : kSentinel;
  prev = i > 0 && i <= N ? keys[i - 1] : kSentinel;
  return k != kSentinel && (i == 0 || prev != k);
}

__global__ __launch_bounds__(kThreads) void entry_count_kernel(const uint64_t* keys, int64_t N, int32_t* tile_cnt) {
  __shared__ int32_t sh[kWaves + 1];
  const int64_t base = blockIdx.x * kTile + threadIdx.x;
  int32_t c = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    uint64_t k, prev;
    c += is_entry(keys, base + j * kThreads, N, k, prev);
  }
  c = block_sum(c, sh);
  if (threadIdx.x == 0) tile_cnt[blockIdx.x] = c;
}

// Entries of a tile at its scanned position; the first entry of a row writes
// the offsets of that row and of up to kGap empty rows before it (the rows
// after the last entry likewise, from the first sentinel or the end).  Rows
// of longer gaps keep -1 for gap_kernel.  A histogram of the rows with one
// atomic per entry took 2.98 ms for 33.5 M keys, the hubs' entries all on one
// address, in place of this kernel's 0.15 ms.
constexpr int kGap = 64;

__global__ __launch_bounds__(kThreads) void emit_kernel(const uint64_t* keys, int64_t N, const int64_t* tile_off, int B,
                                                        int64_t n, int32_t* cols, int64_t* row_offsets) {
  __shared__ int32_t s_w[kWaves];
  const int w = threadIdx.x / kWave;
  const uint64_t low = (1ull << B) - 1, lt = lanemask_lt();
  const int64_t base = blockIdx.x * kTile + w * kPart + lane();
  uint64_t key[kItems], mask[kItems];
  uint32_t first = 0;  // bit j: entry j starts a row (or the sentinels)
  int32_t prow[kItems];  // row of the key before
  int32_t c = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    uint64_t prev;
    const int64_t i = base + j * kWave;
    const bool e = is_entry(keys, i, N, key[j], prev);
    mask[j] = __ballot(e);
    c += __popcll(mask[j]);
    prow[j] = i == 0 ? -1 : static_cast<int32_t>(prev >> B);
    // the position just past the last entry closes the remaining rows
    const bool end = i <= N && key[j] == kSentinel && (i == 0 || prev != kSentinel);
    const int64_t row = end ? n : static_cast<int64_t>(key[j] >> B);
    if ((e && row != prow[j]) || end) first |= 1u << j;
  }
  if (lane() == 0) s_w[w] = c;
  __syncthreads();
  int64_t pos = tile_off[blockIdx.x];
  for (int q = 0; q < w; ++q) pos += s_w[q];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t at = pos + __popcll(mask[j] & lt);
    const bool end = key[j] == kSentinel;
    if ((mask[j] >> lane()) & 1ull) cols[at] = static_cast<int32_t>(key[j] & low);
    if ((first >> j) & 1u) {
      const int64_t row = end ? n : static_cast<int64_t>(key[j] >> B);
      const int64_t from = row - prow[j] > kGap ? row : static_cast<int64_t>(prow[j]) + 1;
      for (int64_t r = from; r <= row; ++r) row_offsets[r] = at;
    }
    pos += __popcll(mask[j]);
  }
}

// Rows of long gaps start where the next row with an entry does.
__global__ void gap_kernel(const uint64_t* keys, int64_t N, int B, int64_t n, int64_t* row_offsets) {
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    if (row_offsets[r] >= 0) continue;
    const int64_t i = lower_bound_dev(keys, 0, N, static_cast<uint64_t>(r) << B);
    row_offsets[r] = row_offsets[i < N && keys[i] != kSentinel ? static_cast<int64_t>(keys[i] >> B) : n];
  }
}

// count_src: the same keys for the histogram (the pairs are checked there).
template <class Src>
int radix_pass(const Src& count_src, const Src& src, int64_t N, int shift, int bits, char* scratch, uint64_t* out, hipStream_t s) {
  const int64_t nblocks = (N + kTile - 1) / kTile;
  const int radix = 1 << bits;
  Carver c(scratch);
  int32_t* ghist = c.take<int32_t>(kRadix * nblocks + 1);
  int64_t* gpos = c.take<int64_t>(kRadix * nblocks + 2);
  hist_kernel<Src><<<(unsigned)nblocks, kThreads, 0, s>>>(count_src, N, shift, bits, nblocks, ghist);
  TC_TRY(scan_exclusive<int32_t>(ghist, gpos, radix * nblocks, c, s));
  scatter_kernel<Src><<<(unsigned)nblocks, kThreads, 0, s>>>(src, N, shift, bits, nblocks, gpos, out);
  TC_HIP(hipGetLastError());
  return TC_OK;
}

// Digits of equal width (within one bit), at most kMaxBits each.
int digit_bits(int left) {
  const int passes = (left + kMaxBits - 1) / kMaxBits;
  return (left + passes - 1) / passes;
}

int bits_for(int64_t n) {
  int B = 1;
  while (B < 31 && (int64_t(1) << B) < n) ++B;
  return B;
}

}  // namespace

size_t radix_ws_bytes(int64_t N) {
  Carver c(nullptr);
  const int64_t nblocks = (N + kTile - 1) / kTile;
  c.take<int32_t>(kRadix * nblocks + 1);
  c.take<int64_t>(kRadix * nblocks + 2);
  c.take<char>(scan_ws_bytes(kRadix * nblocks + 1));
  return c.used();
}

int radix_sort_u64(uint64_t* keys, uint64_t* tmp, int64_t N, int bit_lo, int bit_hi, char* scratch,
                   hipStream_t s, uint64_t** result) {
  *result = keys;
  if (N <= 0) return TC_OK;
  for (int at = bit_lo; at < bit_hi;) {
    const int bits = digit_bits(bit_hi - at);
    const KeyArray src{*result};
    TC_TRY(radix_pass(src, src, N, at, bits, scratch, tmp, s));
    std::swap(*result, tmp);
    at += bits;
  }
  return TC_OK;
}

size_t build_ws_bytes(int64_t n, int64_t num_pairs) {
  Carver c(nullptr);
  const int64_t N = 2 * num_pairs;
  const int64_t tiles = N / kTile + 1;
  c.take<uint64_t>(N + 1);
  c.take<uint64_t>(N + 1);
  c.take<int32_t>(tiles + 1);
  c.take<int64_t>(tiles + 2);
  c.take<int32_t>(4);
  const size_t a = radix_ws_bytes(N), b = scan_ws_bytes(tiles + 1);
  c.take<char>(a > b ? a : b);
  return c.used();
}

int build_run(int64_t n, int64_t P, const int32_t* src, const int32_t* dst, int64_t* row_offsets,
              int32_t* cols, int64_t* nnz_out, void* ws, size_t ws_bytes, hipStream_t s) {
  if (ws_bytes < build_ws_bytes(n, P))
    return fail(TC_ERR_WORKSPACE, "tc_build_csr: workspace %zu < %zu bytes", ws_bytes, build_ws_bytes(n, P));
  const int64_t N = 2 * P;
  if (P == 0) {
    TC_TRY(fill_i64(row_offsets, 0, n + 1, s));
    TC_HIP(hipStreamSynchronize(s));
    *nnz_out = 0;
    return TC_OK;
  }
  Carver c(ws);
  // one position past the last key is looked at too: it closes the last rows
  const int64_t tiles = N / kTile + 1;
  uint64_t* ka = c.take<uint64_t>(N + 1);
  uint64_t* kb = c.take<uint64_t>(N + 1);
  int32_t* tile_cnt = c.take<int32_t>(tiles + 1);
  int64_t* tile_off = c.take<int64_t>(tiles + 2);
  int32_t* bad = c.take<int32_t>(4);
  char* scratch = c.take<char>(1);
  TC_TRY(fill_i32(bad, 0, 1, s));
  TC_TRY(fill_i64(row_offsets, -1, n + 1, s));
  const int B = bits_for(n);
  // the first pass reads the pairs; the check of their ids rides with its histogram
  const int bits0 = digit_bits(2 * B);
  const uint32_t un = static_cast<uint32_t>(n);
  TC_TRY(radix_pass(KeyPairs{src, dst, un, B, bad}, KeyPairs{src, dst, un, B, nullptr}, N, 0, bits0, scratch, ka, s));
  TC_TRY(radix_sort_u64(ka, kb, N, bits0, 2 * B, scratch, s, &ka));
  entry_count_kernel<<<(unsigned)tiles, kThreads, 0, s>>>(ka, N, tile_cnt);
  Carver sc(scratch);
  TC_TRY(scan_exclusive<int32_t>(tile_cnt, tile_off, tiles, sc, s));
  emit_kernel<<<(unsigned)tiles, kThreads, 0, s>>>(ka, N, tile_off, B, n, cols, row_offsets);
  gap_kernel<<<grid_for(n, kThreads, 16384), kThreads, 0, s>>>(ka, N, B, n, row_offsets);
  TC_HIP(hipGetLastError());
  int64_t nnz = 0;
  int32_t hbad = 0;
  TC_HIP(hipMemcpyAsync(&nnz, row_offsets + n, sizeof nnz, hipMemcpyDeviceToHost, s));
  TC_HIP(hipMemcpyAsync(&hbad, bad, sizeof hbad, hipMemcpyDeviceToHost, s));
  TC_HIP(hipStreamSynchronize(s));
  if (hbad) return fail(TC_ERR_OUT_OF_RANGE, "tc_build_csr: a pair has an id outside [0, %lld)", (long long)n);
  *nnz_out = nnz;
  return TC_OK;
}

}  // namespace tc

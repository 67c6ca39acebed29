// tc_common.h -- internal helpers shared by the libtc HIP sources (device
// primitives for 64-lane wavefronts, workspace carving, error plumbing).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/tc.h"

namespace tc {

constexpr int kWave = 64;

// ------------------------------------------------------------ errors
// Records the text of a failure for tc_last_error (thread-local) and returns
// the status.
int fail(int status, const char* fmt, ...);

#define TC_HIP(call)                                                         \
  do {                                                                       \
    hipError_t e_ = (call);                                                  \
    if (e_ != hipSuccess)                                                    \
      return ::tc::fail(TC_ERR_HIP, "%s failed: %s (%s:%d)", #call,          \
                        hipGetErrorString(e_), __FILE__, __LINE__);          \
  } while (0)

#define TC_TRY(expr)            \
  do {                          \
    int s_ = (expr);            \
    if (s_ != TC_OK) return s_; \
  } while (0)

// ----------------------------------------------------------- workspace
// Bump allocator over the caller's workspace.  With base == nullptr it only
// measures (used by tc_workspace_bytes), so sizing and carving share code.
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base(static_cast<char*>(b)) {}
  template <class T>
  T* take(size_t count) {
    size_t bytes = (count * sizeof(T) + 255) & ~size_t(255);
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += bytes;
    return p;
  }
  size_t used() const { return off; }
};

// --------------------------------------------------------- profiling
// Stage markers: when profiling is on, record an event pair per stage on the
// stream of the call (see tc_profile_read).
void prof_begin_call(hipStream_t s);
void prof_stage(const char* name);  // closes the previous stage, opens this one
void prof_end_call();

// Grid size for a grid-stride kernel over `work` items with `per_block`
// items per block, capped to keep launches reasonable.
inline unsigned grid_for(int64_t work, int per_block, unsigned cap = 1u << 20) {
  int64_t g = (work + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return static_cast<unsigned>(g);
}

int num_cus();

// Auxiliary streams (default priority) for fork/join concurrency inside one
// call, created once per host thread and device.
constexpr int kForkWays = 3;
struct Fork {
  hipStream_t aux[kForkWays];
  hipEvent_t fork;
  hipEvent_t join[kForkWays];
};
// Returns nullptr (and records the error) if streams/events cannot be made.
Fork* fork_for_device();
int fork_begin(Fork* f, hipStream_t s);  // aux streams wait for s
int fork_end(Fork* f, hipStream_t s);    // s waits for the aux streams

// ------------------------------------------------------ device helpers
__device__ __forceinline__ int lane() { return static_cast<int>(__lane_id()); }
__device__ __forceinline__ uint64_t lanemask_lt() { return __lanemask_lt(); }

// Moves a value between lanes with a DPP control (row shifts of 16 lanes,
// row broadcasts) where a shuffle would go through the LDS unit; a lane
// without a source, or outside RMASK's rows, keeps `old`.  All 64 lanes take
// part.
template <int CTRL, int RMASK, class T>
__device__ __forceinline__ T dpp_move(T old, T v) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two registers");
  if constexpr (sizeof(T) == 4) {
    return static_cast<T>(__builtin_amdgcn_update_dpp(static_cast<int>(old), static_cast<int>(v), CTRL, RMASK, 0xf, false));
  } else {
    const uint64_t o = static_cast<uint64_t>(old), x = static_cast<uint64_t>(v);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
        static_cast<int>(o), static_cast<int>(x), CTRL, RMASK, 0xf, false));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
        static_cast<int>(o >> 32), static_cast<int>(x >> 32), CTRL, RMASK, 0xf, false));
    return static_cast<T>((static_cast<uint64_t>(hi) << 32) | lo);
  }
}

// The value of one lane (the same in every lane's argument), in all of them.
template <class T>
__device__ __forceinline__ T wave_read(T v, int src) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two registers");
  if constexpr (sizeof(T) == 4) {
    return static_cast<T>(__builtin_amdgcn_readlane(static_cast<int>(v), src));
  } else {
    const uint64_t x = static_cast<uint64_t>(v);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), src));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x >> 32), src));
    return static_cast<T>((static_cast<uint64_t>(hi) << 32) | lo);
  }
}

// Inclusive prefix sum across the 64 lanes: shifts by 1, 2, 4 and 8 within
// rows of 16 lanes, then the last lane of a row added to the next one and
// that of the lower half to the upper.
template <class T>
__device__ __forceinline__ T wave_incl_scan(T v) {
  v += dpp_move<0x111, 0xf>(T(0), v);
  v += dpp_move<0x112, 0xf>(T(0), v);
  v += dpp_move<0x114, 0xf>(T(0), v);
  v += dpp_move<0x118, 0xf>(T(0), v);
  v += dpp_move<0x142, 0xa>(T(0), v);
  v += dpp_move<0x143, 0xc>(T(0), v);
  return v;
}

template <class T>
__device__ __forceinline__ T wave_sum(T v) {
  return wave_read(wave_incl_scan(v), kWave - 1);
}

template <class T>
__device__ __forceinline__ T wave_max(T v) {
  const auto up = [](T a, T b) { return b > a ? b : a; };
  v = up(v, dpp_move<0x111, 0xf>(v, v));
  v = up(v, dpp_move<0x112, 0xf>(v, v));
  v = up(v, dpp_move<0x114, 0xf>(v, v));
  v = up(v, dpp_move<0x118, 0xf>(v, v));
  v = up(v, dpp_move<0x142, 0xa>(v, v));
  v = up(v, dpp_move<0x143, 0xc>(v, v));
  return wave_read(v, kWave - 1);
}

// Block-wide exclusive scan of one value per thread; `sh` must hold
// blockDim.x / 64 + 1 elements of T.  Returns the exclusive prefix and writes
// the block total to *total.  Contains __syncthreads.  Every wave scans the
// waves' sums for itself (at most 16), so two barriers do.
template <class T>
__device__ __forceinline__ T block_excl_scan(T v, T* sh, T* total) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), nw = blockDim.x / kWave;
  const T inc = wave_incl_scan(v);
  if (lane() == kWave - 1) sh[w] = inc;
  __syncthreads();
  const T sums = wave_incl_scan(lane() < nw ? sh[lane()] : T(0));
  *total = wave_read(sums, nw - 1);
  const T before = w > 0 ? wave_read(sums, w - 1) : T(0);
  __syncthreads();
  return inc - v + before;
}

// Block-wide sum (result valid in every thread).  `sh` holds nw + 1 elements.
template <class T>
__device__ __forceinline__ T block_sum(T v, T* sh) {
  const int w = threadIdx.x / kWave, nw = blockDim.x / kWave;
  v = wave_sum(v);
  if (lane() == 0) sh[w] = v;
  __syncthreads();
  const T r = wave_sum(lane() < nw ? sh[lane()] : T(0));
  __syncthreads();
  return r;
}

// First index i in [lo, hi) with a[i] > key (a ascending); hi if none.
template <class T, class K>
__device__ __forceinline__ int64_t upper_bound_dev(const T* a, int64_t lo, int64_t hi, K key) {
  while (lo < hi) {
    int64_t mid = lo + ((hi - lo) >> 1);
    if (a[mid] <= key) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// First index i in [lo, hi) with a[i] >= key.
template <class T, class K>
__device__ __forceinline__ int64_t lower_bound_dev(const T* a, int64_t lo, int64_t hi, K key) {
  while (lo < hi) {
    int64_t mid = lo + ((hi - lo) >> 1);
    if (a[mid] < key) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

template <class T>
__device__ __forceinline__ T load_relaxed(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------ device scan
// Exclusive scan of `count` values (int32 or int64) into out[0..count]
// (out[count] = total).  `total_dev` (nullable) also receives the total.
// Temporary space comes from the carver.
template <class T>
int scan_exclusive(const T* in, int64_t* out, int64_t count, Carver& ws, hipStream_t s);
// The same over in[i * stride].
int scan_exclusive_strided(const int32_t* in, int64_t stride, int64_t* out, int64_t count, Carver& ws,
                           hipStream_t s);
size_t scan_ws_bytes(int64_t count);

// Fill helpers (kernels, never hipMemset, so the call sequence stays
// capturable without memset nodes).
int fill_i32(int32_t* p, int32_t v, int64_t count, hipStream_t s);
int fill_i64(int64_t* p, int64_t v, int64_t count, hipStream_t s);

}  // namespace tc

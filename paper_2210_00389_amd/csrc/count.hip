// count.hip -- the intersection stage of Alg. 1 and of the comparator.
//
// The count of Alg. 1 is a sum over (cover edge (u,v), apex w) pairs.  With
// the level-class layout (split.hip) a common neighbour w of a cover edge
// (u, v), u < v, on level l is in exactly one class:
//   up    w on level l-1:  w in Up(u)   ∩ Up(v)     (always counted)
//   same  w on level l:    w in Hfwd(u) ∩ Hfwd(v)   (counted: w > v; Hfwd(v)
//                          holds exactly the same-level neighbours above v)
//   down  w on level l+1:  w in Down(u) ∩ Down(v)   (always counted)
// The down class is summed from the apex side: for every edge x -> w with
// w in Down(x), count the t in Up(w) that lie in Hfwd(x); each (u, v, w)
// with u < v is met once, at x = u, t = v.  This is the same set of (edge,
// apex) pairs, enumerated per apex the way the paper's distributed variant
// enumerates the apexes a processor owns; it streams the short up-lists of
// the apexes instead of the long down-lists of hub pairs.
//
// Every intersection is a task: stream one sorted list S and test each
// element for membership in the probe set P(x) = Up(x) ∪ Hfwd(x) of an
// anchor x.  Ownership rules pick the cheaper side per task:
//   up     anchor = u if |Up(v)| <= |Up(u)| else v; stream Up(other)
//   same   a = |Hfwd(u) ∩ (v,inf)|, b = |Hfwd(v)|; if b < a anchor u streams
//          Hfwd(v), else anchor v streams Hfwd(u) ∩ (v,inf)
//   down   anchor x streams Up(w)
// A streamed list lies on one level, so the members of P(x) it can meet are
// in one segment: Up(x) for the up class, Hfwd(x) for the others.
//
// Every vertex x owns the descriptors [down | forward cover edges | backward
// cover edges]: deg(x) - sfe (when Hfwd(x) is not empty), |Hfwd(x)|, and
// its same-level neighbours below x.  One pass over all descriptors applies
// the ownership rules from x's side.  Light anchors (short probe set, few
// down-neighbours) merge their tasks at once.  Heavy anchors emit stream
// records, compacted per block, and the block cuts its records into work
// items of about kElemChunk elements of one anchor, tagged with the on-chip
// table the anchor needs (2 KB .. 128 KB of the 160 KB LDS: a bitmap over the
// probe set's id window, or a hash table) or row search beyond that.  The
// streaming kernel builds the table once per item and hands each lane chunks
// of 8 elements of one stream.  On larger graphs (kCoreNnz) the anchors beyond
// the 2 KB tables stream their lists as 16-bit offsets into the core of a
// level (core_kernel), and what lies outside the core apart.  Per-lane counts are reduced wave -> block ->
// one 64-bit atomic; the count runs without a host synchronisation.
//
// The comparator (plain direction-oriented edge iterator) runs through the
// same kernels with up = 0, Hfwd = forward list N+(x), no down class.
#include "tc_internal.h"

namespace tc {

namespace {

constexpr int kThreads = 256;
constexpr int kDnLight = 32;  // default: light anchors have at most this many down-neighbours
constexpr int kLightMax = 32; // and a probe set of at most this many ids (the register capacity
                              // of light_kernel, so the tuned bound never exceeds it)
constexpr int kBins = 5;      // the four bins below, then the core items
constexpr int kBinCore = 4;

// Bins of heavy anchors by the LDS table they need: 2 KB, 32 KB, 128 KB, or
// none (bin 3: search the sorted rows).  The probe set P(x) lies in the id
// window [min P, max P] of R ids.  It is held as a bitmap of R + 1 bits (bit
// R stays clear and absorbs every id outside the window) when clearing that
// bitmap costs little next to the anchor's work (at most four words per
// member plus 64, or 16 words per descriptor), else as a hash table filling
// the bin's whole table (at most half full).
constexpr int kBinWords0 = 512, kBinWords1 = 8192, kBinWords2 = 32768;

__host__ __device__ constexpr int bin_words(int b) {
  return b == 0 ? kBinWords0 : (b == 1 ? kBinWords1 : (b == 2 ? kBinWords2 : 0));
}

__device__ __forceinline__ int64_t bitmap_words(int64_t R) { return (R + 32) >> 5; }

// Two-level table of a probe set too large for an LDS bitmap or hash table:
// in LDS one bit per block of 32 ids of the window (set when the block holds
// a member) and, per 32 such bits, the number of set bits before them; in
// global memory the 32-bit member word of every non-empty block, in block
// order.  Words of LDS it needs for a window of R ids:
__device__ __forceinline__ int64_t twolevel_words(int64_t R) { return 2 * (((R >> 5) + 32) >> 5); }

enum TableKind { kKindHash = 0, kKindBitmap = 1, kKindTwoLevel = 2 };

// Bin of an anchor whose bitmap (two parts) takes `need` words, with joint
// window R, probe-set size P, D descriptors and deg row entries; *kind
// tells the table kind.  A two-level table's block bits
// are also kept in global memory at the anchor's row positions (so an item
// copies them instead of inserting |P| ids), hence they must fit in deg
// words.
__device__ __forceinline__ int choose_bin(int64_t need, int64_t R, int P, int64_t D, int64_t deg, int* kind,
                                          const CountParams& prm) {
  // the smallest-table bin streams an item with one wave: only anchors with
  // few tasks go there
  const int b0 = (prm.bin0_max_desc >= 0 && D > prm.bin0_max_desc) ? 1 : 0;
  if (need <= prm.bm_member * static_cast<int64_t>(P) + 64 || need <= prm.bm_desc * D) {
    for (int b = b0; b < 3; ++b)
      if (need <= bin_words(b)) {
        *kind = kKindBitmap;
        return b;
      }
  }
  const int64_t tw = twolevel_words(R);
  const bool tl_fits = tw <= kBinWords2 && tw / 2 <= deg;
  *kind = kKindHash;
  for (int b = b0; b < 3; ++b)
    if (2 * static_cast<int64_t>(P) <= bin_words(b)) {
      // a sparse set of the largest hash bin: most probes miss, and a
      // two-level table rejects them with one LDS read
      if (b == 2 && tl_fits && prm.tl_sparsity > 0 && R >= static_cast<int64_t>(prm.tl_sparsity) * P)
        *kind = kKindTwoLevel;
      return b;
    }
  if (tl_fits) {
    *kind = kKindTwoLevel;
    return 2;
  }
  return 3;
}

enum Acc {
  kAccT = 0, kAccElems = 1, kAccBuild = 3, kAccRecs = 4, kAccItems = 5, kAccHeavyElems = 6,
  kAccH = 7, kAccTwoLevelElems = 8, kAccBinCount = 9, kAccBinOff = kAccBinCount + kBins,
  kAccBinCur = kAccBinOff + kBins, kAccBinNext = kAccBinCur + kBins, kAccBinElems = kAccBinNext + kBins
};
constexpr int kAccSlots = kAccBinElems + kBins;
// Sums that only the last kernel reads are added in stripes of their own: the
// blocks of a short kernel end together, and their additions to one place take
// 4 ns each (two of them from 2800 blocks were 24 us of 169 of the light tasks
// at R-MAT scale 20).
constexpr int kAccStripes = 32, kAccPad = 48;
static_assert(kAccPad >= kAccSlots, "a stripe holds every slot");
constexpr int kAccAll = kAccPad * (1 + kAccStripes);  // the slots, then the stripes
constexpr int kElemChunkLog = 19;  // default: 2^19 elements per work item (target)
// stream record flag (in the length word): probe the anchor's Up list
constexpr int32_t kFlagUp = 1 << 29;
constexpr int32_t kLenMask = kFlagUp - 1;
// stream slot in LDS (s_cl.y): length | kClUp when the stream probes Up(x)
constexpr int32_t kClUp = 1 << 30;
// work item word: stream count | bin << 24 | kItemRest | kItemBitmap | kItemTwoLevel
constexpr int32_t kItemCountMask = (1 << 24) - 1;
constexpr int kItemBinShift = 24;
constexpr int32_t kItemRest = 1 << 27;  // the parts outside the core of a core anchor's lists
constexpr int32_t kItemBitmap = 1 << 30;
constexpr int32_t kItemTwoLevel = static_cast<int32_t>(0x80000000u);
// per-vertex plan: kViHeavy | two-level << 3 | bitmap << 2 | bin for the whole
// probe set, and where the anchor streams the core parts of its lists apart,
// kViCore | bitmap << 10 | bin << 8 for its members outside the core
constexpr uint16_t kViHeavy = 0x80;
constexpr uint16_t kViTwoLevel = 0x08;
constexpr uint16_t kViBitmap = 0x04;
constexpr uint16_t kViCore = 0x8000;
constexpr int kViRestShift = 8;

__device__ __forceinline__ void add_pv(int64_t* pv, int32_t v, int64_t count) {
  atomicAdd(reinterpret_cast<unsigned long long*>(&pv[v]), static_cast<unsigned long long>(count));
}

// Per-vertex counts of the apexes a block finds, in LDS: an apex takes the
// first of kPvProbes slots from its hash on that is free or its own, one that
// finds none goes to memory.  The apexes of an anchor are its probe set, so
// they repeat; the sums go out when the anchor changes.  Bound by the atomics
// to memory: with three of them per triangle the 32 KB bin took 3.67 ms on a
// Chung-Lu graph of 500009 vertices, with one slot an apex 0.27 ms; the
// counts of R-MAT scale 20 (424 M triangles) take 8.9 ms, 9.1 with two slots
// an apex, 11.1 with one.
constexpr uint32_t kPvFree = 0xFFFFFFFFu;
constexpr int kPvProbes = 4;  // slots an apex may take

template <int SLOTS>
struct PvCache {
  uint32_t* key;
  int32_t* sum;
  int32_t* osum;  // per stream of the batch: its hits, the streamed vertex's count
  __device__ __forceinline__ void add(int64_t* pv, int32_t v) const {
    if (SLOTS > 0) {
      uint32_t slot = (static_cast<uint32_t>(v) * 0x9E3779B1u) >> (32 - __builtin_ctz(SLOTS > 0 ? SLOTS : 2));
      for (int p = 0; p < kPvProbes; ++p) {
        const uint32_t was = atomicCAS(&key[slot], kPvFree, static_cast<uint32_t>(v));
        if (was == kPvFree || was == static_cast<uint32_t>(v)) {
          atomicAdd(&sum[slot], 1);
          return;
        }
        slot = (slot + 1) & (SLOTS - 1);
      }
    }
    add_pv(pv, v, 1);
  }
  // All threads; the caller has synchronised the block and does so after.
  __device__ __forceinline__ void flush(int64_t* pv, int threads) const {
    for (int i = threadIdx.x; i < SLOTS; i += threads) {
      if (sum[i]) add_pv(pv, static_cast<int32_t>(key[i]), sum[i]);
      key[i] = kPvFree;
      sum[i] = 0;
    }
  }
};

// What the counting kernels do with each triangle they find:
//   kOutNone  count only;
//   kOutPV    also add one to each of its three vertices (per-vertex counts:
//             the anchor's per item or task, the streamed list's per batch or
//             task, the apex's here);
//   kOutRec   also record every work unit's count (ucnt: heavy items by their
//             index in the item array, then light tasks by their index);
//   kOutEmit  write it at its work unit's offset (uoff) as three caller ids,
//             ascending (the second pass of triangle finding).
enum OutKind { kOutNone = 0, kOutPV = 1, kOutRec = 2, kOutEmit = 3 };

struct Out {
  int64_t* pv;
  int32_t* ucnt;
  const int64_t* uoff;
  int32_t* tri;          // [3 * cap]
  int64_t cap;
  const int32_t* order;  // layout id -> caller id (null: the same)
};

__host__ __device__ constexpr bool needs_oth(int k) { return k == kOutPV || k == kOutEmit; }

// a and b are caller ids already (mapped once per task or stream), c is a
// layout id.
__device__ __forceinline__ void write_tri(const Out& o, int64_t at, int32_t a, int32_t b, int32_t c) {
  if (at >= o.cap) return;
  if (o.order) c = o.order[c];
  int32_t t;
  if (a > b) { t = a; a = b; b = t; }
  if (b > c) { t = b; b = c; c = t; }
  if (a > b) { t = a; a = b; b = t; }
  o.tri[3 * at] = a;
  o.tri[3 * at + 1] = b;
  o.tri[3 * at + 2] = c;
}

__device__ __forceinline__ int32_t caller_id(const Out& o, int32_t v) { return o.order ? o.order[v] : v; }

// One triangle {x, oth, w} found by a thread that writes sequentially (for
// kOutEmit x and oth are caller ids, w a layout id).
template <int kOut>
__device__ __forceinline__ void on_hit(const Out& o, int32_t x, int32_t oth, int32_t w, int64_t& at) {
  if (kOut == kOutPV) add_pv(o.pv, w, 1);
  else if (kOut == kOutEmit) write_tri(o, at++, x, oth, w);
}

// Membership of t in a sorted list [p, p + len) in global memory.
__device__ __forceinline__ bool gsearch(const int32_t* p, int len, int32_t t) {
  int lo = 0, hi = len;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (p[mid] < t) lo = mid + 1;
    else hi = mid;
  }
  return lo < len && p[lo] == t;
}

__device__ __forceinline__ int probe_size(const VMeta& m) { return m.up + (m.sfe - m.hfb); }

// The record of the part of x's probe set outside the core.
__device__ __forceinline__ VMeta rest_meta(VMeta m) {
  m.up = m.ncu;
  m.sfe = m.hfb + m.nch;
  return m;
}

// Heavy anchors get work items; every task of a light anchor is merged by
// the planning kernels.  Must be the same predicate everywhere.
__device__ __forceinline__ bool is_heavy(const VMeta& m, bool cover, const CountParams& prm) {
  if (probe_size(m) > prm.light_max) return true;
  return cover && (m.sfe - m.hfb) > 0 && (m.deg - m.sfe) > prm.dn_light;
}

__device__ __forceinline__ void block_acc(unsigned long long* acc, int slot, int64_t v, int64_t* sh) {
  int64_t s = block_sum(v, sh);
  if (threadIdx.x == 0 && s)
    atomicAdd(&acc[kAccPad * (1 + blockIdx.x % kAccStripes) + slot], static_cast<unsigned long long>(s));
}


// Id window [lo, lo + R) of the probe set (R = 0 when it is empty).
__device__ __forceinline__ void probe_window(const int32_t* lc, const VMeta& m, int32_t& lo, int64_t& R) {
  const int hf = m.sfe - m.hfb;
  int32_t mn = 0x7FFFFFFF, mx = -1;
  if (m.up > 0) {
    mn = lc[m.begin];
    mx = lc[m.begin + m.up - 1];
  }
  if (hf > 0) {
    mn = min(mn, lc[m.begin + m.hfb]);
    mx = max(mx, lc[m.begin + m.sfe - 1]);
  }
  lo = mn;
  R = mx >= mn ? static_cast<int64_t>(mx) - mn + 1 : 0;
}

// A bitmap table is two bitmaps, one over the id window of Up(x) and one
// over that of Hfwd(x), each with its always-clear bit R (a part with no
// member is one word): a streamed list meets only one of the two segments
// (it lies on one level), and each part's window is usually far narrower
// than the window of both, which spans the gap between the two levels.
struct SplitWindow {
  int32_t lo_up, lo_hf;
  int64_t R_up, R_hf;
};

__device__ __forceinline__ SplitWindow split_window(const int32_t* lc, const VMeta& m) {
  SplitWindow w{0, 0, 0, 0};
  const int hf = m.sfe - m.hfb;
  if (m.up > 0) {
    w.lo_up = lc[m.begin];
    w.R_up = static_cast<int64_t>(lc[m.begin + m.up - 1]) - w.lo_up + 1;
  }
  if (hf > 0) {
    w.lo_hf = lc[m.begin + m.hfb];
    w.R_hf = static_cast<int64_t>(lc[m.begin + m.sfe - 1]) - w.lo_hf + 1;
  }
  return w;
}

// Words of the two bitmaps.
__device__ __forceinline__ int64_t split_words(const SplitWindow& w) {
  return bitmap_words(w.R_up) + bitmap_words(w.R_hf);
}

// The window of the whole probe set (for two-level tables), from its parts.
__device__ __forceinline__ void joint_window(const SplitWindow& w, int32_t& lo, int64_t& R) {
  int64_t mn = 0x7FFFFFFFFFFFFFFFll, mx = -1;
  if (w.R_up > 0) {
    mn = w.lo_up;
    mx = w.lo_up + w.R_up - 1;
  }
  if (w.R_hf > 0) {
    mn = min(mn, static_cast<int64_t>(w.lo_hf));
    mx = max(mx, w.lo_hf + w.R_hf - 1);
  }
  lo = mx >= 0 ? static_cast<int32_t>(mn) : 0x7FFFFFFF;
  R = mx >= 0 ? mx - mn + 1 : 0;
}


// The fields of a vertex record that the resolution reads of a neighbour
// (begin, up, hfb, sfe) in one 16-byte word, so that the random read of a
// neighbour's record is one request instead of two:
//   x = begin bits 0..31, y = begin bits 32..39 | up << 8, z = hfb, w = sfe.
// Bit 31 of z and w say that Up and Hfwd have entries outside the core (list
// lengths are below 2^29).  A record whose begin needs more than 40 bits or
// whose up is 2^24 - 1 or more gets y = kPmFull: the reader then takes the
// full record.
constexpr uint32_t kPmFull = 0xFFFFFFFFu;
constexpr uint32_t kPmRest = 0x80000000u;

__device__ __forceinline__ uint4 pack_record(const VMeta& m) {
  const uint64_t b = static_cast<uint64_t>(m.begin);
  if ((b >> 40) != 0 || m.up >= 0xFFFFFF) return make_uint4(0u, kPmFull, 0u, 0u);
  return make_uint4(static_cast<uint32_t>(b), static_cast<uint32_t>(b >> 32) | (static_cast<uint32_t>(m.up) << 8),
                    static_cast<uint32_t>(m.hfb) | (m.ncu > 0 ? kPmRest : 0u),
                    static_cast<uint32_t>(m.sfe) | (m.nch > 0 ? kPmRest : 0u));
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // loaded whole, in one instruction

// Record of vertex v for the resolution from its packed word q = pm[v] (deg
// is not filled in, ncu and nch are 0 or not 0 only).
__device__ __forceinline__ VMeta unpack_record(u32x4 q, const VMeta* meta, int32_t v) {
  VMeta m;
  m.begin = static_cast<int64_t>(q.x | (static_cast<uint64_t>(q.y & 0xFFu) << 32));
  m.up = static_cast<int32_t>(q.y >> 8);
  m.hfb = static_cast<int32_t>(q.z & ~kPmRest);
  m.sfe = static_cast<int32_t>(q.w & ~kPmRest);
  m.deg = 0;
  m.ncu = static_cast<int32_t>(q.z >> 31);
  m.nch = static_cast<int32_t>(q.w >> 31);
  if (q.y == kPmFull) m = meta[v];
  return m;
}

// ------------------------------------------------------------ planning
// One thread per vertex: descriptor count, |Hfwd| (for |H|), and for heavy
// anchors the table bin.
template <bool kCover>
__global__ __launch_bounds__(kThreads) void plan_kernel(const int32_t* lc, const VMeta* meta, int64_t n,
                                                        int32_t* ndesc, uint16_t* vinfo, uint4* pm,
                                                        unsigned long long* acc, CountParams prm, bool core) {
  __shared__ int64_t sh[kThreads / kWave + 1];
  int64_t h = 0;
  for (int64_t x0 = blockIdx.x * (int64_t)blockDim.x; x0 < n; x0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t x = x0 + threadIdx.x;
    if (x >= n) continue;
    const VMeta m = meta[x];
    const int hf = m.sfe - m.hfb;
    const int nB = (kCover && hf > 0) ? m.deg - m.sfe : 0;
    const int nU = (kCover && prm.up_anchor_min >= 0 && m.up > prm.up_anchor_min) ? m.up : 0;
    const int D = nB + hf + (m.hfb - m.up) + nU;
    h += hf;
    uint16_t vi = 0;
    if (D > 0 && is_heavy(m, kCover, prm)) {
      const SplitWindow sw = split_window(lc, m);
      int32_t lo;
      int64_t R;
      joint_window(sw, lo, R);
      int kind = kKindHash;
      const int b = choose_bin(split_words(sw), R, probe_size(m), D, m.deg, &kind, prm);
      vi = static_cast<uint16_t>(kViHeavy | (kind == kKindBitmap ? kViBitmap : 0) |
                                 (kind == kKindTwoLevel ? kViTwoLevel : 0) | b);
      // anchors beyond the smallest tables stream the core parts of their
      // lists against a 16 KB bitmap of the core; what they hold outside it
      // has to fit an LDS table of its own
      if (kCover && core && b > 0) {
        const VMeta mr = rest_meta(m);
        int rest = 0;
        if (probe_size(mr) > 0) {
          const SplitWindow rw = split_window(lc, mr);
          joint_window(rw, lo, R);
          rest = choose_bin(split_words(rw), R, probe_size(mr), D, 0, &kind, prm);
          if (kind == kKindBitmap) rest |= kViBitmap;
        }
        if ((rest & 3) < 3) vi |= kViCore | static_cast<uint16_t>(rest << kViRestShift);
      }
    }
    ndesc[x] = D;
    vinfo[x] = vi;
    pm[x] = pack_record(m);
  }
  block_acc(acc, kAccH, h, sh);
}

// ------------------------------------------------------------ resolution
// One thread per descriptor, chunks of kResChunk descriptors per block.  A
// descriptor yields at most two tasks with its vertex x as anchor (slot 0:
// up or down class, slot 1: same class).  Tasks of heavy anchors become
// stream records (from the front of the record arrays), tasks of light
// anchors go to the light list (from the back), merged by light_kernel.
constexpr int kResThreads = 256;
constexpr int kResPer = 2;  // descriptors per thread, resolved in lockstep
constexpr int kSampStride = 32;  // one column sample per 128-byte line
constexpr int kResChunk = kResThreads * kResPer;
constexpr int kResRecs = 2 * kResChunk;
constexpr int kResSpan = 2 * kResChunk;  // vertex offsets staged in LDS

struct Task {
  int64_t beg;   // stream begin in the columns
  int32_t len;   // stream length (0: no task) | kFlagUp
  int32_t oth;   // vertex whose list is streamed
  int32_t rest;  // its first entries outside the core that the anchor's own may meet (core anchors)
};

// Forward lists whose backward cover edges are resolved from the column
// samples (kLong).  Shorter ones are searched: their lines are few, and the
// entries up to the next sample would be most of the list.  kLong goes with
// the core streams, which read whole 128-byte lines of 16-bit ids, so that
// starting at a sample costs them nothing (R-MAT scale 24: resolution 14.4 ->
// 11.8 ms, core streams 18.8 ms either way); 32-bit streams lose by it what
// the resolution wins (per-vertex counts of a Chung-Lu graph, n = 500009:
// 1.76 -> 1.85 ms).
template <bool kLong>
__device__ __forceinline__ bool long_list(int len) { return kLong && len > kSampStride; }
// The first sampled place at or past the entry b + 1 places before `end`.
__device__ __forceinline__ int64_t taken_from(int64_t end, int b) {
  return (end - b - 1 + kSampStride - 1) / kSampStride * kSampStride;
}

enum DescKind { kDown = 0, kFwd = 1, kBwd = 2, kNone = 3, kUpD = 4 };

// Tasks of kResPer descriptors (vertex x[j], index k[j] in its descriptor
// space) with x[j] as the anchor of every returned task.  The steps run in
// lockstep over the descriptors so that their dependent loads (neighbour
// id, its record, the search of x in Hfwd(u)) are in flight together.
// A vertex's descriptors are [down | fwd | bwd | upd]: one per vertex of
// Down(x) (when Hfwd(x) is not empty), of Hfwd(x), of the same-level
// neighbours below x, and (cover count, |Up(x)| > upa) of Up(x).
template <bool kCover, bool kLong>
__device__ __forceinline__ void describe_all(const int32_t* lc, const int32_t* samp, const VMeta* meta,
                                             const uint4* pm, const int32_t* x, const VMeta* mx, const int* kin,
                                             int upa, const bool* core, Task* ta, Task* tb) {
  int kind[kResPer], k[kResPer];
  int32_t nb[kResPer];
  int64_t pos[kResPer];
  // positions first, without branches, so that the column loads of all
  // descriptors are in flight together (an idle slot reads column 0)
#pragma unroll
  for (int j = 0; j < kResPer; ++j) {
    ta[j] = Task{0, 0, 0, 0};
    tb[j] = Task{0, 0, 0, 0};
    const int hf = mx[j].sfe - mx[j].hfb;
    const int nB = (kCover && hf > 0) ? mx[j].deg - mx[j].sfe : 0;
    const int nS = mx[j].hfb - mx[j].up;
    const int kk = kin[j];
    const bool dn = kk < nB, fw = !dn && kk - nB < hf;
    const bool bw = !dn && !fw && (!kCover || kk - nB - hf < nS);
    kind[j] = kk < 0 ? kNone : (dn ? kDown : (fw ? kFwd : (bw ? kBwd : kUpD)));
    k[j] = dn ? kk : (fw ? kk - nB : (bw ? kk - nB - hf : kk - nB - hf - nS));
    const int32_t seg = dn ? mx[j].sfe : (fw ? mx[j].hfb : (bw ? mx[j].up : 0));
    pos[j] = kk < 0 ? 0 : mx[j].begin + seg + k[j];
  }
#pragma unroll
  for (int j = 0; j < kResPer; ++j) nb[j] = lc[pos[j]];
  // the neighbours' packed records, all loads issued before any is used
  u32x4 q[kResPer];
#pragma unroll
  for (int j = 0; j < kResPer; ++j) q[j] = *reinterpret_cast<const u32x4*>(pm + (kind[j] != kNone ? nb[j] : 0));
  VMeta mo[kResPer];
#pragma unroll
  for (int j = 0; j < kResPer; ++j)
    if (kind[j] != kNone) mo[j] = unpack_record(q[j], meta, nb[j]);
  // Backward same class, cover edge (u, x) with u < x.  Where Hfwd(u) is
  // short the rule compares a = |Hfwd(u) ∩ (x, inf)| with b = |Hfwd(x)|: the
  // entry b + 1 places before the end of Hfwd(u) decides it with one load:
  // above x, a > b and the forward descriptor of u takes the pair; equal to
  // x, a = b; below, x lies among the last b entries, and only they are
  // searched for it.  Where it is long (long_list) the column samples decide:
  // x takes the pair from the first sampled entry at or past that place on,
  // and streams Hfwd(u) from the last sampled entry at or below it (what lies
  // below x meets nothing of Hfwd(x)), so that neither the entry nor x's
  // place, a cache miss each, is read from the columns.
  int64_t lo[kResPer], hi[kResPer], blo[kResPer], bhi[kResPer];
  const int32_t* pp[kResPer];
  bool srch[kResPer], prb[kResPer], lng[kResPer];
#pragma unroll
  for (int j = 0; j < kResPer; ++j) {
    srch[j] = prb[j] = lng[j] = false;
    lo[j] = hi[j] = blo[j] = bhi[j] = 0;
    pp[j] = lc;
    const int b = mx[j].sfe - mx[j].hfb, lu = mo[j].sfe - mo[j].hfb;
    if (kind[j] == kBwd && b > 0 && lu > 0) {
      lo[j] = mo[j].begin + mo[j].hfb;
      hi[j] = mo[j].begin + mo[j].sfe;
      lng[j] = long_list<kLong>(lu);
      prb[j] = b + 1 < lu;
      srch[j] = !(lng[j] && prb[j]) || taken_from(hi[j], b) < hi[j];
      prb[j] = prb[j] && srch[j];
      blo[j] = lng[j] && prb[j] ? taken_from(hi[j], b) / kSampStride : (lo[j] + kSampStride - 1) / kSampStride;
      bhi[j] = lng[j] ? (hi[j] - 1) / kSampStride + 1 : blo[j];
      if (prb[j]) pp[j] = lng[j] ? samp + blo[j] : lc + (hi[j] - b - 1);
    }
  }
  {
    int32_t pv[kResPer];
#pragma unroll
    for (int j = 0; j < kResPer; ++j) pv[j] = *pp[j];  // an idle slot reads column 0
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      if (!prb[j]) continue;
      const int b = mx[j].sfe - mx[j].hfb;
      if (pv[j] > x[j]) {
        srch[j] = false;
        bhi[j] = blo[j];
      } else if (lng[j]) {
        ++blo[j];
      } else if (pv[j] == x[j]) {
        lo[j] = hi[j] = hi[j] - b - 1;
      } else {
        lo[j] = hi[j] - b;
      }
    }
  }
  while (kLong) {  // long lists: first sample in [blo, bhi) above x
    bool any = false;
    int32_t v[kResPer];
    int64_t mid[kResPer];
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      mid[j] = blo[j] + ((bhi[j] - blo[j]) >> 1);
      v[j] = blo[j] < bhi[j] ? samp[mid[j]] : 0;
    }
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      if (!(blo[j] < bhi[j])) continue;
      if (v[j] <= x[j]) blo[j] = mid[j] + 1;
      else bhi[j] = mid[j];
      any |= blo[j] < bhi[j];
    }
    if (!any) break;
  }
  for (;;) {  // short lists: the place of x
    bool any = false;
    int32_t v[kResPer];
    int64_t mid[kResPer];
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      mid[j] = lo[j] + ((hi[j] - lo[j]) >> 1);
      v[j] = (srch[j] && !lng[j] && lo[j] < hi[j]) ? lc[mid[j]] : 0;
    }
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      if (!(srch[j] && !lng[j] && lo[j] < hi[j])) continue;
      if (v[j] < x[j]) lo[j] = mid[j] + 1;
      else hi[j] = mid[j];
      any |= lo[j] < hi[j];
    }
    if (!any) break;
  }
#pragma unroll
  for (int j = 0; j < kResPer; ++j) {
    const VMeta& m = mx[j];
    const VMeta& o = mo[j];
    const int hf = m.sfe - m.hfb;
    if (kind[j] == kDown) {  // stream Up(w), unless w anchors the pair (see kUpD)
      if (o.up > 0 && !(upa >= 0 && o.up > upa && o.up > hf)) ta[j] = Task{o.begin, o.up, nb[j], 0};
    } else if (kind[j] == kUpD) {
      // u = nb in Up(x), x one level below u: when Up(x) (longer than upa)
      // is also longer than Hfwd(u), x anchors the down-class pair (u, x)
      // and streams Hfwd(u) against the Up part of its table; every cover
      // edge (u, v) with v in Up(x) closes a triangle
      const int hu = o.sfe - o.hfb;
      if (kCover && hu > 0 && m.up > hu) ta[j] = Task{o.begin + o.hfb, hu | kFlagUp, nb[j], 0};
    } else if (kind[j] == kFwd) {  // forward cover edge (x, v)
      if (kCover && o.up > 0 && o.up <= m.up) ta[j] = Task{o.begin, o.up | kFlagUp, nb[j], 0};
      const int a = hf - k[j] - 1, b = o.sfe - o.hfb;
      const bool mine = long_list<kLong>(hf) ? b + 1 < hf && pos[j] < taken_from(m.begin + m.sfe, b) : b < a;
      if (a > 0 && b > 0 && mine) tb[j] = Task{o.begin + o.hfb, b, nb[j], 0};
    } else if (kind[j] == kBwd) {  // backward cover edge (u, x), u < x
      if (kCover && o.up > 0 && o.up < m.up) ta[j] = Task{o.begin, o.up | kFlagUp, nb[j], 0};
      if (srch[j] && lng[j]) {
        const int64_t from = max(lo[j], (blo[j] - 1) * kSampStride), end = o.begin + o.sfe;
        tb[j] = Task{from, static_cast<int32_t>(end - from), nb[j], 0};
      } else if (srch[j]) {
        const int a = static_cast<int>(o.begin + o.sfe - lo[j]) - 1;  // lo = position of x
        if (a > 0 && hf >= a) tb[j] = Task{lo[j] + 1, a, nb[j], 0};
      }
    }
  }
  // Where both the streamed list and the anchor's segment have entries
  // outside the core, the list's are streamed apart: their number is read
  // from the neighbour's record (at most a prefix of the task's stream).
#pragma unroll
  for (int j = 0; j < kResPer; ++j) {
    if (!kCover || !core[j]) continue;
    const bool hfl = kind[j] == kUpD;  // slot 0 streams Hfwd(nb), not Up(nb)
    const bool ra = ta[j].len != 0 && (hfl ? mo[j].nch : mo[j].ncu) != 0 &&
                    ((ta[j].len & kFlagUp) ? mx[j].ncu : mx[j].nch) > 0;
    const bool rb = tb[j].len != 0 && mo[j].nch != 0 && mx[j].nch > 0;
    if (!ra && !rb) continue;
    const int2 nc = *reinterpret_cast<const int2*>(&meta[nb[j]].ncu);
    if (ra) ta[j].rest = hfl ? nc.y : nc.x;
    if (rb) {
      const int64_t end = mo[j].begin + mo[j].hfb + nc.y;  // of Hfwd(nb)'s entries outside the core
      tb[j].rest = static_cast<int32_t>(max(end - tb[j].beg, static_cast<int64_t>(0)));
    }
  }
}

// The tables of the two-level anchors (plan byte kViTwoLevel), at anchor x's
// row positions [begin, begin + deg):
//   words[begin + r]        the bits of its probe-set members in the r-th
//                           non-empty block of 32 ids of its window (the
//                           blocks number at most |P| <= deg(x));
//   l1[begin + i], i < nw   block bits (bit j of word i: block 32 i + j holds
//                           a member), copied into LDS by every item of x
//                           (nw <= deg(x) by the bin rule).
// One wave per anchor; the anchors are found 64 vertices at a time.
__global__ void twolevel_words_kernel(const int32_t* lc, const VMeta* meta, const uint16_t* vinfo, int64_t n,
                                      uint32_t* words, uint32_t* l1) {
  const int64_t wid = (blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x) / kWave;
  const int64_t nwv = (static_cast<int64_t>(gridDim.x) * blockDim.x) / kWave;
  const int ln = lane();
  for (int64_t x0 = wid * kWave; x0 < n; x0 += nwv * kWave) {
    const int64_t xl = x0 + ln;
    uint64_t mask = __ballot(xl < n && (vinfo[xl] & kViTwoLevel));
    while (mask) {
      const int j = __ffsll(static_cast<unsigned long long>(mask)) - 1;
      mask &= mask - 1;
      const VMeta m = meta[x0 + j];
      int32_t lo;
      int64_t R;
      probe_window(lc, m, lo, R);
      const int P = probe_size(m);
      const int nw = static_cast<int>(twolevel_words(R) >> 1);
      uint32_t* wx = words + m.begin;
      uint32_t* lx = l1 + m.begin;
      for (int i = ln; i < P; i += kWave) wx[i] = 0u;
      for (int i = ln; i < nw; i += kWave) lx[i] = 0u;
      __threadfence();
      int carry = 0;       // non-empty blocks before this round
      int32_t prevb = -1;  // block of the last member of the previous round
      for (int base = 0; base < P; base += kWave) {
        const int i = base + ln;
        int32_t b = -1;
        uint32_t d = 0;
        if (i < P) {
          const int32_t key = i < m.up ? lc[m.begin + i] : lc[m.begin + m.hfb + (i - m.up)];
          d = static_cast<uint32_t>(key - lo);
          b = static_cast<int32_t>(d >> 5);
        }
        int32_t pb = __shfl_up(b, 1, kWave);
        if (ln == 0) pb = prevb;
        const int start = (i < P && b != pb) ? 1 : 0;
        const int incl = wave_incl_scan(start);
        if (i < P) {
          atomicOr(&wx[carry + incl - 1], 1u << (d & 31));
          if (start) atomicOr(&lx[b >> 5], 1u << (b & 31));
        }
        carry += wave_read(incl, kWave - 1);
        prevb = __shfl(b, kWave - 1, kWave);  // a later round exists only if all 64 lanes were members
      }
    }
  }
}

// Column samples for the searches of the resolution: samp[b] = lc[b * kSampStride].
__global__ void sample_kernel(const int32_t* lc, int64_t nnz, int32_t* samp) {
  const int64_t nb = (nnz + kSampStride - 1) / kSampStride;
  for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < nb; b += (int64_t)gridDim.x * blockDim.x)
    samp[b] = lc[b * kSampStride];
}

// First vertex of every chunk of kResChunk descriptors: chunk c starts at
// descriptor c * kResChunk, owned by the vertex x with so[x] <= it < so[x+1].
// cx0[nchunks] = n - 1 closes the last chunk.
__global__ void chunk_start_kernel(const int64_t* so, int64_t n, int32_t* cx0) {
  const int64_t total = so[n];
  const int64_t nch = (total + kResChunk - 1) / kResChunk;
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c0 = (so[x] + kResChunk - 1) / kResChunk, c1 = (so[x + 1] + kResChunk - 1) / kResChunk;
    for (int64_t c = c0; c < c1; ++c) cx0[c] = static_cast<int32_t>(x);
    if (x == n - 1) cx0[nch] = static_cast<int32_t>(n - 1);
  }
}

// Chunk c owns the record region [2 d0, 2 d1) of its descriptors [d0, d1):
// records of heavy anchors from the front, tasks of light anchors from the
// back, its work items at the same offsets of items_raw; ccnt[c] = (heavy
// records, light tasks, items).  No counter is shared between blocks.
// Thread t takes descriptors d0 + t + j * kResThreads; records are placed in
// descriptor order (j-major).
template <bool kCover, bool kLong>
__global__ __launch_bounds__(kResThreads) void resolve_kernel(
    const int32_t* lc, const int32_t* samp, const VMeta* meta, const uint4* pm, const uint16_t* vinfo,
    const int64_t* so, const int32_t* cx0, int64_t n, int64_t* sbeg, int32_t* slen, int32_t* soth, int32_t* sx,
    int4* items_raw, int4* ccnt, int64_t nchunk_cap, int item_log2, int upa) {
  __shared__ int64_t sh[kResThreads / kWave + 1];
  __shared__ int32_t shi[kResThreads / kWave + 1];
  __shared__ int64_t s_so[kResSpan];
  __shared__ int32_t s_x[kResRecs];
  __shared__ int64_t s_pre[kResRecs];
  __shared__ int32_t s_first[kResRecs + 1];
  const int tid = threadIdx.x;
  const int64_t total = so[n];
  const int64_t nch = (total + kResChunk - 1) / kResChunk;
  for (int64_t c = blockIdx.x; c < nchunk_cap; c += gridDim.x) {
    if (c >= nch) {  // past the descriptors: nothing for the scan of the counts
      if (tid == 0) ccnt[c] = make_int4(0, 0, 0, 0);
      continue;
    }
    const int64_t d0 = c * kResChunk;
    const int64_t d1 = min(d0 + kResChunk, total);
    const int64_t xa = cx0[c], xz = cx0[c + 1];  // the vertex of d1 - 1 is in [xa, xz]
    const int64_t span = xz - xa + 2;            // so[xa .. xz + 1]
    const bool staged = span <= kResSpan;
    if (staged)
      for (int i = tid; i < span; i += kResThreads) s_so[i] = so[xa + i];
    __syncthreads();
    int32_t xi[kResPer];
    int kk[kResPer];
    bool heavy[kResPer];
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      const int64_t d = d0 + tid + j * kResThreads;
      xi[j] = 0;
      kk[j] = -1;
      heavy[j] = false;
      if (d >= d1) continue;
      int64_t x, xb;
      if (staged) {
        int lo = 0, hi = static_cast<int>(span);  // first index with s_so > d
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (s_so[mid] <= d) lo = mid + 1;
          else hi = mid;
        }
        x = xa + lo - 1;
        xb = s_so[lo - 1];
      } else {
        x = upper_bound_dev(so, xa, xz + 2, d) - 1;
        xb = so[x];
      }
      xi[j] = static_cast<int32_t>(x);
      kk[j] = static_cast<int>(d - xb);
    }
    VMeta mx[kResPer];
    uint16_t vi[kResPer];
    bool core[kResPer];
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {  // loads of all slots together (an idle slot reads vertex 0's)
      mx[j] = meta[xi[j]];
      vi[j] = vinfo[xi[j]];
    }
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      heavy[j] = kk[j] >= 0 && (vi[j] & kViHeavy) != 0;
      core[j] = heavy[j] && (vi[j] & kViCore) != 0;
    }
    Task ta[kResPer], tb[kResPer];
    describe_all<kCover, kLong>(lc, samp, meta, pm, xi, mx, kk, upa, core, ta, tb);
    // Records outside the core follow the heavy records; where the region has
    // no room for them the chunk's core anchors stream whole lists.
    int64_t nr = 0;
#pragma unroll
    for (int j = 0; j < kResPer; ++j)
      nr |= static_cast<int64_t>((ta[j].rest > 0) + (tb[j].rest > 0)) << (16 * j);
    // ---- counts: light tasks, heavy records, heavy elements (per j, j-major)
    int64_t nl = 0, nh = 0;
    int64_t he[kResPer];
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      const int64_t cnt = (ta[j].len != 0) + (tb[j].len != 0);
      he[j] = heavy[j] ? static_cast<int64_t>(ta[j].len & kLenMask) + (tb[j].len & kLenMask) : 0;
      nl |= (heavy[j] ? 0 : cnt) << (16 * j);  // kResPer * 16 bits: counts <= 2 per descriptor
      nh |= (heavy[j] ? cnt : 0) << (16 * j);
    }
    int64_t ltot_p, htot_p, rtot_p = 0, rpre_p = 0;
    const int64_t lpre_p = block_excl_scan(nl, sh, &ltot_p);
    const int64_t hpre_p = block_excl_scan(nh, sh, &htot_p);
    if (kCover) rpre_p = block_excl_scan(nr, sh, &rtot_p);
    int32_t lslot[kResPer], hslot[kResPer], rslot[kResPer];
    int32_t ltot = 0, htot = 0, rtot = 0;
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      // slots of descriptor group j start after all groups before it
      lslot[j] = ltot + static_cast<int32_t>((lpre_p >> (16 * j)) & 0xFFFF);
      hslot[j] = htot + static_cast<int32_t>((hpre_p >> (16 * j)) & 0xFFFF);
      rslot[j] = rtot + static_cast<int32_t>((rpre_p >> (16 * j)) & 0xFFFF);
      rtot += static_cast<int32_t>((rtot_p >> (16 * j)) & 0xFFFF);
      ltot += static_cast<int32_t>((ltot_p >> (16 * j)) & 0xFFFF);
      htot += static_cast<int32_t>((htot_p >> (16 * j)) & 0xFFFF);
    }
    int64_t ebase = 0;
    int64_t epre[kResPer];
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      int64_t et;
      epre[j] = ebase + block_excl_scan(he[j], sh, &et);
      ebase += et;
    }
    const int64_t rbase = 2 * d0, rend = 2 * d1;
    const bool apart = htot + rtot + ltot <= static_cast<int>(rend - rbase);  // block-uniform
    if (!apart) rtot = 0;
#pragma unroll
    for (int j = 0; j < kResPer; ++j) {
      const Task* tt[2] = {&ta[j], &tb[j]};
      if (!heavy[j]) {  // light tasks to the back of the region
        int64_t pos = rend - 1 - lslot[j];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (!tt[q]->len) continue;
          sbeg[pos] = tt[q]->beg;
          slen[pos] = tt[q]->len;
          soth[pos] = tt[q]->oth;
          sx[pos] = xi[j];
          --pos;
        }
      } else {  // heavy records to the front
        int sl = hslot[j], rs = htot + rslot[j];
        int64_t e = epre[j];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (!tt[q]->len) continue;
          const int32_t rest = apart ? tt[q]->rest : 0;
          sbeg[rbase + sl] = tt[q]->beg + rest;
          slen[rbase + sl] = tt[q]->len - rest;
          soth[rbase + sl] = tt[q]->oth;
          s_x[sl] = xi[j];
          s_pre[sl] = e;
          e += tt[q]->len & kLenMask;
          ++sl;
          if (rest > 0) {
            sbeg[rbase + rs] = tt[q]->beg;
            slen[rbase + rs] = rest | (tt[q]->len & kFlagUp);
            soth[rbase + rs] = tt[q]->oth;
            s_x[rs] = xi[j];
            s_pre[rs] = 0;  // one item per anchor and chunk
            ++rs;
          }
        }
      }
    }
    if (htot == 0) {  // block-uniform
      if (tid == 0) ccnt[c] = make_int4(0, ltot, 0, 0);
      continue;
    }
    __syncthreads();
    // ---- cut into work items: a new item starts where the anchor changes
    // or the record's element offset enters the next 2^item_log2
    // The slots are taken kResRecs / kResThreads consecutive ones a thread.
    auto starts = [&](int q) {
      return q == 0 || q == htot || s_x[q] != s_x[q - 1] || (s_pre[q] >> item_log2) != (s_pre[q - 1] >> item_log2);
    };
    constexpr int kPerThread = kResRecs / kResThreads;
    const int nrec = htot + rtot;
    int ns = 0;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const int q = tid * kPerThread + i;
      ns += q < nrec && starts(q);
    }
    int nitems;
    int it = block_excl_scan(ns, shi, &nitems);
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const int q = tid * kPerThread + i;
      if (q < nrec && starts(q)) s_first[it++] = q;
    }
    if (tid == 0) {
      s_first[nitems] = nrec;
      ccnt[c] = make_int4(nrec, ltot, nitems, 0);
    }
    __syncthreads();
    for (int i = tid; i < nitems; i += kResThreads) {
      const int32_t x = s_x[s_first[i]];
      const uint16_t vi = vinfo[x];
      const int64_t r0 = rbase + s_first[i];
      const int cntr = s_first[i + 1] - s_first[i];
      int32_t w;
      if (s_first[i] >= htot) {
        const int rest = vi >> kViRestShift;
        w = cntr | ((rest & 3) << kItemBinShift) | ((rest & kViBitmap) ? kItemBitmap : 0) | kItemRest;
      } else if (kCover && apart && (vi & kViCore)) {
        w = cntr | (kBinCore << kItemBinShift);
      } else {
        w = cntr | ((vi & 3) << kItemBinShift) | ((vi & kViBitmap) ? kItemBitmap : 0) |
            ((vi & kViTwoLevel) ? kItemTwoLevel : 0);
      }
      items_raw[rbase + i] = make_int4(x, static_cast<int>(r0 & 0xFFFFFFFF), static_cast<int>(r0 >> 32), w);
    }
    __syncthreads();
  }
}

// Tasks of light anchors, read from the back of every chunk's region; one
// thread per task, found from the scan lpre of the per-chunk task counts
// between the chunks ltab[g], ltab[g + 1] of the wave's and the next wave's
// first task.  The probe segment (at most kLightMax ids) and a stream of
// at most kLightMax ids are loaded into registers with independent loads and
// compared pairwise, eight by eight up to the wave's longest segment and
// stream (comparing all 32 x 32 for lists of six ids on average took 195 us
// at R-MAT scale 20, VALU-bound); a longer stream (down class) is searched
// for every probe id, all searches advancing together.
constexpr int kLightStep = 8;

template <int kOut>
__global__ __launch_bounds__(kThreads) void light_kernel(const int32_t* lc, const VMeta* meta, const int64_t* so,
                                                         int64_t n, const int64_t* lpre, const int32_t* ltab,
                                                         int64_t nchunk_cap, const int64_t* sbeg, const int32_t* slen,
                                                         const int32_t* soth, const int32_t* sx,
                                                         unsigned long long* acc, Out o) {
  __shared__ int64_t sh[kThreads / kWave + 1];
  const int64_t total = so[n];
  const int64_t nl = lpre[nchunk_cap];
  // light tasks follow the heavy items in the unit numbering
  const int64_t ubase = (kOut == kOutRec || kOut == kOutEmit) ? static_cast<int64_t>(acc[kAccItems]) : 0;
  int64_t cnt = 0, elems = 0;
  const int64_t wave0 = blockIdx.x * static_cast<int64_t>(kThreads / kWave) +
                        __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  for (int64_t w0 = wave0 * kWave; w0 < nl; w0 += (int64_t)gridDim.x * kThreads) {  // the whole wave takes part
    const int64_t i = w0 + lane();
    const bool mine = i < nl;
    const int64_t ca = ltab[w0 / kWave];
    const int64_t cz = w0 + kWave < nl ? ltab[w0 / kWave + 1] + 1 : nchunk_cap + 1;
    int32_t x = 0, oth = 0, lf = 0;
    int64_t at = 0;
    const int32_t* P = lc;
    const int32_t* S = lc;
    int np = 0, len = 0;
    if (mine) {
      const int64_t c = upper_bound_dev(lpre, ca + 1, cz, i) - 1;
      const int64_t pos = 2 * min((c + 1) * kResChunk, total) - 1 - (i - lpre[c]);
      x = sx[pos];
      lf = slen[pos];
      if (needs_oth(kOut)) oth = soth[pos];
      if (kOut == kOutEmit) at = o.uoff[ubase + i];
      const VMeta mx = meta[x];
      len = lf & kLenMask;
      const bool up = (lf & kFlagUp) != 0;
      P = lc + mx.begin + (up ? 0 : mx.hfb);
      np = up ? mx.up : mx.sfe - mx.hfb;
      S = lc + sbeg[pos];
    }
    // the ids a hit reports: caller ids when writing triangles
    const int32_t hx = kOut == kOutEmit ? caller_id(o, x) : x;
    const int32_t ho = kOut == kOutEmit ? caller_id(o, oth) : oth;
    int64_t tc = 0;
    const bool pairs = len <= kLightMax;
    const int maxp = wave_max(np), maxs = wave_max(pairs ? len : 0);
    int32_t pr[kLightMax];
#pragma unroll
    for (int g = 0; g < kLightMax; g += kLightStep) {
      if (g >= maxp) break;  // uniform
#pragma unroll
      for (int q = g; q < g + kLightStep; ++q) pr[q] = q < np ? P[q] : -1;
    }
#pragma unroll
    for (int gs = 0; gs < kLightMax; gs += kLightStep) {
      if (gs >= maxs) break;  // uniform
      int32_t sv[kLightStep];
      uint32_t m = 0;
#pragma unroll
      for (int q = 0; q < kLightStep; ++q) sv[q] = pairs && gs + q < len ? S[gs + q] : -2;
#pragma unroll
      for (int g = 0; g < kLightMax; g += kLightStep) {
        if (g >= maxp) break;  // uniform
#pragma unroll
        for (int q = 0; q < kLightStep; ++q) {
          bool eq = false;
#pragma unroll
          for (int j = 0; j < kLightStep; ++j) eq |= sv[q] == pr[g + j];
          m |= static_cast<uint32_t>(eq) << q;
        }
      }
      tc += __popc(m);
      if (kOut == kOutPV || kOut == kOutEmit) {
#pragma unroll
        for (int q = 0; q < kLightStep; ++q)
          if ((m >> q) & 1u) on_hit<kOut>(o, hx, ho, sv[q], at);
      }
    }
    if (pairs) {
      elems += len;
    } else {
      // probes in groups of 8: lower bound of each in S by binary lifting
      for (int q0 = 0; q0 < np; q0 += 8) {
        int32_t pv[8];
        int lo[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          pv[j] = q0 + j < np ? P[q0 + j] : 0x7FFFFFFF;
          lo[j] = 0;
        }
        for (int step = 1 << (31 - __clz(len)); step > 0; step >>= 1) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int probe_at = lo[j] + step - 1;
            const int32_t v = (q0 + j < np && probe_at < len) ? S[probe_at] : 0x7FFFFFFF;
            if (v < pv[j]) lo[j] += step;
          }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bool m = q0 + j < np && lo[j] < len && S[lo[j]] == pv[j];
          tc += m;
          if (m) on_hit<kOut>(o, hx, ho, pv[j], at);
        }
      }
      elems += np;
    }
    cnt += tc;
    if (kOut == kOutPV && tc) {
      add_pv(o.pv, x, tc);
      add_pv(o.pv, oth, tc);
    }
    if (kOut == kOutRec && mine) o.ucnt[ubase + i] = static_cast<int32_t>(tc);
  }
  if (kOut != kOutEmit) {
    block_acc(acc, kAccT, cnt, sh);
    block_acc(acc, kAccElems, elems, sh);
  }
}

// Items grouped by bin, in chunk order within each block of chunks (so the
// consecutive items of one anchor stay adjacent).  One thread per chunk;
// kFill = false counts per bin, kFill = true scatters.
template <bool kFill>
__global__ __launch_bounds__(kThreads) void bin_split_kernel(const int64_t* so, int64_t n, const int4* ccnt,
                                                             const int4* items_raw, int4* items, const int64_t* lpre,
                                                             int32_t* ltab, unsigned long long* acc) {
  __shared__ unsigned long long s_base[kBins], s_off[kBins];
  __shared__ int64_t sh[kThreads / kWave + 1];
  if (kFill && threadIdx.x == 0) {  // the bins one after another; block 0 tells the later kernels
    unsigned long long run = 0;
    for (int b = 0; b < kBins; ++b) {
      s_off[b] = run;
      if (blockIdx.x == 0) acc[kAccBinOff + b] = run;
      run += acc[kAccBinCount + b];
    }
    if (blockIdx.x == 0) acc[kAccItems] = run;
  }
  __syncthreads();
  const int64_t total = so[n];
  const int64_t nch = (total + kResChunk - 1) / kResChunk;
  int64_t recs = 0;
  for (int64_t c0 = blockIdx.x * (int64_t)blockDim.x; c0 < nch; c0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = c0 + threadIdx.x;
    int ni = 0;
    int k[kBins] = {};
    if (c < nch) {
      ni = ccnt[c].z;
      if (!kFill) recs += ccnt[c].x;
      if (kFill) {  // the chunk of every 64th light task
        const int64_t lz = lpre[c + 1];
        for (int64_t g = (lpre[c] + kWave - 1) / kWave; g * kWave < lz; ++g) ltab[g] = static_cast<int32_t>(c);
      }
      for (int i = 0; i < ni; ++i) {
        const int b = (items_raw[2 * c * kResChunk + i].w >> kItemBinShift) & 7;
#pragma unroll
        for (int q = 0; q < kBins; ++q) k[q] += b == q;
      }
    }
    // per-bin exclusive offsets within the block, two bins per 64-bit word
    // (at most 2^18 items per bin and block)
    constexpr int kWords = (kBins + 1) / 2;
    int64_t tot[kWords], pre[kWords];
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
      const int64_t hi = 2 * i + 1 < kBins ? k[2 * i + 1] : 0;
      pre[i] = block_excl_scan(static_cast<int64_t>(k[2 * i]) | (hi << 32), sh, &tot[i]);
    }
    if (threadIdx.x < kBins) {
      unsigned long long kb = 0;
#pragma unroll
      for (int q = 0; q < kBins; ++q)
        if (threadIdx.x == q) kb = static_cast<unsigned long long>((tot[q >> 1] >> (32 * (q & 1))) & 0xFFFFFFFF);
      if (kb) {
        if (!kFill) atomicAdd(&acc[kAccBinCount + threadIdx.x], kb);
        else s_base[threadIdx.x] = s_off[threadIdx.x] + atomicAdd(&acc[kAccBinCur + threadIdx.x], kb);
      }
    }
    __syncthreads();
    if (kFill && ni) {
      int64_t pos[kBins];
#pragma unroll
      for (int q = 0; q < kBins; ++q)
        pos[q] = static_cast<int64_t>(s_base[q]) + ((pre[q >> 1] >> (32 * (q & 1))) & 0xFFFFFFFF);
      for (int i = 0; i < ni; ++i) {
        const int4 item = items_raw[2 * c * kResChunk + i];
        const int b = (item.w >> kItemBinShift) & 7;
        int64_t q = 0;
#pragma unroll
        for (int j = 0; j < kBins; ++j)
          if (b == j) q = pos[j]++;
        items[q] = item;
      }
    }
    __syncthreads();
  }
  if (!kFill) block_acc(acc, kAccRecs, recs, sh);
}

// ------------------------------------------------------------ streaming
// Multiplicative hash on the top bits of a 32-bit product; the id's bits
// above 24 are folded in first so that the multiply is the full-rate 24-bit
// one (a 32-bit integer multiply issues at a quarter of the rate).  HIP's
// __umul24 returns int: the product is taken as unsigned before the shift,
// so that the slot stays below 2^(32 - shift).
__device__ __forceinline__ uint32_t hslot(int32_t key, int shift) {
  const uint32_t k = static_cast<uint32_t>(key);
  return static_cast<uint32_t>(__umul24(k ^ (k >> 24), 0x9E3779u)) >> shift;
}

// Hash tables (linear probing, at most half full) hold the ids in the low
// 31 bits of a slot; kHashEmpty is no vertex id (ids are below 2^31 - 1).
// Bit 31 of a slot says that a key whose home is this slot was placed
// further on: a probe that finds another key in its home slot with that
// bit clear is a miss at once, and only a flagged home is walked until the
// key or an empty slot.  (Keys are never removed, so a key lies before the
// first empty slot after its home.)
constexpr uint32_t kHashEmpty = 0x7FFFFFFFu;
constexpr uint32_t kHashMoved = 0x80000000u;

enum ProbeMode { kBitmap = 0, kHash = 1, kSearch = 2, kTwoLevel = 3 };

// Probe set P(x) = Up(x) ∪ Hfwd(x) of the block's current anchor.
struct ProbeSet {
  const uint32_t* tab;
  int32_t lo;      // two-level: id of bit 0 of the joint window
  uint32_t R;      // two-level: window length (ids >= R miss)
  int32_t lo_up, lo_hf;  // bitmap: id of bit 0 of the Up and the Hfwd part
  uint32_t R_up, R_hf;   // bitmap: window lengths; bit R of each part is kept clear
  uint32_t off_hf;       // bitmap: first word of the Hfwd part
  int nw;          // two-level: LDS words of block bits (their prefix counts follow)
  const uint32_t* words;  // two-level: the member words of the non-empty blocks
  int cap, shift;  // hash: slot count (power of two) and hslot shift
  const int32_t* up_row;
  const int32_t* hf_row;
  int up_len, hf_len;
};

// 1 if t is in the probe set, else 0.  t may be any value (the tail of a
// chunk past the stream end is probed and masked afterwards).
template <int MODE>
__device__ __forceinline__ uint32_t probe(const ProbeSet& ps, int32_t t, bool up_side) {
  if (MODE == kBitmap) {
    // the part of the stream's segment (uniform over a chunk)
    const uint32_t lo = static_cast<uint32_t>(up_side ? ps.lo_up : ps.lo_hf);
    const uint32_t R = up_side ? ps.R_up : ps.R_hf;
    const uint32_t* tb = up_side ? ps.tab : ps.tab + ps.off_hf;
    const uint32_t d = min(static_cast<uint32_t>(t) - lo, R);
    return (tb[d >> 5] >> (d & 31)) & 1u;
  } else if (MODE == kTwoLevel) {
    const uint32_t d = static_cast<uint32_t>(t) - static_cast<uint32_t>(ps.lo);
    if (d >= ps.R) return 0u;
    const uint32_t b = d >> 5;
    const uint32_t w1 = ps.tab[b >> 5];
    if (!((w1 >> (b & 31)) & 1u)) return 0u;  // an empty block: no member
    const uint32_t r = ps.tab[ps.nw + (b >> 5)] + __popc(w1 & ((1u << (b & 31)) - 1u));
    return (ps.words[r] >> (d & 31)) & 1u;
  } else if (MODE == kHash) {
    uint32_t h = hslot(t, ps.shift);
    const uint32_t w = ps.tab[h];
    if ((w & kHashEmpty) == static_cast<uint32_t>(t)) return 1u;
    if (!(w & kHashMoved)) return 0u;
    for (;;) {
      h = (h + 1) & (ps.cap - 1);
      const uint32_t k = ps.tab[h] & kHashEmpty;
      if (k == static_cast<uint32_t>(t)) return 1u;
      if (k == kHashEmpty) return 0u;
    }
  }
  return (up_side ? gsearch(ps.up_row, ps.up_len, t) : gsearch(ps.hf_row, ps.hf_len, t)) ? 1u : 0u;
}

// Streams are cut into chunks of kChunk consecutive elements that never
// cross a stream end; a lane takes one chunk at a time (kChunk independent
// loads in flight, one 64-bit address).  The column buffers carry kColPad
// readable entries past nnz, so the tail of a stream's last chunk is loaded
// unconditionally and masked.
constexpr int kChunk = 8;
constexpr int kWinIters = 8;  // chunk rounds of the block per window
// Work items a block claims at once: the counter gives out 80 M claims a
// second, which bounds the small items of the 2 KB bin (R-MAT scale 24, 1.34 M
// items by 2 / 4 / 8 / 16: 8.52 / 4.92 / 4.27 / 4.46 ms); the others are
// longer, and the last claims end the later the more they hold (32 KB bin at
// scale 20 by 1 / 2 / 4 / 8: 37 / 43 / 63 / 89 us; core items 886 / 677 / 676 /
// 710 us).  Per-vertex counts keep an anchor's sums over its items (R-MAT scale
// 18 by 2 / 4: 4.67 / 4.18 ms).
constexpr int kClaimSmall = 8, kClaim = 2, kClaimPv = 4;
// Chunk slots per lane whose loads are in flight together: two where the
// registers allow (the 128 KB bin and row search, whose blocks are limited
// by LDS or run four waves per SIMD), one in the small-table bins compiled
// for six waves per SIMD (a second slot spills there).
template <int WORDS>
constexpr int ahead_of() { return (WORDS == kBinWords2 || WORDS == 0) ? 2 : 1; }
static_assert(kChunk <= kColPad, "chunk tail must stay inside the padded columns");

// Hits of one chunk whose entries v (len of them valid) are loaded.
template <int MODE, int kOut, int SLOTS>
// Called by every lane of the wave (a lane with no chunk passes len = 0);
// wq: the wave's queue of kWave ids in LDS (hash tables, counting only).
__device__ __forceinline__ uint32_t chunk_probe(const int32_t (&v)[kChunk], int len, const ProbeSet& ps, bool up_side,
                                                int32_t x, int32_t oth, const Out& o, int64_t ebase, int* s_pos,
                                                int32_t* wq, const PvCache<SLOTS>& pvc) {
  const uint32_t lenmask = len >= kChunk ? ((1u << kChunk) - 1u) : ((1u << len) - 1u);
  uint32_t hits = 0;
  if (MODE == kHash) {
    // all first probes in flight together; the chains of flagged homes are
    // walked afterwards, one slot per round for all
    uint32_t h[kChunk], w[kChunk];
    uint32_t pend = 0;
#pragma unroll
    for (int q = 0; q < kChunk; ++q) h[q] = hslot(v[q], ps.shift);
    // every home slot's read is issued before any is compared
#pragma unroll
    for (int q = 0; q < kChunk; ++q) w[q] = ps.tab[h[q]];
#pragma unroll
    for (int q = 0; q < kChunk; ++q) {
      const bool eq = (w[q] & kHashEmpty) == static_cast<uint32_t>(v[q]);
      hits |= static_cast<uint32_t>(eq) << q;
      pend |= static_cast<uint32_t>(!eq && (w[q] & kHashMoved) != 0) << q;
    }
    pend &= lenmask;
    if (kOut == kOutNone || kOut == kOutRec) {
      // Counting only: the ids still pending in the whole wave (about 1% of
      // them) go to the wave's queue, kWave at a time, and each lane walks
      // at most one chain from the home slot on, instead of every lane
      // stepping all 8 of its slots until the wave's longest walk ends.
      const int np = __popc(pend);
      const int incl = wave_incl_scan(np);
      const int total = wave_read(incl, kWave - 1);
      uint32_t walked = 0;
      for (int base = 0; base < total; base += kWave) {  // uniform across the wave
        int pos = incl - np - base;
#pragma unroll
        for (int q = 0; q < kChunk; ++q)
          if ((pend >> q) & 1u) {
            if (pos >= 0 && pos < kWave) wq[pos] = v[q];
            ++pos;
          }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (base + lane() < total) {
          const int32_t t = wq[lane()];
          uint32_t hq = hslot(t, ps.shift);
          for (;;) {
            hq = (hq + 1) & static_cast<uint32_t>(ps.cap - 1);
            const uint32_t k = ps.tab[hq] & kHashEmpty;
            if (k == static_cast<uint32_t>(t)) {
              ++walked;
              break;
            }
            if (k == kHashEmpty) break;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();  // the next batch overwrites the queue
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
      return static_cast<uint32_t>(__popc(hits & lenmask)) + walked;
    }
    while (pend) {
#pragma unroll
      for (int q = 0; q < kChunk; ++q) {
        const uint32_t pb = (pend >> q) & 1u;
        h[q] = (h[q] + pb) & static_cast<uint32_t>(ps.cap - 1);
        const uint32_t k = ps.tab[h[q]] & kHashEmpty;
        const bool eq = k == static_cast<uint32_t>(v[q]);
        hits |= (pb & static_cast<uint32_t>(eq)) << q;
        pend &= ~(static_cast<uint32_t>(eq || k == kHashEmpty) << q);
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < kChunk; ++q) hits |= probe<MODE>(ps, v[q], up_side) << q;
  }
  hits &= lenmask;
  if (kOut == kOutPV && hits) {
    atomicAdd(&pvc.osum[oth], __popc(hits));
#pragma unroll
    for (int q = 0; q < kChunk; ++q)
      if ((hits >> q) & 1u) pvc.add(o.pv, v[q]);
  }
  if (kOut == kOutEmit) {
    // The item's triangles fill [ebase, ebase + its count) in any order; a
    // wave takes one range per round and its lanes write consecutive parts
    // of it (called by every lane of the wave).
    const int nh = __popc(hits);
    const int incl = wave_incl_scan(nh);
    int wbase = 0;
    if (lane() == kWave - 1 && incl > 0) wbase = atomicAdd(s_pos, incl);
    wbase = __shfl(wbase, kWave - 1, kWave);
    int64_t at = ebase + wbase + (incl - nh);
#pragma unroll
    for (int q = 0; q < kChunk; ++q)
      if ((hits >> q) & 1u) write_tri(o, at++, x, oth, v[q]);
  }
  return static_cast<uint32_t>(__popc(hits));
}

template <int MODE, int kOut, int SLOTS>
__device__ __forceinline__ uint32_t chunk_hits(const int32_t* p, int len, const ProbeSet& ps, bool up_side,
                                               int32_t x, int32_t oth, const Out& o, int64_t ebase, int* s_pos,
                                               int32_t* wq, const PvCache<SLOTS>& pvc) {
  int32_t v[kChunk];
#pragma unroll
  for (int q = 0; q < kChunk; ++q) v[q] = p[q];
  return chunk_probe<MODE, kOut>(v, len, ps, up_side, x, oth, o, ebase, s_pos, wq, pvc);
}

// The streams that start in a window of kTiles * 64 chunks from w0 on: a bit
// per chunk (s_M), and per tile of 64 chunks the streams begun before it
// (s_tb).  Every stream sets its own bit; a lane per tile that looked for its
// streams one after another left the rest of the block waiting (R-MAT scale
// 20: core items 0.79 -> 0.69 ms, 2 KB bin 0.38 -> 0.33 ms; scale 24: 32 KB
// bin 1.40 -> 1.02 ms).  The caller has synchronised the block; it is synchronised
// on return.
template <int THREADS, int kTiles>
__device__ __forceinline__ void mark_window(int w0, int nslots, const int2* s_cl, uint64_t* s_M, int32_t* s_tb) {
  const int tid = threadIdx.x;
  for (int t = tid; t < kTiles; t += THREADS) s_M[t] = 0ull;
  __syncthreads();
  uint32_t* m = reinterpret_cast<uint32_t*>(s_M);
  for (int i = tid; i < nslots; i += THREADS) {
    const int f = s_cl[i].x - w0;
    if (f >= 0 && f < kTiles * kWave) atomicOr(&m[f >> 5], 1u << (f & 31));
  }
  __syncthreads();
  if (tid < kWave) {
    int lo = 0, hi = w0 > 0 ? nslots : 0;  // first stream starting at or after w0
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (s_cl[mid].x < w0) lo = mid + 1;
      else hi = mid;
    }
#pragma unroll
    for (int t0 = 0; t0 < kTiles; t0 += kWave) {
      const int t = t0 + tid;
      const int k = t < kTiles ? __popcll(s_M[t]) : 0;
      const int incl = wave_incl_scan(k);
      if (t < kTiles) s_tb[t] = lo + incl - k;
      lo += wave_read(incl, kWave - 1);
    }
  }
  __syncthreads();
}

// All chunks of one batch of streams.  The chunk space [0, C) is walked in
// windows of THREADS * kWinIters chunks, each split into tiles of 64 chunks,
// one per wave and round (mark_window).  Lane i of a wave then finds the
// stream of its chunk as s_tb + popcount(mask bits <= i) - 1, with no search.
template <int MODE, int THREADS, int kOut, int kAhead, int SLOTS>
__device__ __forceinline__ uint32_t run_chunks(int C, int nslots, const int2* s_cl, const int64_t* s_beg,
                                               const int32_t* s_oth, uint64_t* s_M,
                                               int32_t* s_tb, const int32_t* lc, const ProbeSet& ps, int32_t x,
                                               const Out& o, int64_t ebase, int* s_pos, int32_t* s_q,
                                               const PvCache<SLOTS>& pvc) {
  constexpr int kWin = THREADS * kWinIters;
  constexpr int kTiles = kWin / kWave;
  static_assert(THREADS % kWave == 0, "block must be whole waves");
  const int tid = threadIdx.x;
  const uint32_t ln = static_cast<uint32_t>(lane());
  uint32_t cnt = 0;
  for (int w0 = 0; w0 < C; w0 += kWin) {
    mark_window<THREADS, kTiles>(w0, nslots, s_cl, s_M, s_tb);
    int32_t* wq = s_q + (tid & ~(kWave - 1));  // this wave's queue
    if (kOut != kOutEmit && kAhead == 1) {
      // every lane of a wave with work takes part (a lane past the end
      // probes nothing); a wave with none skips the round
#pragma unroll 2
      for (int i = 0; i < kWinIters; ++i) {
        if (w0 + i * THREADS >= C) break;  // the block's remaining slots are all past the end
        const int rel = i * THREADS + tid;
        const int c = w0 + rel;
        if (__ballot(c < C) == 0) continue;
        const int32_t* p = lc;
        int len = 0;
        int32_t ot = 0;
        bool upside = false;
        if (c < C) {
          const int t = rel >> 6;
          const uint64_t M = s_M[t];
          const int below = static_cast<int>(__builtin_amdgcn_mbcnt_hi(
              static_cast<uint32_t>(M >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(M), 0u)));
          const int j = s_tb[t] + below + static_cast<int>((M >> ln) & 1ull) - 1;
          const int2 cl = s_cl[j];
          const int k = c - cl.x;
          p = lc + s_beg[j] + static_cast<int64_t>(k) * kChunk;
          len = (cl.y & kLenMask) - k * kChunk;
          if (kOut == kOutPV) ot = j;
          upside = (cl.y & kClUp) != 0;
        }
        cnt += chunk_hits<MODE, kOut>(p, len, ps, upside, x, ot, o, ebase, s_pos, wq, pvc);
      }
    } else if (kOut != kOutEmit) {
      // kAhead chunk slots per lane at a time: every slot's loads are issued
      // before any is probed (a slot past the end reads entry 0 and probes
      // nothing), so a wave keeps kAhead chunks of memory reads in flight
      for (int i = 0; i < kWinIters; i += kAhead) {
        if (w0 + i * THREADS >= C) break;  // the block's remaining slots are all past the end
        int len[kAhead];
        int64_t e[kAhead];
        int32_t oth[kAhead];
        bool up[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int rel = (i + u) * THREADS + tid;
          const int c = w0 + rel;
          len[u] = 0;
          e[u] = 0;
          oth[u] = 0;
          up[u] = false;
          if (c < C) {
            const int t = rel >> 6;
            const uint64_t M = s_M[t];
            const int below = static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                static_cast<uint32_t>(M >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(M), 0u)));
            const int j = s_tb[t] + below + static_cast<int>((M >> ln) & 1ull) - 1;
            const int2 cl = s_cl[j];
            const int k = c - cl.x;
            e[u] = s_beg[j] + static_cast<int64_t>(k) * kChunk;
            len[u] = (cl.y & kLenMask) - k * kChunk;
            if (kOut == kOutPV) oth[u] = j;
            up[u] = (cl.y & kClUp) != 0;
          }
        }
        int32_t v[kAhead][kChunk];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
          for (int q = 0; q < kChunk; ++q) v[u][q] = lc[e[u] + q];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
          cnt += chunk_probe<MODE, kOut>(v[u], len[u], ps, up[u], x, oth[u], o, ebase, s_pos, wq, pvc);
      }
    } else {
      // writing triangles: the whole wave takes part in every round (the
      // writes are placed by a wave scan); lanes past the end probe nothing
#pragma unroll 2
      for (int i = 0; i < kWinIters; ++i) {
        const int rel = i * THREADS + tid;
        const int c = w0 + rel;
        const int32_t* p = lc;
        int len = 0;
        int32_t ot = 0;
        bool upside = false;
        if (c < C) {
          const int t = rel >> 6;
          const uint64_t M = s_M[t];
          const int below = static_cast<int>(__builtin_amdgcn_mbcnt_hi(
              static_cast<uint32_t>(M >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(M), 0u)));
          const int j = s_tb[t] + below + static_cast<int>((M >> ln) & 1ull) - 1;
          const int2 cl = s_cl[j];
          const int k = c - cl.x;
          p = lc + s_beg[j] + static_cast<int64_t>(k) * kChunk;
          len = (cl.y & kLenMask) - k * kChunk;
          ot = s_oth[j];
          upside = (cl.y & kClUp) != 0;
        }
        cnt += chunk_hits<MODE, kOut>(p, len, ps, upside, x, ot, o, ebase, s_pos, wq, pvc);
      }
    }
    __syncthreads();
  }
  return cnt;
}

// One block per work item (anchor x, range of resolved streams).  WORDS is
// the LDS table size in 32-bit words (0: search the sorted rows); the item
// says whether the anchor's table is a bitmap or a hash table.  Stream records are
// loaded D at a time (R per thread), the non-empty ones are compacted into
// LDS with their first chunk, and run_chunks streams them.
template <int WORDS, int THREADS, int D, int WPE, int kOut, bool kRoundRobin>
__global__ __launch_bounds__(THREADS, WPE) void heavy_kernel(const int32_t* lc, const VMeta* meta, int bin,
                                                        const int4* items, const int64_t* sbeg,
                                                        const int32_t* slen, const int32_t* soth,
                                                        const uint32_t* tl_words, const uint32_t* tl_l1,
                                                        unsigned long long* acc, Out o) {
  constexpr int R = D / THREADS;  // records loaded per thread
  static_assert(R * THREADS == D, "D must be a multiple of THREADS");
  constexpr int kTiles = THREADS * kWinIters / kWave;
  __shared__ uint32_t tab[WORDS > 0 ? WORDS : 1];
  __shared__ int64_t s_beg[D];
  __shared__ int2 s_cl[D + 1];  // (first chunk, length) of each non-empty stream
  __shared__ int32_t s_oth[needs_oth(kOut) ? D : 1];
  __shared__ int s_pos;  // triangles of the current item written so far (kOutEmit)
  __shared__ uint64_t s_M[kTiles];
  __shared__ int32_t s_tb[kTiles];
  __shared__ int32_t s_q[WORDS > 0 ? THREADS : 1];  // per wave: its queue of pending hash probes
  __shared__ int64_t sh[THREADS / kWave + 1];
  __shared__ int32_t shi[THREADS / kWave + 1];
  __shared__ unsigned long long s_item;
  // slots for the apexes' counts: 2 KB bin 128 / 256 / 512 / 1024 of them 15.2 /
  // 14.6 / 11.1 / 11.2 ms at R-MAT scale 20 (one slot an apex); 32 KB bin 512 /
  // 1024 / 2048 of them 42.5 / 22.4 / 14.6 ms, 4096 leave room for one block a
  // CU (10.7 ms against 8.9 with four slots an apex)
  constexpr int kPv = kOut != kOutPV ? 0 : (WORDS == kBinWords0 ? 512 : (WORDS == kBinWords2 ? 512 : 2048));
  __shared__ uint32_t s_pk[kPv > 0 ? kPv : 1];
  __shared__ int32_t s_ps[kPv > 0 ? kPv : 1];
  // the streamed lists' counts, one atomic to memory per stream (one per chunk
  // with a hit took 6.1 ms more on the R-MAT graph above, 0.23 ms on the other)
  __shared__ int32_t s_os[kPv > 0 ? D : 1];
  const PvCache<kPv> pvc{s_pk, s_ps, s_os};
  int32_t pv_x = -1;
  if (kPv > 0)
    for (int i = threadIdx.x; i < D; i += THREADS) s_os[i] = 0;
  for (int i = threadIdx.x; i < kPv; i += THREADS) {
    s_pk[i] = kPvFree;
    s_ps[i] = 0;
  }

  const unsigned long long first = acc[kAccBinOff + bin];
  const unsigned long long count = acc[kAccBinCount + bin];
  // nothing for this block (all of an empty bin's, whose sums took 16 us)
  if (kRoundRobin ? blockIdx.x >= count : count == 0) return;
  const int tid = threadIdx.x;
  int64_t cnt = 0, elems = 0, builds = 0, tl_elems = 0;
  int32_t cur_x = -1;
  bool cur_rest = false;
  // blocks claim kC consecutive items at a time (consecutive items of
  // one anchor share the table); the next claim is fetched while the
  // current one is processed.  kRoundRobin: block b takes items b, b + G,
  // b + 2G, ... (G blocks) one at a time, with no counter.
  constexpr unsigned long long kC = kRoundRobin ? 1 : (WORDS == kBinWords0 ? kClaimSmall : (kOut == kOutPV ? kClaimPv : kClaim));
  if (tid == 0)
    s_item = kRoundRobin ? static_cast<unsigned long long>(blockIdx.x)
                         : atomicAdd(&acc[kAccBinNext + bin], kC);
  __syncthreads();
  unsigned long long claim = s_item;
  while (claim < count) {
    unsigned long long next = 0;
    if (tid == 0)
      next = kRoundRobin ? claim + gridDim.x
                         : atomicAdd(&acc[kAccBinNext + bin], kC);
    const unsigned long long claim_end = min(claim + kC, count);
    for (unsigned long long it = claim; it < claim_end; ++it) {
    const int64_t gi = static_cast<int64_t>(first + it);  // unit index of this item
    const int4 item = items[gi];
    const int32_t x = item.x;
    const int64_t sa = static_cast<int64_t>(static_cast<uint32_t>(item.y)) | (static_cast<int64_t>(item.z) << 32);
    const int64_t sb = sa + (item.w & kItemCountMask);
    VMeta mx = meta[x];
    const bool rest = (item.w & kItemRest) != 0;
    if (rest) mx = rest_meta(mx);
    if (kPv > 0 && x != pv_x) {  // the last item's barriers are behind its additions
      pvc.flush(o.pv, THREADS);
      __syncthreads();
      pv_x = x;
    }
    const int P = mx.up + (mx.sfe - mx.hfb);
    ProbeSet ps;
    ps.tab = tab;
    ps.lo = 0;
    ps.R = 0;
    ps.cap = 64;
    ps.shift = 26;
    ps.up_row = lc + mx.begin;
    ps.up_len = mx.up;
    ps.hf_row = lc + mx.begin + mx.hfb;
    ps.hf_len = mx.sfe - mx.hfb;
    ps.nw = 0;
    ps.words = tl_words + mx.begin;
    int mode = kSearch;
    if (WORDS > 0) {
      const SplitWindow sw = split_window(lc, mx);
      int64_t R64;
      joint_window(sw, ps.lo, R64);
      ps.R = static_cast<uint32_t>(R64);
      ps.lo_up = sw.lo_up;
      ps.lo_hf = sw.lo_hf;
      ps.R_up = static_cast<uint32_t>(sw.R_up);
      ps.R_hf = static_cast<uint32_t>(sw.R_hf);
      ps.off_hf = static_cast<uint32_t>(bitmap_words(sw.R_up));
      mode = (item.w & kItemBitmap) ? kBitmap : ((item.w & kItemTwoLevel) ? kTwoLevel : kHash);
      ps.cap = WORDS;
      ps.shift = 32 - __builtin_ctz(WORDS);
      ps.nw = static_cast<int>(twolevel_words(R64) >> 1);
      if (x != cur_x || rest != cur_rest) {
        if (WORDS == kBinWords2 && mode == kTwoLevel) {
          // the block bits as the planning pass wrote them at the anchor's
          // row positions, then per word the number of set bits before it
          const uint32_t* lx = tl_l1 + mx.begin;
          const int nw = ps.nw;
          constexpr int kPer = WORDS > 0 ? (WORDS / 2 + THREADS - 1) / THREADS : 1;  // words per thread
          uint32_t wv[kPer];
          int mine = 0;
#pragma unroll
          for (int j = 0; j < kPer; ++j) {
            const int i = tid * kPer + j;
            wv[j] = i < nw ? lx[i] : 0u;
            mine += __popc(wv[j]);
          }
          int32_t tot;
          int run = block_excl_scan(mine, shi, &tot);
#pragma unroll
          for (int j = 0; j < kPer; ++j) {
            const int i = tid * kPer + j;
            if (i < nw) {
              tab[i] = wv[j];
              tab[nw + i] = static_cast<uint32_t>(run);
            }
            run += __popc(wv[j]);
          }
        } else if (mode == kBitmap) {
          const int words = static_cast<int>(ps.off_hf + bitmap_words(sw.R_hf));
          for (int i = tid; i < words; i += THREADS) tab[i] = 0u;
          __syncthreads();
          for (int i = tid; i < P; i += THREADS) {
            const bool upm = i < mx.up;
            const int32_t key = upm ? lc[mx.begin + i] : lc[mx.begin + mx.hfb + (i - mx.up)];
            const uint32_t d = static_cast<uint32_t>(key - (upm ? ps.lo_up : ps.lo_hf));
            atomicOr(&tab[(upm ? 0u : ps.off_hf) + (d >> 5)], 1u << (d & 31));
          }
        } else {
          for (int i = tid; i < ps.cap; i += THREADS) tab[i] = kHashEmpty;
          __syncthreads();
          for (int i = tid; i < P; i += THREADS) {
            const int32_t key = i < mx.up ? lc[mx.begin + i] : lc[mx.begin + mx.hfb + (i - mx.up)];
            const uint32_t h0 = hslot(key, ps.shift);
            uint32_t h = h0;
            while (atomicCAS(&tab[h], kHashEmpty, static_cast<uint32_t>(key)) != kHashEmpty)
              h = (h + 1) & (ps.cap - 1);
            if (h != h0) atomicOr(&tab[h0], kHashMoved);  // the home is occupied, so it stays a key
          }
        }
        __syncthreads();
        cur_x = x;
        cur_rest = rest;
        // ids inserted (bitmap, hash) or words copied (two-level)
        builds += tid == 0 ? (mode == kTwoLevel ? ps.nw : P) : 0;
      }
    }
    int64_t ebase = 0;
    int32_t hx = x;  // the anchor as hits report it (a caller id when writing triangles)
    if (kOut == kOutEmit) {
      hx = caller_id(o, x);
      ebase = o.uoff[gi];
      if (tid == 0) s_pos = 0;
      __syncthreads();
    }
    int64_t icnt = 0;
    for (int64_t bs = sa; bs < sb; bs += D) {
      const int nd = static_cast<int>(min(static_cast<int64_t>(D), sb - bs));
      int64_t lbeg[R];
      int32_t llen[R], loth[R];
      bool lup[R];
      int nne = 0, nch = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int dl = tid * R + r;
        lbeg[r] = 0;
        llen[r] = 0;
        loth[r] = x;
        lup[r] = false;
        if (dl < nd) {
          const int64_t k = bs + dl;
          const int32_t lf = slen[k];
          lbeg[r] = sbeg[k];
          llen[r] = lf & kLenMask;
          lup[r] = (lf & kFlagUp) != 0;
          if (needs_oth(kOut)) loth[r] = kOut == kOutEmit ? caller_id(o, soth[k]) : soth[k];
        }
        if (llen[r] > 0) {
          ++nne;
          nch += (llen[r] + kChunk - 1) / kChunk;
          elems += llen[r];
          if (mode == kTwoLevel) tl_elems += llen[r];
        }
      }
      int32_t nslots, C;
      int slot = block_excl_scan(nne, shi, &nslots);
      int cb = block_excl_scan(nch, shi, &C);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (llen[r] <= 0) continue;
        s_cl[slot] = make_int2(cb, llen[r] | (lup[r] ? kClUp : 0));
        s_beg[slot] = lbeg[r];
        if (needs_oth(kOut)) s_oth[slot] = loth[r];
        cb += (llen[r] + kChunk - 1) / kChunk;
        ++slot;
      }
      if (tid == 0) s_cl[nslots] = make_int2(C, 0);
      __syncthreads();
      uint32_t got;
      if (WORDS == 0) {
        got = run_chunks<kSearch, THREADS, kOut, ahead_of<WORDS>()>(C, nslots, s_cl, s_beg, s_oth, s_M, s_tb, lc, ps, hx, o,
                                                 ebase, &s_pos, s_q, pvc);
      } else if (mode == kBitmap) {
        got = run_chunks<kBitmap, THREADS, kOut, ahead_of<WORDS>()>(C, nslots, s_cl, s_beg, s_oth, s_M, s_tb, lc, ps, hx, o,
                                                 ebase, &s_pos, s_q, pvc);
      } else if (WORDS == kBinWords2 && mode == kTwoLevel) {
        got = run_chunks<kTwoLevel, THREADS, kOut, ahead_of<WORDS>()>(C, nslots, s_cl, s_beg, s_oth, s_M, s_tb, lc, ps, hx, o,
                                                   ebase, &s_pos, s_q, pvc);
      } else {
        got = run_chunks<kHash, THREADS, kOut, ahead_of<WORDS>()>(C, nslots, s_cl, s_beg, s_oth, s_M, s_tb, lc, ps, hx, o,
                                               ebase, &s_pos, s_q, pvc);
      }
      if (kOut == kOutPV)  // (run_chunks ends with a barrier)
        for (int i = tid; i < nslots; i += THREADS) {
          if (s_os[i]) add_pv(o.pv, s_oth[i], s_os[i]);
          s_os[i] = 0;
        }
      // the per-item count is kept only where it is recorded
      if (kOut == kOutRec || kOut == kOutPV) icnt += got;
      else cnt += got;
    }
    if (kOut == kOutRec || kOut == kOutPV) {
      cnt += icnt;
      const int64_t t = block_sum(icnt, sh);
      if (kOut == kOutRec && tid == 0) o.ucnt[gi] = static_cast<int32_t>(t);
      if (kOut == kOutPV && tid == 0 && t) add_pv(o.pv, x, t);
    }
    }
    __syncthreads();
    if (tid == 0) s_item = next;
    __syncthreads();
    claim = s_item;
  }
  if (kPv > 0) pvc.flush(o.pv, THREADS);
  if (kOut == kOutEmit) return;
  block_acc(acc, kAccT, cnt, sh);
  block_acc(acc, kAccHeavyElems, elems, sh);
  block_acc(acc, kAccBinElems + bin, elems, sh);
  block_acc(acc, kAccBuild, builds, sh);
  block_acc(acc, kAccTwoLevelElems, tl_elems, sh);
}


// ---------------------------------------------------- core items
// The core parts of an anchor's streams (kBinCore): the lists' 16-bit offsets
// c16 against two bitmaps of the core, 8 KB for the level above (Up(x)) and
// 8 KB for the row's own (Hfwd(x)); entries outside the core read as kNoCore,
// whose bit stays clear.  At R-MAT scale 24 the 32 KB bin streamed 48.8 G
// elements as 32-bit ids in 33.0 ms; with half the bytes, half the table
// (four blocks a CU instead of three) and no window to subtract and clamp they
// take 18.4 ms.  Bound by the lines it requests: 1.18 G of 128 bytes, 94% of
// them past the L2, are 7.9 TB/s (the VALU is busy 72% of the time, the LDS
// 53%).
// A chunk is kCoreChunk elements from an even position (dword loads); an odd
// stream's first chunk starts one element early, which is masked.
constexpr int kCoreThreads = 512, kCoreRecs = 1024, kCoreChunk = 16;
constexpr int kCoreWords = (kCoreIds + 1) / 32;  // of one bitmap

__global__ __launch_bounds__(kCoreThreads, 8) void core_kernel(const uint16_t* c16, const VMeta* meta, const int4* items,
                                                               const int64_t* sbeg, const int32_t* slen,
                                                               unsigned long long* acc) {
  constexpr int R = kCoreRecs / kCoreThreads, NW = kCoreThreads / kWave;
  constexpr int kWin = kCoreThreads * kWinIters, kTiles = kWin / kWave;
  static_assert(R * kCoreThreads == kCoreRecs, "whole records per thread");
  static_assert(kCoreChunk <= kColPad, "chunk tail must stay inside the padded columns");
  __shared__ alignas(16) uint32_t tab[2 * kCoreWords];
  __shared__ int64_t s_beg[kCoreRecs];
  __shared__ int2 s_cl[kCoreRecs + 1];  // (first chunk, length | kClUp)
  __shared__ uint64_t s_M[kTiles];
  __shared__ int32_t s_tb[kTiles];
  __shared__ int64_t sh[NW + 1];
  __shared__ int32_t shi[NW + 1];
  __shared__ unsigned long long s_item;
  const unsigned long long first = acc[kAccBinOff + kBinCore];
  const unsigned long long count = acc[kAccBinCount + kBinCore];
  if (count == 0) return;
  const int tid = threadIdx.x;
  const uint32_t ln = static_cast<uint32_t>(lane());
  int64_t cnt = 0, elems = 0, builds = 0;
  int32_t cur_x = -1;
  // items are claimed kClaim at a time, the next claim while these run
  if (tid == 0) s_item = atomicAdd(&acc[kAccBinNext + kBinCore], static_cast<unsigned long long>(kClaim));
  __syncthreads();
  unsigned long long claim = s_item;
  while (claim < count) {
    unsigned long long next = 0;
    if (tid == 0) next = atomicAdd(&acc[kAccBinNext + kBinCore], static_cast<unsigned long long>(kClaim));
    const unsigned long long claim_end = min(claim + kClaim, count);
    for (unsigned long long it = claim; it < claim_end; ++it) {
      const int4 item = items[first + it];
      const int32_t x = item.x;
      const int64_t sa = static_cast<int64_t>(static_cast<uint32_t>(item.y)) | (static_cast<int64_t>(item.z) << 32);
      const int nrec = item.w & kItemCountMask;
      if (x != cur_x) {
        const VMeta mx = meta[x];
        for (int i = tid; i < 2 * kCoreWords / 4; i += kCoreThreads)
          reinterpret_cast<uint4*>(tab)[i] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        const int nu = mx.up - mx.ncu, nh = mx.sfe - mx.hfb - mx.nch;
        for (int i = tid; i < nu + nh; i += kCoreThreads) {
          const bool up = i < nu;
          const uint32_t v = c16[mx.begin + (up ? mx.ncu + i : mx.hfb + mx.nch + (i - nu))];
          atomicOr(&tab[(up ? 0 : kCoreWords) + (v >> 5)], 1u << (v & 31));
        }
        __syncthreads();
        cur_x = x;
        builds += tid == 0 ? nu + nh : 0;
      }
      for (int bs = 0; bs < nrec; bs += kCoreRecs) {
        int64_t lbeg[R];
        int32_t llen[R];
        int nne = 0, nch = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int dl = bs + tid * R + r;
          lbeg[r] = 0;
          llen[r] = 0;
          if (dl < nrec) {
            lbeg[r] = sbeg[sa + dl];
            llen[r] = slen[sa + dl];
          }
          const int len = llen[r] & kLenMask;
          if (len > 0) {
            ++nne;
            nch += (len + static_cast<int>(lbeg[r] & 1) + kCoreChunk - 1) / kCoreChunk;
            elems += len;
          }
        }
        int32_t nslots, C;
        int slot = block_excl_scan(nne, shi, &nslots);
        int cb = block_excl_scan(nch, shi, &C);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int len = llen[r] & kLenMask;
          if (len <= 0) continue;
          s_cl[slot] = make_int2(cb, len | ((llen[r] & kFlagUp) ? kClUp : 0));
          s_beg[slot] = lbeg[r];
          cb += (len + static_cast<int>(lbeg[r] & 1) + kCoreChunk - 1) / kCoreChunk;
          ++slot;
        }
        __syncthreads();
        for (int w0 = 0; w0 < C; w0 += kWin) {
          mark_window<kCoreThreads, kTiles>(w0, nslots, s_cl, s_M, s_tb);
#pragma unroll 2
          for (int i = 0; i < kWinIters; ++i) {
            const int rel = i * kCoreThreads + tid;
            const int c = w0 + rel;
            if (w0 + i * kCoreThreads >= C) break;
            if (c >= C) continue;
            const uint64_t M = s_M[rel >> 6];
            const int below = static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                static_cast<uint32_t>(M >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(M), 0u)));
            const int j = s_tb[rel >> 6] + below + static_cast<int>((M >> ln) & 1ull) - 1;
            const int2 cl = s_cl[j];
            const int k = c - cl.x;
            const int64_t beg = s_beg[j];
            const int lead = static_cast<int>(beg & 1);
            const int rem = (cl.y & kLenMask) + lead - k * kCoreChunk;
            uint32_t valid = rem >= kCoreChunk ? (1u << kCoreChunk) - 1u : (1u << rem) - 1u;
            if (k == 0) valid &= ~static_cast<uint32_t>(lead);
            const uint32_t part = (cl.y & kClUp) ? 0u : static_cast<uint32_t>(kCoreWords) * 4u;
            const uint32_t* p = reinterpret_cast<const uint32_t*>(c16 + (beg - lead)) + k * (kCoreChunk / 2);
            uint32_t d[kCoreChunk / 2];
#pragma unroll
            for (int q = 0; q < kCoreChunk / 2; ++q) d[q] = p[q];
            const char* tb = reinterpret_cast<const char*>(tab);
            uint32_t hits = 0;
#pragma unroll
            for (int q = 0; q < kCoreChunk / 2; ++q) {
              const uint32_t lo = *reinterpret_cast<const uint32_t*>(tb + (((d[q] >> 3) & 0x1FFCu) | part));
              const uint32_t hi = *reinterpret_cast<const uint32_t*>(tb + (((d[q] >> 19) & 0x1FFCu) | part));
              hits |= __builtin_amdgcn_ubfe(lo, d[q] & 31u, 1u) << (2 * q);
              hits |= __builtin_amdgcn_ubfe(hi, (d[q] >> 16) & 31u, 1u) << (2 * q + 1);
            }
            cnt += __popc(hits & valid);
          }
          __syncthreads();
        }
      }
    }
    __syncthreads();
    if (tid == 0) s_item = next;
    __syncthreads();
    claim = s_item;
  }
  block_acc(acc, kAccT, cnt, sh);
  block_acc(acc, kAccHeavyElems, elems, sh);
  block_acc(acc, kAccBuild, builds, sh);
}

// Clears the accumulators and the statistics.
__global__ void count_init_kernel(unsigned long long* acc, int64_t* stats) {
  for (int i = threadIdx.x; i < kAccAll; i += blockDim.x) acc[i] = 0ull;
  if (threadIdx.x < 24) stats[threadIdx.x] = 0;
}

__global__ __launch_bounds__(kWave) void finish_kernel(const unsigned long long* sums, const int64_t* so, int64_t n,
                                                       int64_t nnz, int64_t num_levels, const int64_t* lpre,
                                                       int64_t nchunk_cap, int64_t* triangles, int64_t* h_count,
                                                       int64_t* stats) {
  __shared__ unsigned long long acc[kWave];
  static_assert(kAccSlots <= kWave, "a lane per slot");
  if (threadIdx.x < kAccSlots) {
    unsigned long long v = sums[threadIdx.x];
#pragma unroll
    for (int i = 1; i <= kAccStripes; ++i) v += sums[kAccPad * i + threadIdx.x];
    acc[threadIdx.x] = v;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  stats[0] = n;
  stats[1] = nnz;
  stats[3] = num_levels;
  *triangles = static_cast<int64_t>(acc[kAccT]);
  if (h_count) *h_count = static_cast<int64_t>(acc[kAccH]);
  stats[2] = static_cast<int64_t>(acc[kAccH]);
  stats[4] = static_cast<int64_t>(acc[kAccElems] + acc[kAccHeavyElems]);
  stats[5] = n > 0 ? lpre[nchunk_cap] : 0;
  stats[6] = static_cast<int64_t>(acc[kAccItems]);
  stats[7] = static_cast<int64_t>(acc[kAccRecs]);
  stats[8] = static_cast<int64_t>(acc[kAccHeavyElems]);
  stats[9] = static_cast<int64_t>(acc[kAccBuild]);
  stats[10] = static_cast<int64_t>(acc[kAccElems]);
  for (int b = 0; b < 4; ++b) {
    stats[11 + b] = static_cast<int64_t>(acc[kAccBinElems + b]);
    stats[15 + b] = static_cast<int64_t>(acc[kAccBinCount + b]);
  }
  stats[19] = n > 0 ? so[n] : 0;
  stats[20] = static_cast<int64_t>(acc[kAccTwoLevelElems]);
}

__global__ void forward_meta_kernel(const int64_t* off, const int32_t* cols, int64_t n, VMeta* meta) {
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = off[x], e = off[x + 1];
    const int64_t fb = upper_bound_dev(cols, b, e, static_cast<int32_t>(x));
    const int32_t deg = static_cast<int32_t>(e - b);
    meta[x] = VMeta{b, 0, static_cast<int32_t>(fb - b), deg, deg, 0, 0};
  }
}


// WPE: waves per SIMD the kernel is compiled for (HIP's second launch
// bound), matched to the blocks per CU that the bin's LDS allows.
template <int WORDS, int THREADS, int D, int WPE, int kOut, bool kRoundRobin = false>
int launch_heavy(const CountArgs& a, CountWs& w, const Out& o, int bin, int blocks_per_cu, hipStream_t s) {
  heavy_kernel<WORDS, THREADS, D, WPE, kOut, kRoundRobin><<<static_cast<unsigned>(num_cus() * blocks_per_cu), THREADS, 0, s>>>(
      a.cols, a.meta, bin, w.items, w.sbeg, w.slen, w.soth, w.tl_words, w.tl_l1, w.acc, o);
  TC_HIP(hipGetLastError());
  return TC_OK;
}

// Bin 0: blocks taking items round robin, or one-wave blocks claiming them
// (count_params picks by graph size).  Round robin, four waves a block while
// the items are too few to go round many times (8185 of up to 2^14 elements
// at R-MAT scale 16: whole count 0.60 -> 0.56 ms; scale 18 1.09 -> 1.08),
// two beyond (scale 19 1.79 ms against 1.82 with four).
template <int kOut>
int launch_bin0(const CountArgs& a, CountWs& w, const Out& o, hipStream_t s) {
  if (a.prm.bin0_mode != 2) return launch_heavy<kBinWords0, 64, 256, 6, kOut>(a, w, o, 0, 24, s);
  if (a.g->nnz < (int64_t(1) << 23)) return launch_heavy<kBinWords0, 256, 256, 6, kOut, true>(a, w, o, 0, 6, s);
  return launch_heavy<kBinWords0, 128, 256, 6, kOut, true>(a, w, o, 0, 12, s);
}

// The four bins of heavy items, one after another on the call's stream
// (bins_mode 1) or side by side on forked streams (2).
template <int kOut>
int launch_bins(const CountArgs& a, CountWs& w, const Out& o, hipStream_t s) {
  if (a.c16) {  // the largest share of the work first
    core_kernel<<<static_cast<unsigned>(num_cus() * 4), kCoreThreads, 0, s>>>(a.c16, a.meta, w.items, w.sbeg, w.slen,
                                                                             w.acc);
    TC_HIP(hipGetLastError());
  }
  if (a.prm.bins_mode == 1) {
    // by the largest degree, no probe set may need the largest tables: a hash
    // table of 2 deg words fits 32 KB, as do two bitmaps over all ids
    const bool bin2 = 2 * std::min(a.maxdeg, a.g->nnz) > kBinWords1 || 2 * (a.g->n / 32 + 2) > kBinWords1;
    const bool bin3 = 2 * std::min(a.maxdeg, a.g->nnz) > kBinWords2;
    if (bin2) TC_TRY((launch_heavy<kBinWords2, 1024, 1024, 4, kOut>(a, w, o, 2, 1, s)));
    TC_TRY((launch_heavy<kBinWords1, 512, 1024, 6, kOut>(a, w, o, 1, 3, s)));
    TC_TRY(launch_bin0<kOut>(a, w, o, s));
    return bin3 ? launch_heavy<0, 512, 1024, 4, kOut>(a, w, o, 3, 4, s) : TC_OK;
  }
  Fork* f = fork_for_device();
  if (!f) return TC_ERR_HIP;
  TC_TRY(fork_begin(f, s));
  TC_TRY((launch_heavy<kBinWords2, 1024, 1024, 4, kOut>(a, w, o, 2, 1, s)));
  TC_TRY((launch_heavy<kBinWords1, 512, 1024, 6, kOut>(a, w, o, 1, 3, f->aux[0])));
  TC_TRY(launch_bin0<kOut>(a, w, o, f->aux[1]));
  TC_TRY((launch_heavy<0, 512, 1024, 4, kOut>(a, w, o, 3, 4, f->aux[2])));
  return fork_end(f, s);
}

template <int kOut>
int launch_light(const CountArgs& a, CountWs& w, const Out& o, hipStream_t s) {
  // one thread per task; there are at most two tasks per CSR entry
  const int64_t need = (2 * (a.g->nnz + 1) + kThreads - 1) / kThreads;
  const int64_t cap = static_cast<int64_t>(num_cus()) * 16;
  light_kernel<kOut><<<static_cast<unsigned>(need < cap ? need : cap), kThreads, 0, s>>>(
      a.cols, a.meta, w.so, a.g->n, w.lpre, w.ltab, w.nchunk_cap, w.sbeg, w.slen, w.soth, w.sx, w.acc, o);
  TC_HIP(hipGetLastError());
  return TC_OK;
}

template <bool kCover, int kOut>
int launch_all(const CountArgs& a, CountWs& w, const Out& o, hipStream_t s) {
  const int64_t n = a.g->n;
  const unsigned gv = grid_for(n, kThreads, 16384);
  // kernels over the resolve chunks need at most one block (resolve) or one
  // thread (bin split) per chunk; nchunk_cap bounds the chunk count
  const int64_t gmax = static_cast<int64_t>(num_cus()) * 16;
  const unsigned gr = static_cast<unsigned>(w.nchunk_cap < gmax ? w.nchunk_cap : gmax);
  const int64_t gct = (w.nchunk_cap + kThreads - 1) / kThreads;
  const unsigned gc = static_cast<unsigned>(gct < gmax ? gct : gmax);
  plan_kernel<kCover><<<gv, kThreads, 0, s>>>(a.cols, a.meta, n, w.ndesc, w.vinfo, w.pm, w.acc, a.prm,
                                               a.c16 != nullptr);
  TC_HIP(hipGetLastError());
  // a wave scans 64 vertices per round: about two rounds per wave (one
  // block of a graph of 16 K vertices scanned them in 19 us)
  // (only probe sets beyond the 32 KB hash table get a two-level one)
  if (2 * std::min(a.maxdeg, a.g->nnz) > kBinWords1)
    twolevel_words_kernel<<<grid_for(n, kThreads * 2, 4096), kThreads, 0, s>>>(a.cols, a.meta, w.vinfo, n, w.tl_words,
                                                                               w.tl_l1);
  TC_HIP(hipGetLastError());
  {
    Carver sc(w.scratch);
    TC_TRY(scan_exclusive<int32_t>(w.ndesc, w.so, n, sc, s));
  }
  chunk_start_kernel<<<gv, kThreads, 0, s>>>(w.so, n, w.cx0);
  TC_HIP(hipGetLastError());
  prof_stage("resolve");
  const bool lists = kCover && a.c16;
  if (lists)
    sample_kernel<<<grid_for(a.g->nnz / kSampStride + 1, kThreads, 16384), kThreads, 0, s>>>(a.cols, a.g->nnz, w.samp);
  const auto resolve = lists ? resolve_kernel<kCover, kCover> : resolve_kernel<kCover, false>;
  resolve<<<gr, kResThreads, 0, s>>>(a.cols, w.samp, a.meta, w.pm, w.vinfo, w.so, w.cx0, n, w.sbeg, w.slen, w.soth,
                                     w.sx, w.items_raw, w.ccnt, w.nchunk_cap, a.prm.item_log2, a.prm.up_anchor_min);
  TC_HIP(hipGetLastError());
  {
    Carver sc(w.scratch);
    TC_TRY(scan_exclusive_strided(reinterpret_cast<const int32_t*>(w.ccnt) + 1, 4, w.lpre, w.nchunk_cap, sc, s));
  }
  bin_split_kernel<false><<<gc, kThreads, 0, s>>>(w.so, n, w.ccnt, w.items_raw, w.items, w.lpre, w.ltab, w.acc);
  bin_split_kernel<true><<<gc, kThreads, 0, s>>>(w.so, n, w.ccnt, w.items_raw, w.items, w.lpre, w.ltab, w.acc);
  TC_HIP(hipGetLastError());
  // after the item split: kOutRec keeps its unit counts where the raw items were
  TC_TRY(launch_light<kOut>(a, w, o, s));
  prof_stage("heavy");
  TC_TRY(launch_bins<kOut>(a, w, o, s));
  prof_stage("finish");
  return TC_OK;
}

// Unit counts and offsets of triangle finding live in the raw-item buffer,
// which is dead once the items are split by bin: rcap int32 counts, then
// rcap + 1 int64 offsets (12 rcap + 8 <= 16 rcap bytes for rcap >= 2).
Out unit_out(CountWs& w) {
  Out o{};
  char* base = reinterpret_cast<char*>(w.items_raw);
  o.ucnt = reinterpret_cast<int32_t*>(base);
  o.uoff = reinterpret_cast<int64_t*>(base + ((4 * w.rcap + 7) & ~int64_t(7)));
  return o;
}

}  // namespace

// Graphs of at least this many entries stream the core parts of their lists
// as 16-bit ids (R-MAT scale 18 1.08 -> 1.07 ms, 20 3.16 -> 2.95, 22 14.2 ->
// 12.3, 24 65.0 -> 54.6; the layout's 16-bit ids cost 0.05 and 0.7 ms at 20
// and 24).  Below, levels are small enough for the 32-bit streams to stay in
// the caches.
constexpr int64_t kCoreNnz = int64_t(1) << 22;

int count_params(const tc_tuning* t, bool cover, int64_t nnz, CountParams* out) {
  CountParams p;
  p.light_max = kLightMax;
  p.dn_light = kDnLight;
  p.bm_member = 4;
  // cover count: 8 words per task (R-MAT S24 71.3 -> 69.7 ms, S20 3.71 ->
  // 3.63 ms, S22 within 0.5%); the comparator keeps 16
  p.bm_desc = cover ? 8 : 16;
  // work items of 2^14 elements below 2^24 entries, where the heavy work is
  // too small to fill the chip in 2^19-element items (R-MAT S14 0.708 ->
  // 0.682 ms, S16 0.886 -> 0.842, Chung-Lu n = 10^5 0.844 -> 0.834; S18
  // unchanged)
  p.item_log2 = nnz < (int64_t(1) << 24) ? 14 : kElemChunkLog;
  p.tl_sparsity = 64;
  // Bin 0 (tables of 2 KB): on smaller graphs its items are short (about 500
  // elements at R-MAT S20) and two waves per block with half the blocks
  // finish sooner, taking the items round robin (the claim counter's
  // same-address atomics and the spread of finish times over a 4-item claim
  // cost 0.1 ms of 0.42 at S20); on large graphs (2400 elements per item at
  // S24) the items vary more and one wave per block with claims does
  // (round robin loses 2.4 ms there).
  p.bin0_mode = cover && nnz < (int64_t(1) << 27) ? 2 : 1;
  // The table bins one after another or side by side on forked streams:
  // side by side, bin 0's many small blocks can take the CUs before a
  // larger bin's and the stage time varies from call to call; the cover
  // count runs faster and steadier in sequence (R-MAT S20 heavy stage 2.04
  // ms against a median of 2.28 ms side by side, S24 within 1.5%), the
  // comparator, whose work is spread over the small bins, side by side.
  p.bins_mode = cover ? 1 : 2;
  // an anchor with more than 1024 task descriptors skips the smallest-table
  // bin: its items would be streamed by one wave each (R-MAT S22 15.9 ->
  // 14.5 ms, S20 3.89 -> 3.72 ms; S24, 72.0 ms without the limit, 72.4)
  p.bin0_max_desc = 1024;
  // A down-class pair (x, w) may stream the shorter of Up(w) and Hfwd(x)
  // when Up(w) is long (w then holds one task descriptor per vertex of
  // Up(w)).  On for graphs of at least 2^26 entries: with the layout's
  // degree-ordered levels, R-MAT S24 67.8 -> 66.7 ms and S22 14.59 -> 14.31
  // ms at 256; at S20 it gains nothing (3.77 -> 3.76 ms).
  p.up_anchor_min = cover && nnz >= (int64_t(1) << 26) ? 256 : -1;
  // Four degree groups per level from 2^26 entries (R-MAT S24 8% fewer
  // streamed elements, 2 ms faster overall), two below, where the layout's
  // twelve groups cost more than the shorter forward lists gain (S20 3.61
  // -> 3.72 ms).
  p.degree_groups = nnz >= (int64_t(1) << 26) ? 4 : 2;
  p.core = cover && nnz >= kCoreNnz;
  if (t) {
    if (t->light_max) p.light_max = t->light_max;
    if (t->dn_light) p.dn_light = t->dn_light;
    if (t->bitmap_member_words) p.bm_member = t->bitmap_member_words;
    if (t->bitmap_desc_words) p.bm_desc = t->bitmap_desc_words;
    if (t->item_log2) p.item_log2 = t->item_log2;
    if (t->bin0_mode) p.bin0_mode = t->bin0_mode;
    if (t->bins_mode) p.bins_mode = t->bins_mode;
    if (t->twolevel_sparsity) p.tl_sparsity = t->twolevel_sparsity;
    if (t->bin0_max_desc) p.bin0_max_desc = t->bin0_max_desc;
    if (t->up_anchor_min) p.up_anchor_min = t->up_anchor_min;
    if (t->degree_groups) p.degree_groups = t->degree_groups;
  }
  if (p.light_max < 1 || p.light_max > kLightMax)
    return fail(TC_ERR_INVALID_ARG, "tuning: light_max must be in 1..%d", kLightMax);
  if (p.dn_light < 1) return fail(TC_ERR_INVALID_ARG, "tuning: dn_light must be >= 1");
  if (p.bm_member < 1 || p.bm_member > 1024 || p.bm_desc < 1 || p.bm_desc > 1024)
    return fail(TC_ERR_INVALID_ARG, "tuning: bitmap word factors must be in 1..1024");
  if (p.item_log2 < 12 || p.item_log2 > 24) return fail(TC_ERR_INVALID_ARG, "tuning: item_log2 must be in 12..24");
  if (p.tl_sparsity < -1) return fail(TC_ERR_INVALID_ARG, "tuning: twolevel_sparsity must be >= 1, or -1");
  if (p.bin0_max_desc < -1) return fail(TC_ERR_INVALID_ARG, "tuning: bin0_max_desc must be >= 1, or -1");
  // w must be a heavy anchor (a probe set above every light bound)
  if (p.degree_groups != 2 && p.degree_groups != 4)
    return fail(TC_ERR_INVALID_ARG, "tuning: degree_groups must be 2 or 4");
  if (p.up_anchor_min != -1 && p.up_anchor_min < kLightMax)
    return fail(TC_ERR_INVALID_ARG, "tuning: up_anchor_min must be >= %d, or -1", kLightMax);
  if (p.bin0_mode < 1 || p.bin0_mode > 2 || p.bins_mode < 1 || p.bins_mode > 2)
    return fail(TC_ERR_INVALID_ARG, "tuning: bin0_mode and bins_mode must be 1 or 2");
  *out = p;
  return TC_OK;
}

CountWs count_reserve(Carver& c, int64_t n, int64_t nnz) {
  CountWs w;
  w.ndesc = c.take<int32_t>(n + 1);
  w.vinfo = c.take<uint16_t>(n + 1);
  w.so = c.take<int64_t>(n + 2);
  // a vertex has at most deg(x) descriptors and a descriptor at most two
  // tasks, so 2 nnz bounds the stream records of heavy anchors (front) plus
  // the tasks of light anchors (back), and the work items, for any input
  w.rcap = 2 * nnz + 2;
  w.sbeg = c.take<int64_t>(w.rcap);
  w.slen = c.take<int32_t>(w.rcap);
  w.soth = c.take<int32_t>(w.rcap);
  w.sx = c.take<int32_t>(w.rcap);
  w.items_raw = c.take<int4>(w.rcap);
  w.items = c.take<int4>(w.rcap);
  // descriptors are at most nnz, so chunks at most nnz / kResChunk + 1
  w.nchunk_cap = nnz / kResChunk + 2;
  w.cx0 = c.take<int32_t>(w.nchunk_cap + 1);
  w.ccnt = c.take<int4>(w.nchunk_cap);
  w.lpre = c.take<int64_t>(w.nchunk_cap + 1);
  w.samp = c.take<int32_t>(nnz / kSampStride + 2);
  w.ltab = c.take<int32_t>(2 * nnz / kWave + 2);
  w.pm = c.take<uint4>(n + 1);
  w.tl_words = c.take<uint32_t>(nnz + 1);
  w.tl_l1 = c.take<uint32_t>(nnz + 1);
  w.acc = c.take<unsigned long long>(kAccAll);
  w.stats = c.take<int64_t>(24);
  // scans over vertices, over chunks and over the work units of triangle finding (<= rcap)
  w.scratch = c.take<char>(scan_ws_bytes(std::max(n + w.nchunk_cap + 1, w.rcap)) + 256);
  return w;
}

int forward_meta_run(const tc_csr* g, VMeta* meta, hipStream_t s) {
  if (g->n == 0) return TC_OK;
  forward_meta_kernel<<<grid_for(g->n, kThreads, 16384), kThreads, 0, s>>>(g->row_offsets, g->cols, g->n, meta);
  TC_HIP(hipGetLastError());
  return TC_OK;
}

int count_run(const CountArgs& a, CountWs& w, int64_t* triangles, int64_t* h_count, hipStream_t s) {
  const int64_t n = a.g->n;
  count_init_kernel<<<1, 1024, 0, s>>>(w.acc, w.stats);
  prof_stage("plan");
  if (n > 0) {
    Out o = unit_out(w);
    o.pv = a.per_vertex_out;
    o.order = a.order;
    if (!a.cover) TC_TRY((launch_all<false, kOutNone>(a, w, o, s)));
    else if (a.record_units) TC_TRY((launch_all<true, kOutRec>(a, w, o, s)));
    else if (a.per_vertex) TC_TRY((launch_all<true, kOutPV>(a, w, o, s)));
    else TC_TRY((launch_all<true, kOutNone>(a, w, o, s)));
  }
  finish_kernel<<<1, kWave, 0, s>>>(w.acc, w.so, n, a.g->nnz, a.num_levels, w.lpre, w.nchunk_cap, triangles, h_count,
                                    w.stats);
  TC_HIP(hipGetLastError());
  return TC_OK;
}

int list_run(const CountArgs& a, CountWs& w, int32_t* tri, int64_t cap, int64_t* triangles, int64_t* h_count,
             hipStream_t s) {
  CountArgs ra = a;
  ra.record_units = true;
  ra.per_vertex = false;
  TC_TRY(count_run(ra, w, triangles, h_count, s));
  if (a.g->n == 0 || cap == 0) return TC_OK;
  prof_stage("emit");
  // pass two: every work unit writes its triangles at the scanned offset of
  // its count (the number of units is read back first)
  int64_t host[2] = {0, 0};
  TC_HIP(hipMemcpyAsync(&host[0], w.acc + kAccItems, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  TC_HIP(hipMemcpyAsync(&host[1], w.lpre + w.nchunk_cap, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  TC_HIP(hipStreamSynchronize(s));
  const int64_t units = host[0] + host[1];
  if (units < 0 || units > w.rcap) return TC_ERR_HIP;
  Out o = unit_out(w);
  o.tri = tri;
  o.cap = cap;
  o.order = a.order;
  {
    Carver sc(w.scratch);
    TC_TRY(scan_exclusive<int32_t>(o.ucnt, const_cast<int64_t*>(o.uoff), units, sc, s));
  }
  TC_TRY(fill_i64(reinterpret_cast<int64_t*>(w.acc + kAccBinNext), 0, kBins, s));
  TC_TRY(launch_light<kOutEmit>(a, w, o, s));
  return launch_bins<kOutEmit>(a, w, o, s);
}

}  // namespace tc

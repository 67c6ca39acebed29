// direct_rule.h -- which graphs tc_count counts on the caller's CSR by the
// tiles of batch.hip, without the relabelling.  Plain C++, so that the rule
// and the bounds it rests on are checked without a GPU.
#pragma once

#include <stdint.h>

namespace tc {

constexpr int kTile = 512;       // forward entries of a piece counted together (their streams are kept in LDS)
constexpr int kBChunk = 8;       // consecutive list entries a lane takes at once
constexpr int kChunkBits = 22;   // of a tile's packed count of chunks and streams, the chunks' bits
constexpr uint32_t kLongList = 65536 - kBChunk;
// a tile whose lists are no longer than kLongList counts its chunks in kChunkBits
static_assert(kTile * ((kLongList + kBChunk - 1) / kBChunk) < (1u << kChunkBits), "a tile's chunks fit their field");

// The tiles stream sum over v of d+(v) (d(v) - d+(v)) elements, about a sixth of
// the squared degrees whatever the graph (within 10% on G(n, p), Chung-Lu and
// R-MAT graphs).  The relabelled path streams fewer where the degrees are
// uneven, but has its layout, plan and resolution to pay.  So the squared
// degrees beyond those of equal degrees (nnz^2 / n in all), and beyond the
// largest row's, whose streams are one vertex's, are set against what the
// layout costs: 168 an entry, 150 a vertex, and 2^28 for its launches.
// Measured both ways, us (relabelled / direct; then the excess in units of
// that cost, the direct count being taken up to 1):
//   G(n, d)          70001 d 8 224 / 145, 300007 d 24 701 / 241, 2000003 d 40
//                    11133 / 2333, 20011 d 1000 2896 / 1882 (0.00 to 0.01)
//   Barabasi-Albert  300007 d 12 516 / 262 (0.12), d 40 1177 / 760 (0.46)
//   Chung-Lu 2.1     30011 d 40 309 / 192 (0.37), 100003 d 20 354 / 314 (0.54),
//                    d 30 413 / 661 (0.80), d 40 467 / 730 (1.04), 300007 d 6
//                    474 / 387 (0.39), d 12 511 / 664 (0.77), d 20 725 / 1015
//                    (1.21), 1000003 d 6 1055 / 1026 (0.91), d 12 1350 / 1441
//                    (1.60), 2000003 d 6 1880 / 1785 (1.34)
//   Chung-Lu 2.5     300007 d 40 1374 / 1110 (0.94), 1000003 d 24 2331 / 1331
//                    (0.96)
//   R-MAT (scale, edge factor)  14, 16 282 / 142 (0.39), 15, 16 357 / 305 (0.91),
//                    16, 8 341 / 253 (0.80), 16, 16 415 / 1024 (1.88), 17, 4
//                    357 / 344 (0.62), 18, 3 448 / 568 (0.80), 18, 4 474 / 684
//                    (1.18), 20, 4 1045 / 2734 (3.01)
//   hubs of 65000    G(1000003, d 16) with one 1081 / 758 (0.00), eight 1180 /
//                    2003 (9.0)
// Between 0.5 and 1 no line divides the heavy tails (Chung-Lu 2.1, R-MAT) from
// the milder ones: some of the former lose a tenth to a half there, beyond 2 M
// entries, where a piece grows to 256 or 512 entries and a hub's keep a few
// blocks busy while the others have ended; the latter gain up to three times.
//
// The largest degree is at most kLongList: a longer forward list may stand at
// any vertex of a graph of more than 65536 of them, so that more than a few of
// a tile's 512 could be, and their chunks would not fit the field above.
// n and nnz: ids and positions of 32 bits in the streams.
inline bool direct_fits(int64_t n, int64_t nnz, int64_t maxdeg, uint64_t deg2) {
  if (n >= INT32_MAX || nnz >= (int64_t(1) << 31) || maxdeg > kLongList) return false;
  const uint64_t un = static_cast<uint64_t>(n < 1 ? 1 : n), uz = static_cast<uint64_t>(nnz);
  const uint64_t even = uz * uz / un + static_cast<uint64_t>(maxdeg) * static_cast<uint64_t>(maxdeg);
  return deg2 <= even + 168 * uz + 150 * un + (1ull << 28);
}

}  // namespace tc

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

// The streams are sum over v of d+(v) (d(v) - d+(v)) elements, about a sixth
// of the squared degrees whatever the graph (within 10% on G(n, p), Chung-Lu
// and R-MAT graphs).  The relabelled path streams fewer on graphs with hubs
// but has its layout, plan and resolution to pay.  Measured, both ways, us
// (relabelled / direct): G(300007, d 24) 783 / 293, G(2000003, d 40) 12100 /
// 2340; Chung-Lu n = 300007 mean degree 12 (35 elements an entry) 700 / 673,
// 20 (48) 941 / 1036, 40 (73) 1383 / 1845; n = 1000003 degree 12 (56) 1629 /
// 1463, 20 (76) 2234 / 2440; n = 2000003 degree 6 (49) 2178 / 1809, 12 (74)
// 2724 / 2847; R-MAT scale 14 (61) 358 / 149, 15 (84) 437 / 316, 16 (114) 501
// / 1034, 17 with edge factor 6 (75) 492 / 712.  The line lies at 48 elements
// an entry and 2^25 more, which is what the launches alone are worth.
//
// The largest degree is at most kLongList: a longer forward list may stand at
// any vertex of a graph of more than 65536 of them, so that more than a few of
// a tile's 512 could be, and their chunks would not fit the field above.
// n and nnz: ids and positions of 32 bits in the streams.
inline bool direct_fits(int64_t n, int64_t nnz, int64_t maxdeg, uint64_t deg2) {
  if (n >= INT32_MAX || nnz >= (int64_t(1) << 31) || maxdeg > kLongList) return false;
  return deg2 / 6 <= 48ull * static_cast<uint64_t>(nnz) + (1ull << 25);
}

}  // namespace tc

// Splitting the last tiles of a contraction along k.
//
// A persistent grid of 256 workgroups over T output tiles leaves compute units idle in its last round, or in its only one:
// dHidden of 2300 tokens at H = 2048 has 72 tiles of 2374 k-steps.  The tiles that do not fill a round are therefore cut
// into S parts of the k range; every part leaves its fp32 partial tile in the workspace, and a second kernel adds the
// parts in a fixed order and finishes the tile.  All parts of one k range are consecutive work items, so the workgroups
// of an XCD still stream the same operand panels.
//
// S minimises  rounds(S) * ceil(nk / S)  + what the partials cost (a step of 64 takes 1.5 us per workgroup; a partial tile
// of 256 KiB is written and read once: 0.13 us of the whole chip's memory bandwidth, 0.09 steps).  Many parts are for results of
// a few tiles: dHidden of 64 tokens at H = 2048 is 8 tiles, which 16 parts each leave on half of the compute units
// (233 us with the sum of the parts, now 172).
#pragma once

#include "common.hpp"

namespace atg {

constexpr int kSplitMax = 64;              // parts per tile
constexpr int kSplitSteps = 4;             // k-steps of a part at the least
constexpr int kSplitTiles = 1024;          // partial tiles a launch may leave
constexpr size_t kPartialTileBytes = size_t{256} * 256 * 4;

struct SplitK {
  int full, rest, S, chunk;                // tiles done whole; tiles split; parts per split tile; k-steps per part
};

// bytes of partials that a launch over at most `tiles` tiles of at most `nk` k-steps needs
inline size_t split_k_bytes(int64_t tiles, int64_t nk) {
  const int64_t parts = nk / kSplitSteps < kSplitMax ? nk / kSplitSteps : kSplitMax;
  if (parts < 2) return 0;
  return static_cast<size_t>(tiles * parts < kSplitTiles ? tiles * parts : kSplitTiles) * kPartialTileBytes;
}

#ifdef __HIPCC__
__device__ __forceinline__ SplitK plan_split(int tiles, int nk, int grid) {
  SplitK p;
  p.full = tiles / grid * grid;
  p.rest = tiles - p.full;
  p.S = 1;
  p.chunk = nk;
  if (p.rest == 0) return p;
  int best = nk * 16;                       // in sixteenths of a step
  for (int S = 2; S <= kSplitMax; S += S < 16 ? 1 : 8) {
    if (S * kSplitSteps > nk || p.rest * S > kSplitTiles) continue;
    const int chunk = (nk + S - 1) / S;
    const int cost = (p.rest * S + grid - 1) / grid * chunk * 16 + p.rest * S * 3 / 2 + 80;
    if (cost < best) {
      best = cost;
      p.S = S;
      p.chunk = chunk;
    }
  }
  return p;
}
#endif

}  // namespace atg

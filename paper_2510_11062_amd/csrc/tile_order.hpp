// Order in which a persistent grid walks the tiles of an output.
#pragma once

#include "common.hpp"

namespace atg {

// Persistent-grid tile order.  Workgroups are dealt to the 8 XCDs round-robin by the hardware, so
// workgroup w is given the logical slot (w % 8) * (grid / 8) + w / 8: the 32 workgroups that share
// one XCD's L2 then walk neighbouring tiles.  Tiles are enumerated in bands of `band` A-tiles:
// inside a band the order runs down the band's A-tiles first, then to the next B-tile, so the
// tiles in flight form a compact patch of the output and the operand panels they stream are
// shared through L2 / Infinity Cache.
struct TileOrder {
  int n_a, n_b, band;
  __device__ __forceinline__ int total() const { return n_a * n_b; }
  __device__ __forceinline__ void decode(int t, int* ta, int* tb) const {
    const int per_band = band * n_b;
    const int bi = t / per_band;
    const int first = bi * band;
    const int rows = min(band, n_a - first);
    const int in_band = t - bi * per_band;
    *ta = first + in_band % rows;
    *tb = in_band / rows;
  }
};

__device__ __forceinline__ int logical_workgroup() {
  const int g = gridDim.x, w = blockIdx.x;
  if ((g & 7) != 0) return w;
  return (w & 7) * (g >> 3) + (w >> 3);
}

}  // namespace atg

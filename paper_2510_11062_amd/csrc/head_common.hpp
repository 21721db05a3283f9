// Device helpers shared by the head kernels.
#pragma once

#include "common.hpp"

namespace atg {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

#ifdef __HIPCC__
// four fp32 values at an address that need only be aligned for one of them (the caller's dW): still one 16-byte access
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// list positions of the launch: at most TC of the list's *cnt entries from c0 on
__device__ __forceinline__ int chunk_count(const int32_t* cnt, int c0, int TC) {
  const int n = *cnt - c0;
  return n < 0 ? 0 : (n > TC ? TC : n);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
#endif

// Does a bf16 logits launch of n tokens run on tiles of kNarrowV vocabulary rows instead of 256?  Its partial results are then
// one row of kNarrowStride per kNarrowV vocabulary rows, else one of TC per 256.
constexpr int kNarrowV = 128, kNarrowStride = 256;
#ifdef __HIPCC__
__device__ __forceinline__ bool narrow_launch(int n) { return n <= 192; }
// bf16 weights that a launch of few tokens passes by once and that the Infinity Cache of 256 MB does not hold until the next launch
// reads them: loaded past the caches, by logits and dHidden alike.  Both launches of a step at H = 2048, V = 151936: 8 tokens 328 ->
// 289 us, 64 339 -> 304, 160 349 -> 337 (with the logits' loads alone past the caches dHidden misses what they had left: 138 ->
// 185 us); log-probabilities of 8 tokens at H = 4096 238 -> 218.  205 MB of weights: 38 us by usual loads, 43 past the caches.
__device__ __forceinline__ bool read_once(int n, int V, int H) { return narrow_launch(n) && static_cast<int64_t>(V) * H > (128 << 20); }
#endif
// floats of partial results of one kind that a launch of TC rows over n_vtiles 256-row vocabulary tiles leaves
inline size_t logit_part_floats(int n_vtiles, int64_t TC) {
  const int64_t stride = 256 / kNarrowV * kNarrowStride;
  return static_cast<size_t>(n_vtiles) * static_cast<size_t>(TC > stride ? TC : stride);
}

// persistent grid: one workgroup per compute unit
inline int gemm_grid() {
  const int cus = device_cu_count();
  return cus > 0 ? cus : 256;
}

}  // namespace atg

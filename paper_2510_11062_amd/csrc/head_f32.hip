// fp32 contractions of the LM head (gfx950): log-probabilities, logit gradient, dHidden, dW.
//
// The fp32 matrix instructions run at 1/16 of the bf16 rate, so operand traffic is no concern; what decides is how many
// compute units have a tile.  Tiles are 64 x 64, or 128 x 128 once that fills the chip four times over, one workgroup of
// four wavefronts (2 x 2) each, with several workgroups per compute unit covering each other's latencies.  Contractions
// with few tiles and a long k range (dW of a small head over many tokens) are split along k; the parts are added in a
// fixed order by a second kernel.  Every operand is read where it lies: an operand that is contiguous along k is turned on
// its way into LDS, so no transposed copies exist.
// (256 x 256 tiles and transposed copies before: C1's dW, two workgroups of 40 k-steps, 305 us and dHidden 128 us, now
// 11 and 11 us.)
//
// The log-probabilities keep a fixed order of every sum (k in pairs (0, 4), (1, 5), (2, 6), (3, 7) of each eight; 64
// vocabulary rows in one lane pair; quarters of 256 rows; 256-row tiles in four interleaved chains): losses of the
// sequence-mean kind are sums that nearly cancel, and an fp32 lse of 9 that rounds the other way is felt in them.
#include "head_common.hpp"
#include "head_f32.hpp"

namespace atg {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kF32Threads = 256;
constexpr int kF32StepK = 32;

// LDS panel: 32 k-rows of T values, row stride T + 16 floats, and the values of k-row k rotated by 16 ((k >> 2) & 3) places:
// fragment reads (16 consecutive values of four consecutive k-rows) and both kinds of writes are free of bank conflicts.
template <int T>
struct F32Tile {
  static constexpr int kStride = T + 16, kPanel = kF32StepK * kStride;   // floats
  static constexpr int kItems = T * kF32StepK / 4 / kF32Threads;         // float4 per thread and panel
  static constexpr int kB = T / 32;                                      // 16-wide blocks of a wavefront per side
  static constexpr int kLdsFloats = 4 * kPanel;                          // two panels, two buffers
};

// operand with rows contiguous along k
template <int T>
struct F32Rows {
  const float* p[F32Tile<T>::kItems];
  float4 r[F32Tile<T>::kItems];
  // row_ptr(row): address of k = 0 of tile row `row`
  template <typename F>
  __device__ __forceinline__ void init(F row_ptr) {
#pragma unroll
    for (int q = 0; q < F32Tile<T>::kItems; ++q) p[q] = row_ptr(row(q)) + chunk(q) * 4;
  }
  // 64 lanes cover 16 rows x 16 k
  __device__ __forceinline__ int row(int q) const {
    const int wi = q * (kF32Threads / 64) + (threadIdx.x >> 6);
    return wi % (T / 16) * 16 + (threadIdx.x & 15);
  }
  __device__ __forceinline__ int chunk(int q) const {
    const int wi = q * (kF32Threads / 64) + (threadIdx.x >> 6);
    return wi / (T / 16) * 4 + ((threadIdx.x >> 4) & 3);
  }
  __device__ __forceinline__ void load(int step) {
#pragma unroll
    for (int q = 0; q < F32Tile<T>::kItems; ++q) r[q] = *reinterpret_cast<const float4*>(p[q] + step * kF32StepK);
  }
  __device__ __forceinline__ void store(float* lds) const {
#pragma unroll
    for (int q = 0; q < F32Tile<T>::kItems; ++q) {
      const int c = chunk(q);
      float* at = lds + c * 4 * F32Tile<T>::kStride + ((row(q) + 16 * (c & 3)) & (T - 1));
      at[0] = r[q].x;
      at[F32Tile<T>::kStride] = r[q].y;
      at[2 * F32Tile<T>::kStride] = r[q].z;
      at[3 * F32Tile<T>::kStride] = r[q].w;
    }
  }
};

// k-major operand: rows of k, contiguous along the tile
template <int T, typename RowPtr>
struct F32Columns {
  RowPtr row_ptr;      // row_ptr(k): address of the tile's first column in k-row k
  int k_end, cols;     // k-rows from k_end on and columns from `cols` on (a multiple of 4) read as zero
  float4 r[F32Tile<T>::kItems];
  __device__ __forceinline__ int k_of(int q) const { return (q * kF32Threads + threadIdx.x) / (T / 4); }
  __device__ __forceinline__ int col_of() const { return threadIdx.x % (T / 4) * 4; }
  __device__ __forceinline__ void load(int step) {
#pragma unroll
    for (int q = 0; q < F32Tile<T>::kItems; ++q) {
      const int k = step * kF32StepK + k_of(q);
      r[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k < k_end && col_of() < cols) r[q] = *reinterpret_cast<const float4*>(row_ptr(k) + col_of());
    }
  }
  __device__ __forceinline__ void store(float* lds) const {
#pragma unroll
    for (int q = 0; q < F32Tile<T>::kItems; ++q) {
      const int k = k_of(q);
      *reinterpret_cast<float4*>(lds + k * F32Tile<T>::kStride + ((col_of() + 16 * ((k >> 2) & 3)) & (T - 1))) = r[q];
    }
  }
};

struct F32Coord {
  int lane, wm, wn;
  __device__ __forceinline__ F32Coord() : lane(threadIdx.x & 63), wm(threadIdx.x >> 7), wn((threadIdx.x >> 6) & 1) {}
};

// acc[i][j][r] += sum_k A[a][k] B[b][k] over k-steps s0 .. s1-1, with a = wm T/2 + i 16 + 4 (lane / 16) + r and
// b = wn T/2 + j 16 + lane % 16.  Ends with a workgroup barrier: LDS may be reused.
template <int T, typename LA, typename LB>
__device__ __forceinline__ void gemm_f32(f32x4 (&acc)[F32Tile<T>::kB][F32Tile<T>::kB], LA& la, LB& lb, int s0, int s1,
                                         float* lds) {
  using L = F32Tile<T>;
  constexpr int kB = L::kB;
  const F32Coord co;
#pragma unroll
  for (int i = 0; i < kB; ++i)
#pragma unroll
    for (int j = 0; j < kB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (s0 < s1) {
    la.load(s0);
    lb.load(s0);
    la.store(lds);
    lb.store(lds + L::kPanel);
  }
  __syncthreads();
  for (int s = s0; s < s1; ++s) {
    float* cur = lds + ((s - s0) & 1) * 2 * L::kPanel;
    float* nxt = lds + ((s - s0 + 1) & 1) * 2 * L::kPanel;
    if (s + 1 < s1) {
      la.load(s + 1);
      lb.load(s + 1);
    }
    const float* pa = cur + (co.lane >> 4) * L::kStride + (co.lane & 15);
    const float* pb = pa + L::kPanel;
#pragma unroll
    for (int kk = 0; kk < kF32StepK / 4; ++kk) {
      float a[kB], b[kB];
#pragma unroll
      for (int i = 0; i < kB; ++i) {
        a[i] = pa[kk * 4 * L::kStride + ((co.wm * (T / 2) + i * 16 + 16 * (kk & 3)) & (T - 1))];
        b[i] = pb[kk * 4 * L::kStride + ((co.wn * (T / 2) + i * 16 + 16 * (kk & 3)) & (T - 1))];
      }
#pragma unroll
      for (int i = 0; i < kB; ++i)
#pragma unroll
        for (int j = 0; j < kB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (s + 1 < s1) {
      la.store(nxt);
      lb.store(nxt + L::kPanel);
    }
    __syncthreads();
  }
}

// logits of a T x T tile: A = W rows (v0 ..), B = gathered hidden rows (list positions t0 ..)
template <int T>
__device__ __forceinline__ void logit_tile_f32(f32x4 (&acc)[F32Tile<T>::kB][F32Tile<T>::kB], const float* hidden, const float* W,
                                               const int32_t* idx, int c0, int n, int v0, int t0, int H, int V, float* lds) {
  F32Rows<T> la, lb;
  la.init([&](int row) { return W + static_cast<size_t>(min(v0 + row, V - 1)) * H; });
  lb.init([&](int row) { return hidden + static_cast<size_t>(idx[c0 + min(t0 + row, n - 1)]) * H; });
  gemm_f32<T>(acc, la, lb, 0, H / kF32StepK, lds);
}

// ------------------------------------------------------------------------------------------------
// log-probabilities: tiles of 64 vocabulary rows x 128 tokens, a wavefront per 32 tokens (two 32 x 32 blocks, so that the
// 64 rows of a token are summed inside one lane pair).  part_m / part_s / part_u[v / 64][token]: maximum (log2 domain),
// sum of exponentials and of exponentials times logits.
// ------------------------------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kFwdV = 64, kFwdT = 128;

// LDS panel of T rows: as in F32Tile, but with row stride T + 8 and rotation 16 ((k >> 3) & 1): the two halves of a wavefront
// read k-rows four apart here
template <int T>
struct FwdPanel {
  static constexpr int kStride = T + 8, kFloats = kF32StepK * kStride, kItems = T * kF32StepK / 4 / kF32Threads;
  const float* p[kItems];
  float4 r[kItems];
  __device__ __forceinline__ int row(int q) const {
    const int wi = q * (kF32Threads / 64) + (threadIdx.x >> 6);
    return wi % (T / 16) * 16 + (threadIdx.x & 15);
  }
  __device__ __forceinline__ int chunk(int q) const {
    const int wi = q * (kF32Threads / 64) + (threadIdx.x >> 6);
    return wi / (T / 16) * 4 + ((threadIdx.x >> 4) & 3);
  }
  template <typename F>
  __device__ __forceinline__ void init(F row_ptr) {
#pragma unroll
    for (int q = 0; q < kItems; ++q) p[q] = row_ptr(row(q)) + chunk(q) * 4;
  }
  __device__ __forceinline__ void load(int step) {
#pragma unroll
    for (int q = 0; q < kItems; ++q) r[q] = *reinterpret_cast<const float4*>(p[q] + step * kF32StepK);
  }
  __device__ __forceinline__ void store(float* lds) const {
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      const int c = chunk(q);
      float* at = lds + c * 4 * kStride + ((row(q) + 16 * ((c >> 1) & 1)) & (T - 1));
      at[0] = r[q].x;
      at[kStride] = r[q].y;
      at[2 * kStride] = r[q].z;
      at[3 * kStride] = r[q].w;
    }
  }
  // value of the lane's row (row0 + lane % 32) at k = 8 g + x + 4 (lane / 32)
  static __device__ __forceinline__ float get(const float* lds, int g, int x, int row0, int lane) {
    return lds[(8 * g + x + 4 * (lane >> 5)) * kStride + ((row0 + (lane & 31) + 16 * (g & 1)) & (T - 1))];
  }
};

template <bool ENT>
__global__ __launch_bounds__(kF32Threads) void k_head_fwd(const float* __restrict__ hidden, const float* __restrict__ W,
                                                          const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt,
                                                          int c0, const int32_t* __restrict__ token_id,
                                                          float* __restrict__ part_m, float* __restrict__ part_s,
                                                          float* __restrict__ part_u, float* __restrict__ zy, int H, int V,
                                                          int TC) {
  using PA = FwdPanel<kFwdV>;
  using PB = FwdPanel<kFwdT>;
  constexpr int kBuf = PA::kFloats + PB::kFloats;
  __shared__ __attribute__((aligned(16))) float lds[2 * kBuf];
  const int n = chunk_count(cnt, c0, TC);
  const int v0 = blockIdx.x * kFwdV, t0 = blockIdx.y * kFwdT;
  if (t0 >= n) return;
  const int lane = threadIdx.x & 63, tw = (threadIdx.x >> 6) * 32;      // the wavefront's first token of the tile
  PA la;
  PB lb;
  la.init([&](int row) { return W + static_cast<size_t>(min(v0 + row, V - 1)) * H; });
  lb.init([&](int row) { return hidden + static_cast<size_t>(idx[c0 + min(t0 + row, n - 1)]) * H; });
  f32x16 acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  const int steps = H / kF32StepK;
  la.load(0);
  lb.load(0);
  la.store(lds);
  lb.store(lds + PA::kFloats);
  __syncthreads();
  for (int s = 0; s < steps; ++s) {
    const float* cur = lds + (s & 1) * kBuf;
    float* nxt = lds + ((s + 1) & 1) * kBuf;
    if (s + 1 < steps) {
      la.load(s + 1);
      lb.load(s + 1);
    }
#pragma unroll
    for (int g = 0; g < kF32StepK / 8; ++g)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const float b = PB::get(cur + PA::kFloats, g, x, tw, lane);
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(PA::get(cur, g, x, i * 32, lane), b, acc[i], 0, 0, 0);
      }
    if (s + 1 < steps) {
      la.store(nxt);
      lb.store(nxt + PA::kFloats);
    }
    __syncthreads();
  }
  const int t = t0 + tw + (lane & 31);
  const int vrem = V - v0;                                   // vocabulary rows of the tile that exist
  const int half4 = 4 * (lane >> 5);
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (i * 32 + 8 * (r >> 2) + half4 + (r & 3) < vrem) mx = fmaxf(mx, acc[i][r]);
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  const float m2 = (mx == -INFINITY) ? 0.f : mx * kLog2e;
  float sum = 0.f, usum = 0.f;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (i * 32 + 8 * (r >> 2) + half4 + (r & 3) < vrem) {
        const float e = fast_exp2(fmaf(acc[i][r], kLog2e, -m2));
        sum += e;
        if (ENT) usum = fmaf(e, acc[i][r], usum);
      }
  sum += __shfl_xor(sum, 32, 64);
  if (ENT) usum += __shfl_xor(usum, 32, 64);
  if (t < n) {
    if (half4 == 0) {
      const size_t at = static_cast<size_t>(blockIdx.x) * TC + t;
      part_m[at] = (mx == -INFINITY) ? -INFINITY : m2;
      part_s[at] = sum;
      if (ENT) part_u[at] = usum;
    }
    const int rel = token_id[idx[c0 + t]] - v0;
    if (rel >= 0 && rel < kFwdV && (rel & 4) == half4) {      // the target logit
      float z = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if ((rel & ~4) == i * 32 + 8 * (r >> 2) + (r & 3)) z = acc[i][r];
      zy[t] = z;
    }
  }
}

// 256 threads = 64 tokens x 4 chains over the 256-row tiles
__global__ __launch_bounds__(256) void k_lse_combine_f32(const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt,
                                                         int c0, int TC, int n_part, const float* __restrict__ part_m,
                                                         const float* __restrict__ part_s, const float* __restrict__ part_u,
                                                         const float* __restrict__ zy, float* __restrict__ logp,
                                                         float* __restrict__ lse, float* __restrict__ entropy) {
  __shared__ float sm[4][64], ss[4][64], su[4][64];
  const int n = chunk_count(cnt, c0, TC);
  const int tx = threadIdx.x & 63, py = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + tx;
  if (static_cast<int>(blockIdx.x) * 64 >= n) return;
  float M = -INFINITY, S = 0.f, U = 0.f;
  if (j < n) {
    for (int p = py; p * 4 < n_part; p += 4) {
      float mq[4], sq[4], uq[4];                // the four quarters of the 256-row tile
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool ok = p * 4 + q < n_part;
        const size_t at = static_cast<size_t>(p * 4 + q) * TC + j;
        mq[q] = ok ? part_m[at] : -INFINITY;
        sq[q] = ok ? part_s[at] : 0.f;
        uq[q] = (ok && part_u) ? part_u[at] : 0.f;
      }
      float m = -INFINITY, s = 0.f, u = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) m = fmaxf(m, mq[q]);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (mq[q] != -INFINITY) {
          const float sc = fast_exp2(mq[q] - m);
          s += sq[q] * sc;
          u += uq[q] * sc;
        }
      if (m == -INFINITY) continue;
      const float Mn = fmaxf(M, m);
      const float so = fast_exp2(M - Mn), sn = fast_exp2(m - Mn);
      S = S * so + s * sn;
      U = U * so + u * sn;
      M = Mn;
    }
  }
  sm[py][tx] = M;
  ss[py][tx] = S;
  su[py][tx] = U;
  __syncthreads();
  if (py == 0 && j < n) {
    const float Mt = fmaxf(fmaxf(sm[0][tx], sm[1][tx]), fmaxf(sm[2][tx], sm[3][tx]));
    float St = 0.f, Ut = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (sm[q][tx] != -INFINITY) {
        const float sc = fast_exp2(sm[q][tx] - Mt);
        St += ss[q][tx] * sc;
        Ut += su[q][tx] * sc;
      }
    const float l = (Mt + __log2f(St)) * kLn2;
    const int row = idx[c0 + j];
    logp[row] = zy[j] - l;
    if (lse) lse[row] = l;
    if (entropy) entropy[row] = l - Ut / St;     // H = lse - E_p[z]
  }
}

// dZ[t][v] = g_t ([v = y_t] - exp(z - lse_t)), zero in the padding columns V .. Vp.  With `clear`: the call's first launch also
// clears d_hidden (n16 pieces of 16 bytes), which the next one writes rows of.
template <int T>
__global__ __launch_bounds__(kF32Threads) void k_head_dz(const float* __restrict__ hidden, const float* __restrict__ W,
                                                         const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt,
                                                         int c0, const int32_t* __restrict__ token_id,
                                                         const float* __restrict__ lse, const float* __restrict__ coef,
                                                         float* __restrict__ dZ, int H, int V, int Vp, int TC,
                                                         uint4* __restrict__ clear, int64_t n16) {
  constexpr int kB = F32Tile<T>::kB;
  __shared__ __attribute__((aligned(16))) float lds[F32Tile<T>::kLdsFloats];
  if (clear) {
    const int64_t block = static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * gridDim.y * kF32Threads;
    for (int64_t e = block * kF32Threads + threadIdx.x; e < n16; e += stride) clear[e] = make_uint4(0, 0, 0, 0);
  }
  const int n = chunk_count(cnt, c0, TC);
  const int v0 = blockIdx.x * T, t0 = blockIdx.y * T;
  if (t0 >= n) return;
  f32x4 acc[kB][kB];
  logit_tile_f32<T>(acc, hidden, W, idx, c0, n, v0, t0, H, V, lds);
  const F32Coord co;
  const int vlane = v0 + co.wm * (T / 2) + 4 * (co.lane >> 4);
#pragma unroll
  for (int j = 0; j < kB; ++j) {
    const int t = t0 + co.wn * (T / 2) + j * 16 + (co.lane & 15);
    if (t >= n) continue;
    const int row = idx[c0 + t];
    const int y = token_id[row];
    const float g = coef[row], nl2 = -lse[row] * kLog2e;
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const int v = vlane + i * 16;
      f32x4 d;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        d[r] = -g * fast_exp2(fmaf(acc[i][j][r], kLog2e, nl2));
        if (v + r == y) d[r] += g;
        if (v + r >= V) d[r] = 0.f;
      }
      if (v < Vp) *reinterpret_cast<f32x4*>(dZ + static_cast<size_t>(t) * Vp + v) = d;
    }
  }
}

// k-steps of part `part` of `parts`
__device__ __forceinline__ void part_range(int steps, int part, int parts, int* s0, int* s1) {
  const int chunk = (steps + parts - 1) / parts;
  *s0 = min(part * chunk, steps);
  *s1 = min(*s0 + chunk, steps);
}

// dHidden and dW of a super-chunk, which only have dZ in common: in one launch where all of their workgroups fit the chip
// together, since a small step is a chain of short launches (C1: 10.2 and 9.8 us one after the other, 11.7 together; 2.6 and 3.2
// for the sums of their parts, now 4.0; two heads of 54 rows at H = 480, V = 2746, 664 workgroups: 22.7 and 17.5).  With more of
// them dW's tiles, which are long, would start unevenly as dHidden's end (16000 rows, H = 256, V = 8000: 577 and 725 us one after
// the other, 1701 together).
struct F32Grads {
  const float* dZ;
  const float* W;
  const float* hidden;
  const int32_t* idx;
  const int32_t* cnt;
  float* d_hidden;
  float* dW;
  float *part_h, *part_w;      // partial results of dHidden and of dW
  int c0, H, V, Vp, TC, accumulate, first_chunk;
  int h_tiles, t_tiles, h_parts;      // of dHidden: tiles along H and along the tokens, parts along k
  int w_tiles, w_parts;               // of dW: all tiles, parts along k
  int of_h;                           // tiles of dHidden times parts; 0: the launch has none
};

// dHidden: A = W columns (h), B = dZ rows (tokens), k = vocabulary.  With one part the result goes to d_hidden, else part p
// goes to rows p TC .. of `part_h`.
template <int T>
__device__ __forceinline__ void dh_tile(const F32Grads& a, int block, int n, float* lds) {
  constexpr int kB = F32Tile<T>::kB;
  const int h0 = block % a.h_tiles * T, t0 = block / a.h_tiles % a.t_tiles * T, z = block / (a.h_tiles * a.t_tiles);
  if (t0 >= n) return;
  int s0, s1;
  part_range(a.Vp / kF32StepK, z, a.h_parts, &s0, &s1);
  auto w_row = [&](int k) { return a.W + static_cast<size_t>(k) * a.H + h0; };
  F32Columns<T, decltype(w_row)> la{w_row, a.V, a.H - h0, {}};
  F32Rows<T> lb;
  lb.init([&](int row) { return a.dZ + static_cast<size_t>(min(t0 + row, n - 1)) * a.Vp; });
  f32x4 acc[kB][kB];
  gemm_f32<T>(acc, la, lb, s0, s1, lds);
  const F32Coord co;
  const int hl = h0 + co.wm * (T / 2) + 4 * (co.lane >> 4);
#pragma unroll
  for (int j = 0; j < kB; ++j) {
    const int t = t0 + co.wn * (T / 2) + j * 16 + (co.lane & 15);
    if (t >= n) continue;
    float* out = a.h_parts == 1 ? a.d_hidden + static_cast<size_t>(a.idx[a.c0 + t]) * a.H
                                : a.part_h + (static_cast<size_t>(z) * a.TC + t) * a.H;
#pragma unroll
    for (int i = 0; i < kB; ++i)
      if (hl + i * 16 < a.H) *reinterpret_cast<f32x4*>(out + hl + i * 16) = acc[i][j];
  }
}

// dW[v][h] (+)= sum_t dZ[t][v] hidden[t][h]: A = hidden columns (gathered rows), B = dZ columns, k = tokens of the chunk.
// With one part the result goes to dW, else part p goes to rows p V .. of `part_w`.  The tiles of one vocabulary range are side
// by side.
template <int T>
__device__ __forceinline__ void dw_tile(const F32Grads& a, int block, int n, float* lds) {
  constexpr int kB = F32Tile<T>::kB;
  if (n <= 0 && a.w_parts == 1 && !(a.first_chunk && !a.accumulate)) return;
  const int h_tiles = (a.H + T - 1) / T, tile = block % a.w_tiles, z = block / a.w_tiles;
  const int h0 = tile % h_tiles * T, v0 = tile / h_tiles * T;
  int s0, s1;
  part_range((n + kF32StepK - 1) / kF32StepK, z, a.w_parts, &s0, &s1);
  auto h_row = [&](int k) { return a.hidden + static_cast<size_t>(a.idx[a.c0 + k]) * a.H + h0; };
  auto z_row = [&](int k) { return a.dZ + static_cast<size_t>(k) * a.Vp + v0; };
  F32Columns<T, decltype(h_row)> la{h_row, n, a.H - h0, {}};
  F32Columns<T, decltype(z_row)> lb{z_row, n, a.Vp - v0, {}};
  f32x4 acc[kB][kB];
  gemm_f32<T>(acc, la, lb, s0, s1, lds);
  const F32Coord co;
  const int hl = h0 + co.wm * (T / 2) + 4 * (co.lane >> 4);
#pragma unroll
  for (int j = 0; j < kB; ++j) {
    const int v = v0 + co.wn * (T / 2) + j * 16 + (co.lane & 15);
    if (v >= a.V) continue;
    float* out = a.w_parts == 1 ? a.dW + static_cast<size_t>(v) * a.H : a.part_w + (static_cast<size_t>(z) * a.V + v) * a.H;
    const bool add = a.w_parts == 1 && a.accumulate;
#pragma unroll
    for (int i = 0; i < kB; ++i)
      if (hl + i * 16 < a.H) {
        f32x4_any* o = reinterpret_cast<f32x4_any*>(out + hl + i * 16);
        *o = add ? *o + acc[i][j] : acc[i][j];
      }
  }
}

// the first a.of_h workgroups have a tile of dHidden each, the others one of dW
template <int T>
__global__ __launch_bounds__(kF32Threads) void k_head_grads(F32Grads a) {
  __shared__ __attribute__((aligned(16))) float lds[F32Tile<T>::kLdsFloats];
  const int n = chunk_count(a.cnt, a.c0, a.TC), block = blockIdx.x;
  if (block < a.of_h) dh_tile<T>(a, block, n, lds);
  else dw_tile<T>(a, block - a.of_h, n, lds);
}

// adds the parts up: the first h_blocks workgroups those of dHidden, the others those of dW
__global__ __launch_bounds__(kF32Threads) void k_head_grads_sum(F32Grads a, int h_blocks) {
  const f32x4* src;
  if (static_cast<int>(blockIdx.x) < h_blocks) {
    const int64_t row = a.H / 4, all = chunk_count(a.cnt, a.c0, a.TC) * row, stride = a.TC * row;
    src = reinterpret_cast<const f32x4*>(a.part_h);
    for (int64_t e = blockIdx.x * static_cast<int64_t>(kF32Threads) + threadIdx.x; e < all; e += h_blocks * static_cast<int64_t>(kF32Threads)) {
      f32x4 x = src[e];
      for (int p = 1; p < a.h_parts; ++p) x += src[p * stride + e];
      reinterpret_cast<f32x4*>(a.d_hidden + static_cast<size_t>(a.idx[a.c0 + e / row]) * a.H)[e % row] = x;
    }
    return;
  }
  const int64_t n4 = static_cast<int64_t>(a.V) * a.H / 4;
  const int64_t threads = (gridDim.x - h_blocks) * static_cast<int64_t>(kF32Threads);
  src = reinterpret_cast<const f32x4*>(a.part_w);
  f32x4_any* dst = reinterpret_cast<f32x4_any*>(a.dW);
  for (int64_t e = (blockIdx.x - h_blocks) * static_cast<int64_t>(kF32Threads) + threadIdx.x; e < n4; e += threads) {
    f32x4 x = src[e];
    for (int p = 1; p < a.w_parts; ++p) x += src[p * n4 + e];
    dst[e] = a.accumulate ? dst[e] + x : x;
  }
}

// 128 x 128 tiles need 512 of them for two workgroups per compute unit; below that 64 x 64 tiles spread the work better
int pick_tile(int64_t a, int64_t b) { return ceil_div(a, 128) * ceil_div(b, 128) >= 512 ? 128 : 64; }

// parts along k: enough workgroups for two per compute unit, parts of at least eight steps
int pick_parts(int64_t tiles, int64_t steps) {
  int64_t p = 512 / (tiles < 1 ? 1 : tiles);
  if (p > steps / 8) p = steps / 8;
  if (p > 32) p = 32;
  return p < 1 ? 1 : static_cast<int>(p);
}

int dh_parts(const HeadGeom& g) {
  const int T = pick_tile(g.H, g.TC);
  return pick_parts(ceil_div(g.H, T) * ceil_div(g.TC, T), g.Vp / kF32StepK);
}
int dw_parts(const HeadGeom& g) {
  const int T = pick_tile(g.H, g.V);
  return pick_parts(ceil_div(g.H, T) * ceil_div(g.V, T), g.TC / kF32StepK);
}

unsigned sum_blocks(int64_t n4) {
  const int64_t b = ceil_div(n4, kF32Threads);
  return static_cast<unsigned>(b > 2048 ? 2048 : (b < 1 ? 1 : b));
}

}  // namespace

static size_t part_h_bytes(const HeadGeom& g) {
  const int parts = dh_parts(g);
  return parts > 1 ? round_up(static_cast<size_t>(parts) * g.TC * g.H * 4, 256) : 0;
}
size_t partial_bytes_f32(const HeadGeom& g) {
  const int parts = dw_parts(g);
  return part_h_bytes(g) + (parts > 1 ? static_cast<size_t>(parts) * g.V * g.H * 4 : 0);
}

int launch_fwd_f32(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                   float* part_m, float* part_s, float* part_u, float* zy, hipStream_t s) {
  static_assert(kFwdV == kVocabTileF32, "one partial per tile");
  const dim3 grid(static_cast<unsigned>(g.n_vtiles), static_cast<unsigned>(ceil_div(g.TC, kFwdT)));
  auto k = part_u ? k_head_fwd<true> : k_head_fwd<false>;
  hipLaunchKernelGGL(k, grid, dim3(kF32Threads), 0, s, static_cast<const float*>(hidden), static_cast<const float*>(W), ch.idx,
                     ch.cnt, ch.c0, token_id, part_m, part_s, part_u, zy, g.H, g.V, g.TC);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_lse_combine_f32(const HeadGeom& g, const HeadChunk& ch, const float* part_m, const float* part_s, const float* part_u,
                           const float* zy, float* logp, float* lse, float* entropy, hipStream_t s) {
  hipLaunchKernelGGL(k_lse_combine_f32, dim3(g.TC / 64), dim3(256), 0, s, ch.idx, ch.cnt, ch.c0, g.TC, g.n_vtiles, part_m,
                     part_s, part_u, zy, logp, lse, part_u ? entropy : nullptr);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

template <int T>
static void dz_t(const HeadGeom& g, const HeadChunk& ch, const float* hidden, const float* W, const int32_t* token_id,
                 const float* lse, const float* coef, float* dZ, uint4* clear, int64_t n16, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(ceil_div(g.V, T)), static_cast<unsigned>(ceil_div(g.TC, T)));
  hipLaunchKernelGGL(k_head_dz<T>, grid, dim3(kF32Threads), 0, s, hidden, W, ch.idx, ch.cnt, ch.c0, token_id, lse, coef, dZ,
                     g.H, g.V, g.Vp, g.TC, clear, n16);
}

int launch_dz_f32(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                  const float* lse, const float* coef, void* dZ, void* clear, int64_t n_bytes, hipStream_t s) {
  const float* h = static_cast<const float*>(hidden);
  const float* w = static_cast<const float*>(W);
  float* z = static_cast<float*>(dZ);
  uint4* c = static_cast<uint4*>(clear);
  if (pick_tile(g.V, g.TC) == 128) dz_t<128>(g, ch, h, w, token_id, lse, coef, z, c, n_bytes / 16, s);
  else dz_t<64>(g, ch, h, w, token_id, lse, coef, z, c, n_bytes / 16, s);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_grads_f32(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* W, const void* hidden, void* d_hidden,
                     float* dW, void* part, int accumulate, int first_chunk, hipStream_t s) {
  const int th = pick_tile(g.H, g.TC), tw = pick_tile(g.H, g.V);
  F32Grads a{};
  a.dZ = static_cast<const float*>(dZ);
  a.W = static_cast<const float*>(W);
  a.hidden = static_cast<const float*>(hidden);
  a.idx = ch.idx;
  a.cnt = ch.cnt;
  a.d_hidden = static_cast<float*>(d_hidden);
  a.dW = dW;
  a.part_h = static_cast<float*>(part);
  a.part_w = reinterpret_cast<float*>(static_cast<char*>(part) + part_h_bytes(g));
  a.c0 = ch.c0;
  a.H = g.H;
  a.V = g.V;
  a.Vp = g.Vp;
  a.TC = g.TC;
  a.accumulate = accumulate;
  a.first_chunk = first_chunk;
  a.h_tiles = static_cast<int>(ceil_div(g.H, th));
  a.t_tiles = static_cast<int>(ceil_div(g.TC, th));
  a.h_parts = dh_parts(g);
  const int64_t w_tiles = ceil_div(g.H, tw) * ceil_div(g.V, tw);
  a.w_tiles = static_cast<int>(w_tiles);
  a.w_parts = dw_parts(g);
  const int64_t of_h = static_cast<int64_t>(a.h_tiles) * a.t_tiles * a.h_parts, of_w = w_tiles * a.w_parts;
  a.of_h = static_cast<int>(of_h);
  const auto launch = [&](int cls, int T, int64_t blocks) {
    ProfScope ps(cls, s);
    auto k = T == 128 ? k_head_grads<128> : k_head_grads<64>;
    hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(blocks)), dim3(kF32Threads), 0, s, a);
  };
  // three workgroups of 64 x 64 tiles fit a compute unit
  const bool together = th == 64 && tw == 64 && of_h + of_w <= 3 * device_cu_count();
  if (together) {
    launch(PROF_HEAD_DH, 64, of_h + of_w);
  } else {
    launch(PROF_HEAD_DH, th, of_h);
    ATG_LAUNCH_CHECK();
    a.of_h = 0;
    launch(PROF_HEAD_DW, tw, of_w);
  }
  ATG_LAUNCH_CHECK();
  const unsigned hb = a.h_parts > 1 ? sum_blocks(static_cast<int64_t>(g.TC) * g.H / 4) : 0;
  const unsigned wb = a.w_parts > 1 ? sum_blocks(static_cast<int64_t>(g.V) * g.H / 4) : 0;
  if (hb + wb > 0) {
    ProfScope ps(together || hb > 0 ? PROF_HEAD_DH : PROF_HEAD_DW, s);
    hipLaunchKernelGGL(k_head_grads_sum, dim3(hb + wb), dim3(kF32Threads), 0, s, a, static_cast<int>(hb));
    ATG_LAUNCH_CHECK();
  }
  return AT_GRPO_OK;
}

}  // namespace atg

// Kernels around the head contractions of the AT-GRPO policy loss (gfx950), and the launchers that choose between the bf16
// (head_bf16.hip) and fp32 (head_f32.hip) contractions.
//
// Forward (log pi_theta(y_t) inside the ratio of Eq. 2): logits tiles z[v, t] = <W[v], hidden[t]> are produced in MFMA
// accumulators, reduced to per-(vocabulary tile, token) (max, sum-exp) partials and the target logit, and discarded.  A
// small combine kernel turns the partials into lse and logp.
//
// Backward: logits tiles are recomputed, turned into dZ = g (onehot - softmax) in registers and written once, as
// dZ[token][vocab] in the element type of the inputs; two further contractions give dHidden = dZ W (k = vocab) and
// dW = dZ^T hidden (k = tokens).
#include "head_bf16.hpp"
#include "head_common.hpp"
#include "head_f32.hpp"
#include "head_kernels.hpp"
#include "split_k.hpp"
#include "token_kernels.hpp"

namespace atg {

namespace {

constexpr int kRowPad = 256;      // rows of a super-chunk are padded to the next multiple of this
constexpr int kRowStep = 64;      // rows of a k-step of dW

// ------------------------------------------------------------------------------------------------
// combine: 1024 threads = 32 tokens x 32 slices of the vocabulary tiles.  Bound by latency where tokens are few (the
// chain of dependent loads per thread) and by memory where they are many.  32 slices leave a thread 19 of the 594
// tiles of the full vocabulary, in three batches of eight independent loads; 32 tokens are one 128-byte line per load.
// Full vocabulary: 122 us with 64 tokens x 4 slices and one load at a time, 8 us now for 197 tokens; 138 and 22 us with
// the entropy sums of 8192 rows.  Sums are taken in a fixed order.
// ------------------------------------------------------------------------------------------------
constexpr int kCmbTokens = 32, kCmbSlices = 32, kCmbThreads = kCmbTokens * kCmbSlices, kCmbBatch = 8;

// how many rows of partial results a launch of n tokens left, and how far apart they are
struct PartialRows {
  int count, stride;
  __device__ __forceinline__ PartialRows(int n, int narrow, int V, int n_vtiles, int TC) {
    const bool nl = narrow && narrow_launch(n);
    count = nl ? (V + kNarrowV - 1) / kNarrowV : n_vtiles;
    stride = nl ? kNarrowStride : TC;
  }
};

// sum over a group of 32 lanes, in a fixed order
__device__ __forceinline__ float group32_sum(float x) {
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

__global__ __launch_bounds__(kCmbThreads) void k_lse_combine(const int32_t* __restrict__ idx,
                                                             const int32_t* __restrict__ cnt, int c0, int TC,
                                                             int V, int n_vtiles, int narrow, const float* __restrict__ part_m,
                                                             const float* __restrict__ part_s,
                                                             const float* __restrict__ part_u,
                                                             const float* __restrict__ zy,
                                                             float* __restrict__ logp, float* __restrict__ lse,
                                                             float* __restrict__ entropy,
                                                             const int32_t* __restrict__ gate, int head, CoefArgs ca,
                                                             float* __restrict__ scale) {
  __shared__ float sm[kCmbSlices][kCmbTokens + 1], ss[kCmbSlices][kCmbTokens + 1], su[kCmbSlices][kCmbTokens + 1];
  if (gate && *gate == 0) return;
  const int n = chunk_count(cnt, c0, TC);
  if (static_cast<int>(blockIdx.x) * kCmbTokens >= n) return;
  {
    const int tx = threadIdx.x & (kCmbTokens - 1), py = threadIdx.x / kCmbTokens;
    const int j = blockIdx.x * kCmbTokens + tx;
    const PartialRows parts(n, narrow, V, n_vtiles, TC);
    float M = -INFINITY, S = 0.f, U = 0.f;
    for (int p = py; p < parts.count; p += kCmbSlices * kCmbBatch) {
      float m[kCmbBatch], s[kCmbBatch], u[kCmbBatch];
#pragma unroll
      for (int e = 0; e < kCmbBatch; ++e) {
        const int q = p + e * kCmbSlices;
        const bool ok = q < parts.count && j < n;
        const size_t at = static_cast<size_t>(q) * parts.stride + j;
        m[e] = ok ? part_m[at] : -INFINITY;
        s[e] = ok ? part_s[at] : 0.f;
        u[e] = (ok && part_u) ? part_u[at] : 0.f;
      }
      float Mn = M;
#pragma unroll
      for (int e = 0; e < kCmbBatch; ++e) Mn = fmaxf(Mn, m[e]);
      if (Mn != -INFINITY) {
        const float so = fast_exp2(M - Mn);
        S *= so;
        U *= so;
#pragma unroll
        for (int e = 0; e < kCmbBatch; ++e) {
          const float sn = fast_exp2(m[e] - Mn);
          S = fmaf(s[e], sn, S);
          U = fmaf(u[e], sn, U);
        }
        M = Mn;
      }
    }
    sm[py][tx] = M;
    ss[py][tx] = S;
    su[py][tx] = U;
  }
  __syncthreads();
  const int py = threadIdx.x & (kCmbSlices - 1), tx = threadIdx.x / kCmbSlices;
  const int j = blockIdx.x * kCmbTokens + tx;
  const float m = sm[py][tx];
  float Mt = m;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) Mt = fmaxf(Mt, __shfl_xor(Mt, o, 64));
  const float sc = (m == -INFINITY) ? 0.f : fast_exp2(m - Mt);
  const float St = group32_sum(ss[py][tx] * sc), Ut = group32_sum(su[py][tx] * sc);
  if (py == 0 && j < n) {
    const float l = (Mt + __log2f(St)) * kLn2;
    const int row = idx[c0 + j];
    const float lp = zy[j] - l;
    logp[row] = lp;
    if (lse) lse[row] = l;
    if (entropy) entropy[row] = l - Ut / St;     // H = lse - E_p[z]
    if (scale) scale[j] = -coef_or_zero(ca, head, row, lp);   // E is about to become softmax - onehot: a = -g
  }
}

// ------------------------------------------------------------------------------------------------
// Forward and backward in one pass over the logits (bf16).  With a per-token reference c_t close
// enough to the row's largest logit, e[t][v] = exp(z[t][v] - c_t) neither overflows nor loses the
// terms that matter, and
//   lse_t = c_t + ln S_t,  S_t = sum_v e[t][v],      softmax = e / S_t,
//   dZ[t][v] = g_t (onehot - softmax) = a_t (e[t][v] - S_t [v = y_t]),  a_t = -g_t / S_t.
// The forward tile therefore writes e once (bf16, as dZ would be written), the combine step patches
// the one element per row that carries the onehot term, and the row factor a_t is applied where it is
// cheap: to the accumulators of dHidden and to the gathered hidden rows that dW contracts with.  The
// logits are not recomputed.  c_t is the target logit z[t][y_t] (one dot product per token): the
// exponent then is ln(p_v / p_y), out of range only if the sampled token is ~e^88 times less likely
// than the mode.  Rows for which S_t leaves [1, 2^60) are reported through a gate word, and the
// caller then runs the two-pass kernels for that launch instead.
// ------------------------------------------------------------------------------------------------
constexpr float kMaxRefSum = 1152921504606846976.f;   // 2^60

// c2[j] = log2(e) * <hidden[row_j], W[y_j]>: one wavefront per token of the launch
__global__ __launch_bounds__(256) void k_ref_logit(const bf16_t* __restrict__ hidden, const bf16_t* __restrict__ W,
                                                   const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt,
                                                   int c0, int TC, const int32_t* __restrict__ token_id, int H,
                                                   float* __restrict__ c2) {
  const int n = chunk_count(cnt, c0, TC);
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= n) return;
  const int row = idx[c0 + j];
  const uint4* a = reinterpret_cast<const uint4*>(hidden + static_cast<size_t>(row) * H);
  const uint4* b = reinterpret_cast<const uint4*>(W + static_cast<size_t>(token_id[row]) * H);
  float acc = 0.f;
  for (int c = lane; c < H / 8; c += 64) {
    const uint4 x = a[c], y = b[c];
    const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc = fmaf(__uint_as_float(xs[e] << 16), __uint_as_float(ys[e] << 16), acc);
      acc = fmaf(__uint_as_float(xs[e] & 0xffff0000u), __uint_as_float(ys[e] & 0xffff0000u), acc);
    }
  }
  acc = wave_sum(acc);
  if (lane == 0) c2[j] = acc * kLog2e;
}

// Thread layout of k_lse_combine.  Per token of the launch: S, lse, logp; the backward coefficient g and the row factor
// a = -g / S; the element of E that carries the onehot term is replaced by e_y - S.  A row whose S is not in
// [.., 2^60) (overflow, NaN) or whose reference is not finite raises the gate and gets a = 0.  Without an advantage it needs no
// gradient, and the whole launch is not redone for its log-probability: it joins the list of such rows (`later`, *n_later of them).
__global__ __launch_bounds__(kCmbThreads) void k_fe_combine(const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt,
                                                            int c0, int TC, int V, int n_vtiles, int narrow, int head,
                                                            const float* __restrict__ part_s,
                                                            const float* __restrict__ c2,
                                                            const float* __restrict__ zy,
                                                            const int32_t* __restrict__ token_id, CoefArgs ca,
                                                            float* __restrict__ logp, float* __restrict__ lse,
                                                            float* __restrict__ scale, bf16_t* __restrict__ E, int Vp,
                                                            int32_t* __restrict__ gate, int32_t* __restrict__ later,
                                                            int32_t* __restrict__ n_later) {
  __shared__ float ss[kCmbSlices][kCmbTokens + 1];
  const int n = chunk_count(cnt, c0, TC);
  if (static_cast<int>(blockIdx.x) * kCmbTokens >= n) return;
  {
    const int tx = threadIdx.x & (kCmbTokens - 1), py = threadIdx.x / kCmbTokens;
    const int j = blockIdx.x * kCmbTokens + tx;
    const PartialRows parts(n, narrow, V, n_vtiles, TC);
    float S = 0.f;
    for (int p = py; p < parts.count; p += kCmbSlices * kCmbBatch) {
      float s[kCmbBatch];
#pragma unroll
      for (int e = 0; e < kCmbBatch; ++e) {
        const int q = p + e * kCmbSlices;
        s[e] = (q < parts.count && j < n) ? part_s[static_cast<size_t>(q) * parts.stride + j] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < kCmbBatch; ++e) S += s[e];
    }
    ss[py][tx] = S;
  }
  __syncthreads();
  const int py = threadIdx.x & (kCmbSlices - 1), tx = threadIdx.x / kCmbSlices;
  const int j = blockIdx.x * kCmbTokens + tx;
  const float St = group32_sum(ss[py][tx]);
  if (py == 0 && j < n) {
    const float c2v = c2[j];
    const float l = (c2v + __log2f(St)) * kLn2;
    const int row = idx[c0 + j];
    const float lp = zy[j] - l;
    logp[row] = lp;
    lse[row] = l;
    const bool ok = (St < kMaxRefSum) && (fabsf(c2v) < INFINITY);
    const float g = coef_or_zero(ca, head, row, lp);
    scale[j] = (ok && g != 0.f) ? -g / St : 0.f;
    const float ey = fast_exp2(fmaf(zy[j], kLog2e, -c2v));
    E[static_cast<size_t>(j) * Vp + token_id[row]] = f32_to_bf16(ey - St);
    if (ok) return;
    if (ca.adv[ca.resp_of_tok[row]] == 0.f) later[atomicAdd(n_later, 1)] = row;
    else atomicOr(gate, 1);
  }
}

// Rows on the clipped branch of Eq. (2) (factor scale[j] == 0) carry no gradient.  They are taken out of the
// super-chunk before the two backward contractions: with L = number of rows with a non-zero factor, every
// such row at a position >= L (a "mover", in ascending order) is copied into the i-th position < L whose
// row has factor 0 (a "hole", in ascending order); afterwards rows 0 .. L-1 of E all carry gradient, and
// perm[j] names the row of the super-chunk that now sits at position j (its token, its factor).  Only the
// rows that fill holes move (at most min(L, n - L) of them).  One workgroup of 1024 threads, each owning a
// run of consecutive rows; sums are taken in a fixed order, so the result does not change from run to run.
constexpr int kPlanThreads = 1024;

__global__ __launch_bounds__(kPlanThreads) void k_compact_plan(const int32_t* __restrict__ cnt, int c0, int TC,
                                                               const float* __restrict__ scale,
                                                               int32_t* __restrict__ perm, int32_t* __restrict__ holes,
                                                               int32_t* __restrict__ movers,
                                                               int32_t* __restrict__ live_cnt,
                                                               int32_t* __restrict__ pair_cnt) {
  __shared__ int lds16[kPlanThreads / 64];
  __shared__ int live_below_L;
  const int n = chunk_count(cnt, c0, TC);
  const int per = (TC + kPlanThreads - 1) / kPlanThreads;
  const int j0 = min(static_cast<int>(threadIdx.x) * per, n), j1 = min(j0 + per, n);
  int c = 0;
  for (int j = j0; j < j1; ++j) c += (scale[j] != 0.f);
  int L;
  const int before = block_exclusive_scan<kPlanThreads>(c, lds16, &L);   // live rows in front of this thread's run
  if (threadIdx.x == 0) live_below_L = L;                        // L == n: every row is live
  __syncthreads();
  if (j0 <= L && L < j1) {                                       // the thread that owns position L
    int lb = before;
    for (int j = j0; j < L; ++j) lb += (scale[j] != 0.f);
    live_below_L = lb;
  }
  __syncthreads();
  const int LB = live_below_L;                                   // holes = L - LB = movers
  int lb = before;
  for (int j = j0; j < j1; ++j) {
    const bool on = scale[j] != 0.f;
    if (j < L) {
      if (on) perm[j] = j;
      else holes[j - lb] = j;
    } else if (on) {
      movers[lb - LB] = j;
    }
    lb += on;
  }
  __threadfence();
  __syncthreads();
  lb = before;
  for (int j = j0; j < j1 && j < L; ++j) {
    const bool on = scale[j] != 0.f;
    if (!on) perm[j] = movers[j - lb];
    lb += on;
  }
  if (threadIdx.x == 0) {
    *live_cnt = L;
    *pair_cnt = L - LB;
  }
}

// E[holes[p]][:] = E[movers[p]][:] for p < *pair_cnt; 16 bytes per lane.  A row is shared by kMoveParts workgroups: a few
// rows of the full vocabulary (300 KB each) are spread over the chip.
constexpr int kMoveParts = 8;

__global__ __launch_bounds__(256) void k_move_rows(bf16_t* __restrict__ E, int Vp, const int32_t* __restrict__ holes,
                                                   const int32_t* __restrict__ movers,
                                                   const int32_t* __restrict__ pair_cnt) {
  const int m = *pair_cnt;
  const int chunks = Vp / 8;   // 16-byte pieces per row (Vp is a multiple of 64)
  const int part = blockIdx.x % kMoveParts;
  for (int p = blockIdx.x / kMoveParts; p < m; p += gridDim.x / kMoveParts) {
    const uint4* src = reinterpret_cast<const uint4*>(E + static_cast<size_t>(movers[p]) * Vp);
    uint4* dst = reinterpret_cast<uint4*>(E + static_cast<size_t>(holes[p]) * Vp);
#pragma unroll 4
    for (int c = part * 256 + threadIdx.x; c < chunks; c += kMoveParts * 256) dst[c] = src[c];
  }
}

// ------------------------------------------------------------------------------------------------
// hG[j][:] = hidden[idx[c0 + j]][:] for j < n, zero rows up to the next multiple of 256 (bf16 rows
// of the super-chunk made contiguous so that the token contraction can stream them k-major).  With E: its rows from n up to
// a whole k-step of that contraction are cleared too (what rows that take no part hold need not be finite).
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_gather_rows(const bf16_t* __restrict__ hidden,
                                                     const int32_t* __restrict__ idx,
                                                     const int32_t* __restrict__ cnt, int c0, int TC, int H,
                                                     const float* __restrict__ scale,
                                                     const int32_t* __restrict__ perm,
                                                     const int32_t* __restrict__ live_cnt, bf16_t* __restrict__ hG,
                                                     bf16_t* __restrict__ E, int Vp) {
  // with perm: row j of hG is list position perm[j], for j < *live_cnt
  const int n = perm ? min(*live_cnt, chunk_count(cnt, c0, TC)) : chunk_count(cnt, c0, TC);
  const int n_pad = (n + kRowPad - 1) / kRowPad * kRowPad;
  const int chunks = H / 8;                       // 16-byte pieces per row
  const int rows_per_block = 256 / 32;
  for (int j = blockIdx.x * rows_per_block + (threadIdx.x >> 5); j < n_pad; j += gridDim.x * rows_per_block) {
    const int jp = (j < n && perm) ? perm[j] : j;
    const uint4* src = (j < n) ? reinterpret_cast<const uint4*>(hidden + static_cast<size_t>(idx[c0 + jp]) * H) : nullptr;
    uint4* dst = reinterpret_cast<uint4*>(hG + static_cast<size_t>(j) * H);
    if (src && scale) {
      const float sc = scale[jp];
      for (int c = threadIdx.x & 31; c < chunks; c += 32) {
        const uint4 x = src[c];
        const uint32_t xs[4] = {x.x, x.y, x.z, x.w};
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[e] = pack_bf16x2(__uint_as_float(xs[e] << 16) * sc, __uint_as_float(xs[e] & 0xffff0000u) * sc);
        dst[c] = make_uint4(o[0], o[1], o[2], o[3]);
      }
    } else {
      for (int c = threadIdx.x & 31; c < chunks; c += 32) dst[c] = src ? src[c] : make_uint4(0, 0, 0, 0);
    }
  }
  if (!E) return;
  const int64_t pieces = static_cast<int64_t>((n + kRowStep - 1) / kRowStep * kRowStep - n) * (Vp / 8);
  uint4* rest = reinterpret_cast<uint4*>(E + static_cast<size_t>(n) * Vp);
  for (int64_t c = blockIdx.x * int64_t{256} + threadIdx.x; c < pieces; c += gridDim.x * int64_t{256}) rest[c] = make_uint4(0, 0, 0, 0);
}

}  // namespace

// ================================================================================================
// launchers
// ================================================================================================
int head_vocab_tile(int dtype) { return dtype == AT_GRPO_BF16 ? 256 : kVocabTileF32; }

int launch_head_fwd(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W,
                    const int32_t* token_id, float* part_m, float* part_s, float* part_u, float* zy,
                    hipStream_t s, const int32_t* gate) {
  ProfScope ps(PROF_HEAD_FWD, s);
  if (g.dtype == AT_GRPO_BF16)
    return launch_fwd_bf16(g, ch, hidden, W, token_id, part_m, part_s, part_u, zy, s, gate);
  return launch_fwd_f32(g, ch, hidden, W, token_id, part_m, part_s, part_u, zy, s);
}

int launch_lse_combine(const HeadGeom& g, const HeadChunk& ch, const float* part_m, const float* part_s,
                       const float* part_u, const float* zy, float* logp, float* lse, float* entropy,
                       hipStream_t s, const int32_t* gate, int head, const CoefArgs* ca, float* scale) {
  ProfScope ps(PROF_LSE_COMBINE, s);
  if (g.dtype != AT_GRPO_BF16) return launch_lse_combine_f32(g, ch, part_m, part_s, part_u, zy, logp, lse, entropy, s);
  hipLaunchKernelGGL(k_lse_combine, dim3(g.TC / kCmbTokens), dim3(kCmbThreads), 0, s, ch.idx, ch.cnt, ch.c0, g.TC,
                     g.V, g.n_vtiles, narrow_launches_bf16(g), part_m, part_s, part_u, zy, logp, lse, part_u ? entropy : nullptr, gate,
                     head, ca ? *ca : CoefArgs{}, scale);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

bool needs_transposed_w(const HeadGeom& g, int64_t n_tok) {
  return g.dtype == AT_GRPO_BF16 && transposes_w_bf16(n_tok);
}

int launch_transpose_w(const HeadGeom& g, const void* W, void* Wt, const int32_t* cnt, hipStream_t s) {
  ProfScope ps(PROF_TRANSPOSE, s);
  return Wt ? launch_transpose_w_bf16(g, W, Wt, cnt, s) : AT_GRPO_OK;
}

int launch_gather_hidden(const HeadGeom& g, const HeadChunk& ch, const void* hidden, void* hG,
                         hipStream_t s, const float* scale, const int32_t* perm, const int32_t* live_cnt, void* E) {
  ProfScope ps(PROF_TRANSPOSE, s);
  if (!hG) return AT_GRPO_OK;
  hipLaunchKernelGGL(k_gather_rows, dim3(2048), dim3(256), 0, s, static_cast<const bf16_t*>(hidden), ch.idx,
                     ch.cnt, ch.c0, g.TC, g.H, scale, perm, live_cnt, static_cast<bf16_t*>(hG), static_cast<bf16_t*>(E), g.Vp);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_head_dz(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W,
                   const int32_t* token_id, const float* lse, const float* coef, void* dZ,
                   hipStream_t s, const int32_t* gate, void* clear, int64_t clear_bytes) {
  ProfScope ps(PROF_HEAD_DZ, s);
  if (g.dtype == AT_GRPO_BF16) return launch_dz_bf16(g, ch, hidden, W, token_id, lse, coef, dZ, s, gate);
  return launch_dz_f32(g, ch, hidden, W, token_id, lse, coef, dZ, clear, clear_bytes, s);
}

int launch_ref_logit(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W,
                     const int32_t* token_id, float* c2, hipStream_t s) {
  ProfScope ps(PROF_LSE_COMBINE, s);
  if (g.dtype != AT_GRPO_BF16) return AT_GRPO_EUNSUPPORTED;
  hipLaunchKernelGGL(k_ref_logit, dim3(g.TC / 4), dim3(256), 0, s, static_cast<const bf16_t*>(hidden),
                     static_cast<const bf16_t*>(W), ch.idx, ch.cnt, ch.c0, g.TC, token_id, g.H, c2);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_head_fe(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W,
                   const int32_t* token_id, const float* c2, void* E, float* part_s, float* zy, hipStream_t s) {
  ProfScope ps(PROF_HEAD_FE, s);
  if (g.dtype != AT_GRPO_BF16) return AT_GRPO_EUNSUPPORTED;
  return launch_fe_bf16(g, ch, hidden, W, token_id, c2, E, part_s, zy, s);
}

int launch_fe_combine(const HeadGeom& g, const HeadChunk& ch, int head, const float* part_s, const float* c2,
                      const float* zy, const int32_t* token_id, const CoefArgs& ca, float* logp, float* lse,
                      float* scale, void* E, int32_t* gate, int32_t* later, int32_t* n_later, hipStream_t s) {
  ProfScope ps(PROF_LSE_COMBINE, s);
  hipLaunchKernelGGL(k_fe_combine, dim3(g.TC / kCmbTokens), dim3(kCmbThreads), 0, s, ch.idx, ch.cnt, ch.c0, g.TC, g.V, g.n_vtiles,
                     narrow_launches_bf16(g), head, part_s, c2, zy, token_id, ca, logp, lse, scale, static_cast<bf16_t*>(E), g.Vp, gate,
                     later, n_later);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_compact_rows(const HeadGeom& g, const HeadChunk& ch, const float* scale, void* E, int32_t* perm,
                        int32_t* holes, int32_t* movers, int32_t* live_cnt, int32_t* pair_cnt, hipStream_t s) {
  ProfScope ps(PROF_COEF, s);
  if (g.dtype != AT_GRPO_BF16 || g.TC > 32 * kPlanThreads) return AT_GRPO_EUNSUPPORTED;
  hipLaunchKernelGGL(k_compact_plan, dim3(1), dim3(kPlanThreads), 0, s, ch.cnt, ch.c0, g.TC, scale, perm, holes,
                     movers, live_cnt, pair_cnt);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_move_rows, dim3(2048), dim3(256), 0, s, static_cast<bf16_t*>(E), g.Vp, holes, movers, pair_cnt);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

size_t head_partial_bytes(const HeadGeom& g) {
  if (g.dtype != AT_GRPO_BF16) return partial_bytes_f32(g);
  const int64_t ht = ceil_div(g.H, 256);
  const size_t dh = split_k_bytes(g.TC / 256 * ht, g.Vp / kRowStep), dw = split_k_bytes(g.n_vtiles * ht, g.TC / kRowStep);
  return dh > dw ? dh : dw;
}

int launch_head_dh(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* W, const void* Wt, void* d_hidden,
                   void* part, hipStream_t s, const float* scale, const int32_t* perm, const int32_t* live_cnt) {
  ProfScope ps(PROF_HEAD_DH, s);
  if (g.dtype != AT_GRPO_BF16) return AT_GRPO_EUNSUPPORTED;
  return launch_dh_bf16(g, ch, dZ, W, Wt, d_hidden, part, s, scale, perm, live_cnt);
}

int launch_head_dw(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* hG, float* dW, void* part, int accumulate, int first_chunk, hipStream_t s, const int32_t* live_cnt) {
  ProfScope ps(PROF_HEAD_DW, s);
  if (g.dtype != AT_GRPO_BF16) return AT_GRPO_EUNSUPPORTED;
  return launch_dw_bf16(g, ch, dZ, hG, dW, part, accumulate, first_chunk, s, live_cnt);
}

int launch_head_grads(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* W, const void* hidden, void* d_hidden,
                      float* dW, void* part, int accumulate, int first_chunk, hipStream_t s) {
  if (g.dtype == AT_GRPO_BF16) return AT_GRPO_EUNSUPPORTED;
  return launch_grads_f32(g, ch, dZ, W, hidden, d_hidden, dW, part, accumulate, first_chunk, s);
}

}  // namespace atg

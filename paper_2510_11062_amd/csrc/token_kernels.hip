// Per-token streaming kernels of the AT-GRPO policy loss (gfx950): routing rows to responses and
// heads (the per-model batches B_m of Sec. 3), stable compaction, the clipped surrogate of
// Eq. (2) with a fixed-order reduction, and the backward coefficient d loss / d logp.
#include "token_kernels.hpp"

namespace atg {

namespace {

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t value) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride)
    p[i] = value;
}

__global__ void k_zero16(uint4* __restrict__ p, int64_t n16) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  const uint4 z = make_uint4(0, 0, 0, 0);
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n16; i += stride)
    p[i] = z;
}

__device__ __forceinline__ int head_of_response(int r, int n_heads, int n_agent,
                                                const int32_t* resp_agent,
                                                const int32_t* head_of_agent, int32_t* err) {
  if (n_heads == 1 || resp_agent == nullptr || head_of_agent == nullptr) return 0;
  const int a = resp_agent[r];
  if (a < 0 || a >= n_agent) {
    atomicOr(err, AT_GRPO_DATA_AGENT_RANGE);
    return -1;
  }
  const int h = head_of_agent[a];
  if (h < 0 || h >= n_heads) {
    atomicOr(err, AT_GRPO_DATA_AGENT_RANGE);
    return -1;
  }
  return h;
}

// one wavefront per response
__global__ __launch_bounds__(256) void k_route(TokenLayout L, int32_t* __restrict__ err,
                                               int32_t* __restrict__ resp_of_tok,
                                               int32_t* __restrict__ flag) {
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int n_waves = (gridDim.x * blockDim.x) >> 6;
  for (int r = wave; r < L.n_resp; r += n_waves) {
    const int64_t lo = L.cu_seqlens[r], hi = L.cu_seqlens[r + 1];
    if (lo < 0 || hi < lo || hi > L.n_tok) {
      if (lane == 0) atomicOr(err, AT_GRPO_DATA_SEQLENS);
      continue;
    }
    const int head = head_of_response(r, L.n_heads, L.n_agent, L.resp_agent, L.head_of_agent, err);
    for (int64_t t = lo + lane; t < hi; t += 64) {
      bool on = (head >= 0) && (L.mask == nullptr || L.mask[t] != 0);
      if (on && L.token_id != nullptr) {
        const int y = L.token_id[t];
        if (y < 0 || y >= L.V) {
          atomicOr(err, AT_GRPO_DATA_TOKEN_RANGE);
          on = false;
        }
      }
      resp_of_tok[t] = r;
      flag[t] = on ? head : -1;
    }
  }
}

__global__ __launch_bounds__(256) void k_count(const int32_t* __restrict__ flag, int64_t n_tok,
                                               int n_heads, int64_t n_blk,
                                               int32_t* __restrict__ blk_cnt) {
  __shared__ int lds4[4];
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kTokPerBlock + threadIdx.x * 8;
  int f[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = (t0 + e < n_tok) ? flag[t0 + e] : -1;
  for (int m = 0; m < n_heads; ++m) {
    int c = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) c += (f[e] == m);
    const int tot = block_sum_256_int(c, lds4);
    if (threadIdx.x == 0) blk_cnt[m * n_blk + blockIdx.x] = tot;
  }
}

// single block: exclusive scan of the per-block counts of every head
__global__ __launch_bounds__(256) void k_scan_blocks(const int32_t* __restrict__ blk_cnt, int n_heads,
                                                     int64_t n_blk, int32_t* __restrict__ blk_off,
                                                     int32_t* __restrict__ cnt) {
  __shared__ int lds4[4];
  for (int m = 0; m < n_heads; ++m) {
    int running = 0;
    for (int64_t base = 0; base < n_blk; base += 256) {
      const int64_t b = base + threadIdx.x;
      const int v = (b < n_blk) ? blk_cnt[m * n_blk + b] : 0;
      int tot;
      const int ex = block_exclusive_scan<256>(v, lds4, &tot);
      if (b < n_blk) blk_off[m * n_blk + b] = running + ex;
      running += tot;
    }
    if (threadIdx.x == 0) cnt[m] = running;
  }
  for (int m = n_heads + threadIdx.x; m < kMaxHeads; m += 256) cnt[m] = 0;
}

__global__ __launch_bounds__(256) void k_scatter(const int32_t* __restrict__ flag, int64_t n_tok,
                                                 int n_heads, int64_t n_blk,
                                                 const int32_t* __restrict__ blk_off,
                                                 int32_t* __restrict__ idx) {
  __shared__ int lds4[4];
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kTokPerBlock + threadIdx.x * 8;
  int f[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = (t0 + e < n_tok) ? flag[t0 + e] : -1;
  for (int m = 0; m < n_heads; ++m) {
    int c = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) c += (f[e] == m);
    int tot;
    int pos = blk_off[m * n_blk + blockIdx.x] + block_exclusive_scan<256>(c, lds4, &tot);
    int32_t* out = idx + static_cast<int64_t>(m) * n_tok;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (f[e] == m) out[pos++] = static_cast<int32_t>(t0 + e);
  }
}

// one wavefront per response: participating rows of the response
__global__ __launch_bounds__(256) void k_resp_len(TokenLayout L, const int32_t* __restrict__ flag,
                                                  int32_t* __restrict__ resp_len) {
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int n_waves = (gridDim.x * blockDim.x) >> 6;
  for (int r = wave; r < L.n_resp; r += n_waves) {
    const int64_t lo = L.cu_seqlens[r], hi = L.cu_seqlens[r + 1];
    int c = 0;
    if (!(lo < 0 || hi < lo || hi > L.n_tok))
      for (int64_t t = lo + lane; t < hi; t += 64) c += (flag[t] >= 0);
    c = wave_sum_int(c);
    if (lane == 0) resp_len[r] = c;
  }
}

// single block: responses with at least one participating row, per head
__global__ __launch_bounds__(256) void k_resp_cnt(TokenLayout L, const int32_t* __restrict__ resp_len,
                                                  int32_t* __restrict__ err,
                                                  int32_t* __restrict__ resp_cnt) {
  __shared__ int lds4[4];
  for (int m = 0; m < L.n_heads; ++m) {
    int c = 0;
    for (int r = threadIdx.x; r < L.n_resp; r += 256)
      if (resp_len[r] > 0 &&
          head_of_response(r, L.n_heads, L.n_agent, L.resp_agent, L.head_of_agent, err) == m)
        ++c;
    const int tot = block_sum_256_int(c, lds4);
    if (threadIdx.x == 0) resp_cnt[m] = tot;
  }
}

// Rows lo .. hi of a response, read by a team of LPR lanes (256, 64, 32 or 16, chosen from the mean response length) in aligned
// 4-row vectors.  each(place in the vector, logp, old_logp) is called for every participating row, in ascending order within a lane,
// and returns the row's clip flags, which are stored when clip_mask is given.  One vector of each input per lane and round: with two
// requested ahead, many rows take longer (28 million rows in responses of about 289, 32 lanes: 105 us, 99 with one), and few
// are bound by launches either way.

// vectors of rows of tensors that need not start on a vector's boundary
typedef float f32x4_rows __attribute__((ext_vector_type(4), aligned(4)));
typedef int i32x4_rows __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u8x4_rows __attribute__((aligned(1)));

// Sums and ors over a team's lanes; every lane gets the result.  A team of 256 is a workgroup: lds holds a word per wavefront.
template <int LPR, typename T, typename Op>
__device__ __forceinline__ T team_reduce(T v, T* lds, Op op) {
#pragma unroll
  for (int o = (LPR < 64 ? LPR : 64) / 2; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o, 64));
  if constexpr (LPR > 64) {
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    v = lds[0];
#pragma unroll
    for (int w = 1; w < LPR / 64; ++w) v = op(v, lds[w]);
  }
  return v;
}
struct Plus {
  template <typename T>
  __device__ __forceinline__ T operator()(T a, T b) const { return a + b; }
};
struct Or {
  __device__ __forceinline__ int operator()(int a, int b) const { return a | b; }
};

// A response's head (0xff: none) and the data errors met in its rows share a word: the kernel that adds the responses up
// also collects the errors, so no word has to be cleared beforehand (two launches of 1.4 us fewer for surrogate and monitors).
constexpr int kNoHead = 0xff, kErrShift = 8;

// head of a response, or -1 and an error bit; its loads wait for nothing but each other
__device__ __forceinline__ int head_or_error(const TokenLayout& L, int r, int* bad) {
  if (L.n_heads == 1 || L.resp_agent == nullptr || L.head_of_agent == nullptr) return 0;
  const int a = L.resp_agent[r];
  const bool known = a >= 0 && a < L.n_agent;
  const int h = L.head_of_agent[known ? a : 0];
  const bool ok = known && h >= 0 && h < L.n_heads;
  *bad |= ok ? 0 : AT_GRPO_DATA_AGENT_RANGE;
  return ok ? h : -1;
}

template <int LPR, typename F>
__device__ __forceinline__ void each_row(const TokenLayout& L, const float* __restrict__ logp,
                                         const float* __restrict__ old_logp, int64_t lo, int64_t hi, int head, int lane,
                                         uint8_t* __restrict__ clip_mask, int* bad, F each) {
  auto one = [&](int64_t t) {
    bool on = (head >= 0) && (L.mask == nullptr || L.mask[t] != 0);
    if (on && L.token_id != nullptr) {
      const int y = L.token_id[t];
      if (y < 0 || y >= L.V) {
        *bad |= AT_GRPO_DATA_TOKEN_RANGE;
        on = false;
      }
    }
    const int bits = on ? each(0, logp[t], old_logp[t]) : 0;
    if (clip_mask) clip_mask[t] = static_cast<uint8_t>(bits);
  };
  for (int64_t u = (lo >> 2) + lane; (u << 2) < hi; u += LPR) {
    const int64_t t0 = u << 2;
    if (t0 + 4 <= L.n_tok) {
      // rows of a neighbouring response inside the vector are read but not used
      const f32x4_rows lp = *reinterpret_cast<const f32x4_rows*>(logp + t0);
      const f32x4_rows ol = *reinterpret_cast<const f32x4_rows*>(old_logp + t0);
      uint32_t m4 = 0x01010101u;
      if (L.mask) m4 = *reinterpret_cast<const u8x4_rows*>(L.mask + t0);
      i32x4_rows y4 = 0;
      if (L.token_id) y4 = *reinterpret_cast<const i32x4_rows*>(L.token_id + t0);
      const bool interior = (t0 >= lo) && (t0 + 4 <= hi);
      uint32_t out = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool mine = interior || (t0 + e >= lo && t0 + e < hi);
        bool on = mine && (head >= 0) && (((m4 >> (8 * e)) & 0xffu) != 0);
        if (on && L.token_id != nullptr && (y4[e] < 0 || y4[e] >= L.V)) {
          *bad |= AT_GRPO_DATA_TOKEN_RANGE;
          on = false;
        }
        if (on) out |= static_cast<uint32_t>(each(e, lp[e], ol[e])) << (8 * e);
      }
      if (clip_mask) {
        if (interior) {
          *reinterpret_cast<u8x4_rows*>(clip_mask + t0) = out;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (t0 + e >= lo && t0 + e < hi) clip_mask[t0 + e] = static_cast<uint8_t>(out >> (8 * e));
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t0 + e >= lo && t0 + e < hi) one(t0 + e);
    }
  }
}

struct SurrogateArgs {
  TokenLayout L;
  const float *logp, *old_logp, *adv;
  ClipConst cc;
  int agg;
  uint8_t* clip_mask;
};

// Every row of response r is read once (logp, old_logp, mask, and token_id when given), its clip flags are written, and
// the response's sum of surrogate terms and its count of participating rows are reduced in a fixed order.  Needs no per-row
// routing arrays: the advantage and the head are per-response scalars, requested together with its bounds (6228 responses 12.9 ->
// 12.4 us, 768 8.4 -> 7.0, 24576 short ones 10.2 -> 8.5, the monitors as much).  `word`: head and errors.
// SUMS (1 or 4): sums that a lane keeps, by the rows' place in their vector.
template <int LPR, int SUMS>
__device__ __forceinline__ void surrogate_response(const SurrogateArgs& a, int r, int lane, float* lds_f, int* lds_i, float* total,
                                                   int* rows, int* word) {
  const TokenLayout& L = a.L;
  const int64_t lo = L.cu_seqlens[r], hi = L.cu_seqlens[r + 1];
  const float A = a.adv[r];
  int bad = 0;
  const int head = head_or_error(L, r, &bad);
  *total = 0.f;
  *rows = 0;
  *word = kNoHead | AT_GRPO_DATA_SEQLENS << kErrShift;
  if (lo < 0 || hi < lo || hi > L.n_tok) return;
  float part[SUMS] = {};
  int cnt = 0;
  each_row<LPR>(L, a.logp, a.old_logp, lo, hi, head, lane, a.clip_mask, &bad, [&](int e, float lp, float ol) {
    int bits;
    float ratio;
    part[e % SUMS] += surrogate_term(lp, ol, A, a.cc, &bits, &ratio);
    ++cnt;
    return bits;
  });
  float sum = SUMS == 1 ? part[0] : (part[0] + part[SUMS / 4]) + (part[SUMS / 2] + part[SUMS - 1]);
  // rows owned by no response (before the first / after the last range) carry no flags
  if (a.clip_mask && r == 0)
    for (int64_t t = lane; t < lo; t += LPR) a.clip_mask[t] = 0;
  if (a.clip_mask && r == L.n_resp - 1)
    for (int64_t t = hi + lane; t < L.n_tok; t += LPR) a.clip_mask[t] = 0;
  sum = team_reduce<LPR>(sum, lds_f, Plus());
  cnt = team_reduce<LPR>(cnt, lds_i, Plus());
  bad = team_reduce<LPR>(bad, lds_i, Or());
  *total = (a.agg == AT_GRPO_AGG_SEQ_MEAN_TOKEN_MEAN && cnt > 0) ? sum / static_cast<float>(cnt) : sum;
  *rows = cnt;
  *word = (head & kNoHead) | bad << kErrShift;
}

// What a workgroup of the row kernels adds up per head, in LDS: each team its responses in ascending order, then the teams in turn.
// The final sums read a word per workgroup and head: a word per response, read by one compute unit, took 16 us for 96000 responses and
// 31 for the monitors' seven.
template <int LPR, int NI, int NF>
struct HeadSums {
  static constexpr int kTeams = 256 / LPR;
  int i[kTeams][kMaxHeads][NI];
  float f[kTeams][kMaxHeads][NF];
  int bad;
  __device__ __forceinline__ void clear() {
    for (int k = threadIdx.x; k < kTeams * kMaxHeads * NI; k += 256) (&i[0][0][0])[k] = 0;
    for (int k = threadIdx.x; k < kTeams * kMaxHeads * NF; k += 256) (&f[0][0][0])[k] = 0.f;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
  }
  // sums of head m over the teams
  __device__ __forceinline__ void total(int m, int (&ti)[NI], float (&tf)[NF]) const {
#pragma unroll
    for (int k = 0; k < NI; ++k) ti[k] = i[0][m][k];
#pragma unroll
    for (int k = 0; k < NF; ++k) tf[k] = f[0][m][k];
#pragma unroll
    for (int t = 1; t < kTeams; ++t) {
#pragma unroll
      for (int k = 0; k < NI; ++k) ti[k] += i[t][m][k];
#pragma unroll
      for (int k = 0; k < NF; ++k) tf[k] += f[t][m][k];
    }
  }
};

template <int LPR>
__global__ __launch_bounds__(256) void k_surrogate_resp(SurrogateArgs a, RowParts p) {
  __shared__ float lds_f[4];
  __shared__ int lds_i[4];
  __shared__ HeadSums<LPR, 2, 1> sums;
  const int lane = threadIdx.x & (LPR - 1), mine = threadIdx.x / LPR;
  const int team = (blockIdx.x * blockDim.x + threadIdx.x) / LPR;
  const int n_teams = (gridDim.x * blockDim.x) / LPR;
  sums.clear();
  for (int r = team; r < a.L.n_resp; r += n_teams) {
    float total;
    int rows, word;
    surrogate_response<LPR, 1>(a, r, lane, lds_f, lds_i, &total, &rows, &word);
    if (lane == 0) {
      const int m = word & kNoHead;
      if (m != kNoHead) {
        sums.f[mine][m][0] += total;
        sums.i[mine][m][0] += rows;
        sums.i[mine][m][1] += rows > 0;
      }
      if (word >> kErrShift) atomicOr(&sums.bad, word >> kErrShift);
    }
  }
  __syncthreads();
  const int m = threadIdx.x;
  if (m == 0) p.err[blockIdx.x] = sums.bad;
  if (m >= a.L.n_heads) return;
  int ti[2];
  float tf[1];
  sums.total(m, ti, tf);
  const size_t at = static_cast<size_t>(m) * gridDim.x + blockIdx.x;
  p.ints[at] = make_int4(ti[0], ti[1], 0, 0);
  p.floats[at] = make_float2(tf[0], 0.f);
}

__device__ __forceinline__ float mean_loss(int agg, float total, int rows, int resps) {
  const int denom = agg == AT_GRPO_AGG_SEQ_MEAN_TOKEN_MEAN ? resps : rows;
  return denom > 0 ? -total / static_cast<float>(denom) : 0.f;
}

// Few responses of few rows: all of it by one workgroup, whose wavefront m then adds up head m.  err: null, or the word that gets
// (first) or adds the data errors.
constexpr int kOneThreads = 1024, kOneResp = 1024;

struct LossOut {
  float* loss;
  int32_t *n_valid, *err;
  int first;
};

template <int LPR, int SUMS>
__device__ __forceinline__ void each_response(const SurrogateArgs& a, float* sums, int* rows, int* words) {
  const int lane = threadIdx.x & (LPR - 1);
  for (int r = threadIdx.x / LPR; r < a.L.n_resp; r += kOneThreads / LPR) {
    float total;
    int n, word;
    surrogate_response<LPR, SUMS>(a, r, lane, nullptr, nullptr, &total, &n, &word);
    if (lane == 0) {
      sums[r] = total;
      rows[r] = n;
      words[r] = word;
    }
  }
}

// A lane of 64 takes four times the rows that it takes where a workgroup shares a long response.  Past kOneChain rows a lane four sums
// (LONG: there may be such batches) keep its chains of additions as short: loss of one response of 16384 rows against 64 bits, root mean
// square of 400 such, 6.7e-8 with one sum a lane, 4.1e-8 with four, 4.4e-8 by a workgroup.  Up to there the three are equal (two
// responses of 8192 rows 3.6e-8, 3.3e-8 and 3.7e-8, one of 4096 4.2e-8, 4.0e-8 and 4.5e-8).
constexpr int kOneChain = 128;

template <bool LONG>
__device__ void surrogate_by_one(const SurrogateArgs& a, int lanes, const LossOut& o) {
  __shared__ float sums[kOneResp];
  __shared__ int rows[kOneResp], words[kOneResp];
  static_assert(kOneThreads / 64 >= kMaxHeads, "a wavefront per head");
  if (LONG && lanes == 64 && a.L.n_tok > 64 * kOneChain) each_response<64, 4>(a, sums, rows, words);
  else if (lanes == 64) each_response<64, 1>(a, sums, rows, words);
  else if (lanes == 32) each_response<32, 1>(a, sums, rows, words);
  else each_response<16, 1>(a, sums, rows, words);
  __syncthreads();
  const int m = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (m >= a.L.n_heads) return;
  float total = 0.f;
  int n = 0, resps = 0, bad = 0;
  for (int r = lane; r < a.L.n_resp; r += 64) {
    const bool mine = (words[r] & kNoHead) == m;
    bad |= words[r] >> kErrShift;
    total += mine ? sums[r] : 0.f;
    n += mine ? rows[r] : 0;
    resps += mine && rows[r] > 0 ? 1 : 0;
  }
  total = wave_sum(total);
  n = wave_sum_int(n);
  resps = wave_sum_int(resps);
  bad = team_reduce<64>(bad, static_cast<int*>(nullptr), Or());
  if (lane != 0) return;
  if (m == 0 && o.err) *o.err = o.first ? bad : *o.err | bad;      // kernels in front of this one may have raised bits
  o.loss[m] = mean_loss(a.agg, total, n, resps);
  if (o.n_valid) o.n_valid[m] = n;
}

__global__ __launch_bounds__(kOneThreads) void k_surrogate_one(SurrogateArgs a, int lanes, LossOut o) {
  surrogate_by_one<false>(a, lanes, o);
}

// One 1024-thread block per head: fixed-order sums over the n workgroups of the row kernel.  Returns the head's totals and, to every
// head, the data errors.  The first NI counts and NF sums of a part: the reductions, one after the other, are most of the kernel where
// workgroups are few (240 responses 3.1 us with four and two of them, 2.2 with the loss's two and one).
template <int NI, int NF>
struct FinalSums {
  int i[NI];
  float f[NF];
  int bad;
};

template <int NI, int NF>
__device__ __forceinline__ FinalSums<NI, NF> final_sums(const RowParts& p, int n) {
  __shared__ int is[NI][16], ie[16];
  __shared__ float fs[NF][16];
  const int4* ints = p.ints + static_cast<size_t>(blockIdx.x) * n;
  const float2* floats = p.floats + static_cast<size_t>(blockIdx.x) * n;
  FinalSums<NI, NF> s{};
#pragma unroll 4
  for (int b = threadIdx.x; b < n; b += 1024) {
    const int4 i4 = ints[b];
    const float2 f2 = floats[b];
    const int i[4] = {i4.x, i4.y, i4.z, i4.w};
    const float f[2] = {f2.x, f2.y};
    s.bad |= p.err[b];
#pragma unroll
    for (int k = 0; k < NI; ++k) s.i[k] += i[k];
#pragma unroll
    for (int k = 0; k < NF; ++k) s.f[k] += f[k];
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    s.i[k] = wave_sum_int(s.i[k]);
    if (lane == 0) is[k][wave] = s.i[k];
  }
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    s.f[k] = wave_sum(s.f[k]);
    if (lane == 0) fs[k][wave] = s.f[k];
  }
  if (__builtin_amdgcn_ballot_w64(s.bad != 0) != 0ull) s.bad = team_reduce<64>(s.bad, ie, Or());
  if (lane == 0) ie[wave] = s.bad;
  __syncthreads();
  s = FinalSums<NI, NF>{};
  if (threadIdx.x != 0) return s;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
#pragma unroll
    for (int k = 0; k < NI; ++k) s.i[k] += is[k][w];
#pragma unroll
    for (int k = 0; k < NF; ++k) s.f[k] += fs[k][w];
    s.bad |= ie[w];
  }
  return s;
}

__global__ __launch_bounds__(1024) void k_loss_final(RowParts p, int n, int agg, LossOut o) {
  const FinalSums<2, 1> s = final_sums<2, 1>(p, n);
  if (threadIdx.x != 0) return;
  const int m = blockIdx.x;
  if (m == 0) *o.err = o.first ? s.bad : *o.err | s.bad;      // kernels in front of this one may have raised bits
  o.loss[m] = mean_loss(agg, s.f[0], s.i[0], s.i[1]);
  if (o.n_valid) o.n_valid[m] = s.i[0];
}

// Diagnostics of the clipped-ratio update, LPR lanes per response: participating rows, rows below / above the clip range, rows on
// the clipped branch, and the sums of ratio - 1 - d and of the ratio.
template <int LPR>
__global__ __launch_bounds__(256) void k_diag_resp(TokenLayout L, const float* __restrict__ logp,
                                                   const float* __restrict__ old_logp,
                                                   const float* __restrict__ adv, ClipConst cc, RowParts p) {
  __shared__ float lds_f[4];
  __shared__ int lds_i[4];
  __shared__ HeadSums<LPR, 4, 2> sums;
  const int lane = threadIdx.x & (LPR - 1), mine = threadIdx.x / LPR;
  const int team = (blockIdx.x * blockDim.x + threadIdx.x) / LPR;
  const int n_teams = (gridDim.x * blockDim.x) / LPR;
  sums.clear();
  for (int r = team; r < L.n_resp; r += n_teams) {
    const int64_t lo = L.cu_seqlens[r], hi = L.cu_seqlens[r + 1];
    const float A = adv[r];
    int bad = 0;
    int head = head_or_error(L, r, &bad);
    int n = 0, low = 0, high = 0, zero = 0;
    float kl = 0.f, rs = 0.f;
    if (lo < 0 || hi < lo || hi > L.n_tok) {
      head = -1;
      bad = AT_GRPO_DATA_SEQLENS;
    } else {
      each_row<LPR>(L, logp, old_logp, lo, hi, head, lane, nullptr, &bad, [&](int, float lp, float ol) {
        const float d = lp - ol;
        const bool is_low = d < cc.lo, is_high = d > cc.hi;
        ++n;
        low += is_low;
        high += is_high;
        zero += (is_high && A > 0.f) || (is_low && A < 0.f);
        kl += expm1f(d) - d;
        rs += expf(d);
        return 0;
      });
    }
    n = team_reduce<LPR>(n, lds_i, Plus());
    low = team_reduce<LPR>(low, lds_i, Plus());
    high = team_reduce<LPR>(high, lds_i, Plus());
    zero = team_reduce<LPR>(zero, lds_i, Plus());
    bad = team_reduce<LPR>(bad, lds_i, Or());
    kl = team_reduce<LPR>(kl, lds_f, Plus());
    rs = team_reduce<LPR>(rs, lds_f, Plus());
    if (lane == 0) {
      if (head >= 0) {
        const int add[4] = {n, low, high, zero};
#pragma unroll
        for (int k = 0; k < 4; ++k) sums.i[mine][head][k] += add[k];
        sums.f[mine][head][0] += kl;
        sums.f[mine][head][1] += rs;
      }
      if (bad) atomicOr(&sums.bad, bad);
    }
  }
  __syncthreads();
  const int m = threadIdx.x;
  if (m == 0) p.err[blockIdx.x] = sums.bad;
  if (m >= L.n_heads) return;
  int ti[4];
  float tf[2];
  sums.total(m, ti, tf);
  const size_t at = static_cast<size_t>(m) * gridDim.x + blockIdx.x;
  p.ints[at] = make_int4(ti[0], ti[1], ti[2], ti[3]);
  p.floats[at] = make_float2(tf[0], tf[1]);
}

__global__ __launch_bounds__(1024) void k_diag_final(RowParts p, int n, int32_t* __restrict__ counts, float* __restrict__ stats,
                                                     int32_t* __restrict__ err) {
  const FinalSums<4, 2> s = final_sums<4, 2>(p, n);
  if (threadIdx.x != 0) return;
  const int m = blockIdx.x;
  if (m == 0) *err = s.bad;
  for (int k = 0; k < 4; ++k) counts[m * 4 + k] = s.i[k];
  for (int k = 0; k < 2; ++k) stats[m * 2 + k] = s.i[0] > 0 ? s.f[k] / static_cast<float>(s.i[0]) : 0.f;
}

__global__ __launch_bounds__(256) void k_coef(int64_t n_tok, int32_t* __restrict__ flag, CoefArgs ca,
                                              const float* __restrict__ logp, float* __restrict__ coef) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (t >= n_tok) return;
  const int f = flag[t];
  float g = 0.f;
  if (f >= 0) {
    g = coef_value(ca, f, t, logp[t]);
    if (g == 0.f) {
      g = 0.f;          // also folds -0
      flag[t] = -1;
    }
  }
  coef[t] = g;
}

__global__ __launch_bounds__(256) void k_split_by_advantage(int64_t n_tok, const int32_t* __restrict__ flag,
                                                            const int32_t* __restrict__ resp_of_tok,
                                                            const float* __restrict__ adv,
                                                            int32_t* __restrict__ flag_b,
                                                            int32_t* __restrict__ flag_f) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (t >= n_tok) return;
  const int f = flag[t];
  bool grad = false;
  if (f >= 0) grad = adv[resp_of_tok[t]] != 0.f;   // NaN counts as non-zero and propagates
  flag_b[t] = (f >= 0 && grad) ? f : -1;
  flag_f[t] = (f >= 0 && !grad) ? f : -1;
}

__global__ __launch_bounds__(256) void k_zero_nonparticipating(int64_t n_tok,
                                                               const int32_t* __restrict__ flag,
                                                               float* __restrict__ logp,
                                                               float* __restrict__ lse) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (t >= n_tok) return;
  if (flag[t] < 0) {
    logp[t] = 0.f;
    if (lse) lse[t] = 0.f;
  }
}

// ------------------------------------------------------------------------------------------------
// Small batches: everything between the layout and the head contractions in one launch of one workgroup.  The general path
// takes 8 to 16 launches of 2 to 5 us for it (fills, routing, counts, scan, scatter, ...), which is most of a small call;
// here the rows' heads stay in LDS from one phase to the next.  Bound by latency: 5 to 9 us for up to 2300 rows.  Step of C1
// (fp32) 126 -> 72 us, log-probabilities of one response 388 -> 372, micro-batch of 2300 rows 3670 -> 3528.
// ------------------------------------------------------------------------------------------------
enum PrepMode {
  PREP_LOGPROB,    // lists of the participating rows; logp / lse / entropy = 0 elsewhere
  PREP_BACKWARD,   // weights and coefficients; lists of the rows whose coefficient is not zero
  PREP_STEP        // weights; lists of the rows with and without an advantage; logp / lse = 0 elsewhere; gates cleared
};

constexpr int kPsThreads = 1024, kPsRows = 32768, kPsPer = 8, kPsTile = kPsThreads * kPsPer;
constexpr int kPsBatch = 4;            // rows of a response that a lane requests before it uses the first
constexpr int kPsNoAdv = 0x40;         // mark of a participating row: its head, with this bit where the advantage is zero
// Up to so many rows without an advantage join the list of a head's other rows, behind them (their factor is zero, so they
// are taken out again in front of the backward contractions); up to kPsMergeMost where as many have one.  A list of their own costs
// a pass over the head's weights and tiles that do not fill the chip; on the common list they cost the write of their exponentials,
// 7 % of their contraction, and few rows with an advantage in front of them a whole tile more of it.  Steps on two lists and on one,
// us, rows with + without an advantage (H = 2048 at V = 32000, H = 2048 and H = 4096 at V = 151936):
//   64 + 64     246, 759, 1352 and 223, 648, 1143     64 + 512    272, 895, 1623 and 283, 870, 1562
//   64 + 1024   311, 1109, 2049 and 343, 1129, 2036   200 + 1536  395, 1514, 2859 and 421, 1508, 2788
//   700 + 768   484, 1823, 3472 and 468, 1801, 3416   700 + 1536  542, 2171, 4128 and 563, 2173, 4113
//   2000 + 1024 847, 3787, 7225 and 863, 3751, 7132   2000 + 2000 941, 4128, 7918 and 954, 4190, 7987
constexpr int kPsMerge = 512, kPsMergeMost = 1024;
static_assert(kMaxHeads <= kPsNoAdv, "head and flag share a byte");

struct PrepArgs {
  TokenLayout L;
  TokenScratch S;
  int lanes;                           // per response
  float *logp, *lse, *entropy;         // zeroed where a row takes no part (LOGPROB, STEP); logp is read by BACKWARD
  CoefArgs ca;                         // BACKWARD
  float* coef;
  const float* adv;                    // STEP
  int32_t *cnt_b, *idx_b, *cnt_f, *idx_f;
  int32_t* gates;
  int n_gates;
};

template <int MODE>
__device__ __forceinline__ void prep_small(const PrepArgs& a) {
  __shared__ __attribute__((aligned(16))) int8_t mark[kPsRows];
  __shared__ int part[2][kPsThreads / 64];
  __shared__ int rows_of_head[kMaxHeads], resps_of_head[kMaxHeads];
  __shared__ uint32_t listed[kMaxHeads];      // rows with an advantage, and in the upper half those without
  const TokenLayout& L = a.L;
  const int tid = threadIdx.x, n = static_cast<int>(L.n_tok);

  if (tid == 0) *a.S.err = 0;
  if (tid < kMaxHeads) rows_of_head[tid] = resps_of_head[tid] = listed[tid] = 0;
  for (int i = tid * 16; i < n; i += kPsThreads * 16) *reinterpret_cast<int4*>(mark + i) = make_int4(-1, -1, -1, -1);
  if (MODE != PREP_LOGPROB)
    for (int t = tid; t < n; t += kPsThreads) a.S.resp_of_tok[t] = -1;
  if (MODE == PREP_STEP)
    for (int i = tid; i < a.n_gates; i += kPsThreads) a.gates[i] = 0;
  __syncthreads();

  // rows of every response: a.lanes lanes each
  const int lanes = a.lanes, lane = tid & (lanes - 1);
  for (int r = tid / lanes; r < L.n_resp; r += kPsThreads / lanes) {
    const int64_t lo = L.cu_seqlens[r], hi = L.cu_seqlens[r + 1];
    if (lo < 0 || hi < lo || hi > L.n_tok) {
      if (lane == 0) {
        atomicOr(a.S.err, AT_GRPO_DATA_SEQLENS);
        a.S.resp_len[r] = 0;
      }
      continue;
    }
    const int head = head_of_response(r, L.n_heads, L.n_agent, L.resp_agent, L.head_of_agent, a.S.err);
    int mine = head;
    if (MODE == PREP_STEP && head >= 0 && a.adv[r] == 0.f) mine |= kPsNoAdv;   // NaN counts as non-zero and propagates
    int c = 0;
    const int end = static_cast<int>(hi);
    for (int t0 = static_cast<int>(lo) + lane; t0 < end; t0 += lanes * kPsBatch) {
      int y[kPsBatch], m[kPsBatch];
#pragma unroll
      for (int b = 0; b < kPsBatch; ++b) {
        const int t = t0 + b * lanes;
        y[b] = 0;
        m[b] = 1;
        if (t < end) {
          if (L.token_id) y[b] = L.token_id[t];
          if (L.mask) m[b] = L.mask[t];
        }
      }
#pragma unroll
      for (int b = 0; b < kPsBatch; ++b) {
        const int t = t0 + b * lanes;
        if (t >= end) break;
        bool on = head >= 0 && m[b] != 0;
        if (on && (y[b] < 0 || y[b] >= L.V)) {
          atomicOr(a.S.err, AT_GRPO_DATA_TOKEN_RANGE);
          on = false;
        }
        if (MODE != PREP_LOGPROB) a.S.resp_of_tok[t] = r;
        mark[t] = static_cast<int8_t>(on ? mine : -1);
        c += on;
      }
    }
    for (int o = lanes >> 1; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if (MODE != PREP_LOGPROB && lane == 0) {
      a.S.resp_len[r] = c;
      if (c > 0) {
        atomicAdd(&rows_of_head[head], c);
        atomicAdd(&resps_of_head[head], 1);
      }
    }
  }
  __syncthreads();

  if (MODE != PREP_LOGPROB && tid < kMaxHeads) {
    a.S.cnt[tid] = rows_of_head[tid];
    a.S.resp_cnt[tid] = resps_of_head[tid];
  }
  if (MODE == PREP_BACKWARD) {
    __syncthreads();
#pragma unroll 4
    for (int t = tid; t < n; t += kPsThreads) {
      const int f = mark[t];
      float g = 0.f;
      if (f >= 0) {
        g = coef_value(a.ca, f, t, a.logp[t]);
        if (g == 0.f) {
          g = 0.f;          // also folds -0
          mark[t] = -1;
        }
      }
      a.coef[t] = g;
    }
    __syncthreads();
  } else {
    for (int t = tid; t < n; t += kPsThreads) {
      if (mark[t] < 0) {
        a.logp[t] = 0.f;
        if (a.lse) a.lse[t] = 0.f;
        if (a.entropy) a.entropy[t] = 0.f;
      }
    }
  }

  // eight consecutive rows per thread; what lies behind the last row is not marked
  const int wlane = tid & 63, wave = tid >> 6;
  static_assert(kPsRows % 16 == 0 && kPsRows < 65536, "whole pieces of marks; both counts of a head fit a word");
  auto load_marks = [&](int t0, int8_t(&f)[kPsPer]) {
    uint2 w = make_uint2(0xffffffffu, 0xffffffffu);
    if (t0 < n) w = *reinterpret_cast<const uint2*>(mark + t0);
#pragma unroll
    for (int e = 0; e < kPsPer; ++e) f[e] = static_cast<int8_t>((e < 4 ? w.x : w.y) >> (8 * (e & 3)));
  };
  // with an advantage: in the lower half, without one: in the upper
  auto count_marks = [&](const int8_t(&f)[kPsPer], int m) {
    uint32_t v = 0;
#pragma unroll
    for (int e = 0; e < kPsPer; ++e) v += f[e] == m ? 1 : (f[e] == (m | kPsNoAdv) ? 0x10000 : 0);
    return v;
  };

  // How long a head's two lists become, counted on the marks that they are made from.  (The responses' counts above say something
  // else where bounds of responses overlap: a row then counts for each of them.  That is a data error, which must not decide where
  // anything is stored.)
  if (MODE == PREP_STEP) {
    for (int m = 0; m < L.n_heads; ++m) {
      uint32_t v = 0;
      for (int t0 = tid * kPsPer; t0 < n; t0 += kPsTile) {
        int8_t f[kPsPer];
        load_marks(t0, f);
        v += count_marks(f, m);
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      if (wlane == 0 && v != 0) atomicAdd(&listed[m], v);
    }
    __syncthreads();
  }

  // lists, ascending; the counts of a tile's rows on both lists travel in one word (at most 8192 each)
  int buf = 0;
  for (int m = 0; m < kMaxHeads; ++m) {
    int run_b = 0, run_f = 0;
    bool merge = false;
    if (m < L.n_heads) {
      int32_t* out_b = a.idx_b + static_cast<size_t>(m) * n;
      int32_t* out_f = MODE == PREP_STEP ? a.idx_f + static_cast<size_t>(m) * n : nullptr;
      const int rows_f = MODE == PREP_STEP ? listed[m] >> 16 : 0, rows_b = MODE == PREP_STEP ? listed[m] & 0xffff : 0;
      merge = rows_b > 0 && rows_f > 0 && rows_f <= max(kPsMerge, min(rows_b, kPsMergeMost));
      if (merge) out_f = out_b + rows_b;
      for (int base = 0; base < n; base += kPsTile) {
        const int t0 = base + tid * kPsPer;
        int8_t f[kPsPer];
        load_marks(t0, f);
        const int v = count_marks(f, m);
        int incl = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int up = __shfl_up(incl, o, 64);
          if (wlane >= o) incl += up;
        }
        if (wlane == 63) part[buf][wave] = incl;
        __syncthreads();          // the other buffer's readers passed the barrier in front of this one's
        int before = incl - v, total = 0;
#pragma unroll
        for (int k = 0; k < kPsThreads / 64; ++k) {
          const int x = part[buf][k];
          before += k < wave ? x : 0;
          total += x;
        }
        buf ^= 1;
        int pos_b = run_b + (before & 0xffff), pos_f = run_f + (before >> 16);
#pragma unroll
        for (int e = 0; e < kPsPer; ++e) {
          if (f[e] == m) out_b[pos_b++] = t0 + e;
          else if (MODE == PREP_STEP && f[e] == (m | kPsNoAdv)) out_f[pos_f++] = t0 + e;
        }
        run_b += total & 0xffff;
        run_f += total >> 16;
      }
    }
    if (tid == 0) {
      a.cnt_b[m] = merge ? run_b + run_f : run_b;
      if (MODE == PREP_STEP) a.cnt_f[m] = merge ? 0 : run_f;
    }
  }
}

template <int MODE>
__global__ __launch_bounds__(kPsThreads) void k_prep_small(PrepArgs a) {
  prep_small<MODE>(a);
}

// Both read the log-probabilities and neither needs the other's results: the backward's preparation by one workgroup, the surrogate
// and the loss by another (which raises no error bits: the first one meets the same data).
__global__ __launch_bounds__(kPsThreads) void k_prep_backward_loss(PrepArgs a, SurrogateArgs sa, LossOut o) {
  if (blockIdx.x == 0) prep_small<PREP_BACKWARD>(a);
  else surrogate_by_one<true>(sa, a.lanes, o);
}

unsigned grid_for(int64_t n, int per_block, int64_t cap = 1 << 20) {
  int64_t g = ceil_div(n, per_block);
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return static_cast<unsigned>(g);
}

// lanes of the one-workgroup preparation that share a response: a batch of four rows per lane covers the mean
int team_lanes_small(const TokenLayout& L) {
  const int64_t mean_rows = L.n_tok / (L.n_resp > 0 ? L.n_resp : 1);
  return mean_rows > 128 ? 64 : mean_rows > 64 ? 32 : 16;
}

// A workgroup per response where there are at most two per compute unit, so that nothing but the longest response counts: 240
// responses of 290 rows in the mean 10.1 -> 5.4 us; 1024 of 288 take 6.0 with a wavefront and 5.8 with a workgroup each, 6144 of 289
// 13.0 and 19.0.
constexpr int kWideTeams = 512;

// One workgroup walks the responses 1024 / lanes at a time, 3 us each time.  Stage of one and of two launches, us on the stream with the
// events around it: 50 responses of 20 rows 8.3 and 10.2, 100 10.0 and 11.5, 200 14.7 and 10.3; 40 of 87 9.8 and 10.4, 80 of 89 13.2 and
// 11.2; 13 of 262 9.3 and 10.9, 27 of 256 12.1 and 10.5.
bool surrogate_is_small(const TokenLayout& L) {
  static_assert(4096 <= 64 * kOneChain, "surrogate_by_one<false>");
  return L.n_tok <= 4096 && L.n_tok <= static_cast<int64_t>(L.n_resp) * 1024 &&
         static_cast<int64_t>(L.n_resp) * team_lanes_small(L) <= 2 * kOneThreads;
}

// Lanes that share a response in the row kernels, by the mean number of rows and by how many responses there are.  The chip
// holds 8192 of these wavefronts.  While the responses are few rounds of it, the call ends with its longest response, which may
// be many times the mean: more lanes (C5, 6228 responses of 289 rows in the mean and up to 4096: surrogate 19 us with 64 lanes,
// 26 with 32; 24 000 such responses 36 and 42).  Beyond that the rate counts, and lanes without rows cost: 28 million rows in
// responses of about 170 take 126 us with 64 lanes, 109 with 32; of about 100, 152 with 32 and 135 with 16; of about 600, 88
// with 64 and 90 with 32.
int team_lanes(const TokenLayout& L) {
  const int64_t mean_rows = L.n_tok / (L.n_resp > 0 ? L.n_resp : 1);
  if (mean_rows >= 160 && L.n_resp <= kWideTeams) return 256;
  if (mean_rows >= 512) return 64;
  if (mean_rows >= 160) return L.n_resp <= 32768 ? 64 : 32;
  return mean_rows >= 60 && L.n_resp <= 8192 ? 32 : 16;
}

// Workgroups of the row kernels, and parts for the final sums: 96000 responses, both passes and both sums with at most 16384 235 us, with
// 4096 216, with 2048 242.
constexpr int kRowBlocks = 4096;
int row_blocks(const TokenLayout& L) { return static_cast<int>(grid_for(L.n_resp, 256 / team_lanes(L), kRowBlocks)); }

}  // namespace

int launch_fill_i32(int32_t* p, int64_t n, int32_t value, hipStream_t s) {
  if (n <= 0) return AT_GRPO_OK;
  hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, p, n, value);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_fill_bytes16(void* p, int64_t n_bytes, hipStream_t s) {
  if (n_bytes <= 0) return AT_GRPO_OK;
  ProfScope ps(PROF_FILL, s);
  hipLaunchKernelGGL(k_zero16, dim3(grid_for(n_bytes / 16, 256, 8192)), dim3(256), 0, s,
                     static_cast<uint4*>(p), n_bytes / 16);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_route(const TokenLayout& L, const TokenScratch& S, hipStream_t s) {
  ProfScope ps(PROF_PREP, s);
  ATG_TRY(launch_fill_i32(S.err, 1, 0, s));
  ATG_TRY(launch_fill_i32(S.resp_of_tok, L.n_tok, -1, s));
  ATG_TRY(launch_fill_i32(S.flag, L.n_tok, -1, s));
  hipLaunchKernelGGL(k_route, dim3(grid_for(L.n_resp, 4, 4096)), dim3(256), 0, s, L, S.err,
                     S.resp_of_tok, S.flag);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_compact(const TokenLayout& L, const TokenScratch& S, bool with_idx, hipStream_t s) {
  ProfScope ps(PROF_PREP, s);
  const unsigned nb = static_cast<unsigned>(S.n_blk);
  hipLaunchKernelGGL(k_count, dim3(nb), dim3(256), 0, s, S.flag, L.n_tok, L.n_heads, S.n_blk, S.blk_cnt);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(256), 0, s, S.blk_cnt, L.n_heads, S.n_blk, S.blk_off,
                     S.cnt);
  ATG_LAUNCH_CHECK();
  if (with_idx) {
    hipLaunchKernelGGL(k_scatter, dim3(nb), dim3(256), 0, s, S.flag, L.n_tok, L.n_heads, S.n_blk,
                       S.blk_off, S.idx);
    ATG_LAUNCH_CHECK();
  }
  return AT_GRPO_OK;
}

int launch_resp_len(const TokenLayout& L, const TokenScratch& S, hipStream_t s) {
  ProfScope ps(PROF_PREP, s);
  hipLaunchKernelGGL(k_resp_len, dim3(grid_for(L.n_resp, 4, 4096)), dim3(256), 0, s, L, S.flag,
                     S.resp_len);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_resp_cnt, dim3(1), dim3(256), 0, s, L, S.resp_len, S.err, S.resp_cnt);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_surrogate(const TokenLayout& L, const TokenScratch& S, const float* logp, const float* old_logp,
                     const float* adv, float eps_low, float eps_high, int agg, float* loss,
                     uint8_t* clip_mask, int32_t* n_valid, bool first, hipStream_t s) {
  ProfScope ps(PROF_SURROGATE, s);
  const SurrogateArgs a{L, logp, old_logp, adv, make_clip(eps_low, eps_high), agg, clip_mask};
  if (surrogate_is_small(L)) {
    hipLaunchKernelGGL(k_surrogate_one, dim3(1), dim3(kOneThreads), 0, s, a, team_lanes_small(L), LossOut{loss, n_valid, S.err, first ? 1 : 0});
    ATG_LAUNCH_CHECK();
    return AT_GRPO_OK;
  }
  const int lanes = team_lanes(L), blocks = row_blocks(L);
  auto k = lanes == 256 ? k_surrogate_resp<256> : lanes == 64 ? k_surrogate_resp<64> : lanes == 32 ? k_surrogate_resp<32> : k_surrogate_resp<16>;
  hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, s, a, S.parts);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_loss_final, dim3(L.n_heads), dim3(1024), 0, s, S.parts, blocks, agg, LossOut{loss, n_valid, S.err, first ? 1 : 0});
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

// Room for a workgroup per response, whatever row_blocks makes of the batch: it falls where responses get more or shorter, and scratch
// memory that was asked for once, for the largest batch, has to serve the smaller ones.
RowParts take_row_parts(int32_t n_resp, int n_heads, WsAlloc& ws) {
  const size_t blocks = static_cast<size_t>(n_resp < kRowBlocks ? n_resp : kRowBlocks);
  RowParts p;
  p.ints = ws.take<int4>(blocks * static_cast<size_t>(n_heads));
  p.floats = ws.take<float2>(blocks * static_cast<size_t>(n_heads));
  p.err = ws.take<int32_t>(blocks);
  return p;
}

// By the number of responses alone, so for all heads that there may be; no less than the seven words per response that this scratch
// memory has always had room for
size_t diagnostics_workspace(int32_t n_resp) {
  WsAlloc ws(nullptr), words(nullptr);
  ws.take<int32_t>(64);
  take_row_parts(n_resp, kMaxHeads, ws);
  words.take<int32_t>(64);
  for (int k = 0; k < 7; ++k) words.take<int32_t>(static_cast<size_t>(n_resp));
  return ws.bytes() > words.bytes() ? ws.bytes() : words.bytes();
}

int launch_diagnostics(const TokenLayout& L, const float* logp, const float* old_logp, const float* adv,
                       float eps_low, float eps_high, int32_t* counts, float* stats, void* workspace,
                       hipStream_t s) {
  ProfScope ps(PROF_SURROGATE, s);
  WsAlloc ws(workspace);
  int32_t* err = ws.take<int32_t>(64);
  const RowParts p = take_row_parts(L.n_resp, L.n_heads, ws);
  const ClipConst cc = make_clip(eps_low, eps_high);
  const int lanes = team_lanes(L), blocks = row_blocks(L);
  auto k = lanes == 256 ? k_diag_resp<256> : lanes == 64 ? k_diag_resp<64> : lanes == 32 ? k_diag_resp<32> : k_diag_resp<16>;
  hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, s, L, logp, old_logp, adv, cc, p);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_diag_final, dim3(L.n_heads), dim3(1024), 0, s, p, blocks, counts, stats, err);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

CoefArgs make_coef_args(const TokenScratch& S, const float* old_logp, const float* adv, float eps_low,
                        float eps_high, int agg, const float* grad_loss) {
  CoefArgs ca;
  ca.resp_of_tok = S.resp_of_tok;
  ca.resp_len = S.resp_len;
  ca.cnt = S.cnt;
  ca.resp_cnt = S.resp_cnt;
  ca.old_logp = old_logp;
  ca.adv = adv;
  ca.grad_loss = grad_loss;
  ca.cc = make_clip(eps_low, eps_high);
  ca.agg = agg;
  return ca;
}

int launch_coef(const TokenLayout& L, const TokenScratch& S, const float* logp, const float* old_logp,
                const float* adv, float eps_low, float eps_high, int agg, const float* grad_loss,
                float* coef, hipStream_t s) {
  ProfScope ps(PROF_COEF, s);
  const CoefArgs ca = make_coef_args(S, old_logp, adv, eps_low, eps_high, agg, grad_loss);
  hipLaunchKernelGGL(k_coef, dim3(static_cast<unsigned>(S.n_blk256)), dim3(256), 0, s, L.n_tok, S.flag, ca, logp,
                     coef);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_split_by_advantage(const TokenLayout& L, const TokenScratch& S, const float* adv, int32_t* flag_b,
                              int32_t* flag_f, hipStream_t s) {
  ProfScope ps(PROF_PREP, s);
  hipLaunchKernelGGL(k_split_by_advantage, dim3(static_cast<unsigned>(S.n_blk256)), dim3(256), 0, s, L.n_tok,
                     S.flag, S.resp_of_tok, adv, flag_b, flag_f);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_zero_nonparticipating(const TokenLayout& L, const TokenScratch& S, float* logp, float* lse,
                                 hipStream_t s) {
  ProfScope ps(PROF_PREP, s);
  hipLaunchKernelGGL(k_zero_nonparticipating, dim3(static_cast<unsigned>(S.n_blk256)), dim3(256), 0, s,
                     L.n_tok, S.flag, logp, lse);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

// One workgroup walks the responses kPsThreads / lanes at a time, about 1 us each time, where the general path takes that
// many launches; beyond 16 times the two meet.
bool prep_is_small(const TokenLayout& L) {
  return L.n_tok <= kPsRows && static_cast<int64_t>(L.n_resp) * team_lanes_small(L) <= 16 * kPsThreads;
}

// Beside the backward's preparation, which takes 1 us each time, the loss's workgroup is the longer one from some rounds on, and the two
// launches saved are 8 us.  Long responses are walked in turn by both workgroups, so they need no rule: steps of 1 response of 1024, 4096
// and 16384 rows (H = 32, V = 200) take 43, 64 and 164 us, and 49, 71 and 170 with the loss in front; 2 of 8192 118 and 129.
bool prep_takes_loss(const TokenLayout& L) {
  return prep_is_small(L) && L.n_tok <= 16384 && static_cast<int64_t>(L.n_resp) * team_lanes_small(L) <= 4 * kOneThreads;
}

static PrepArgs prep_args(const TokenLayout& L, const TokenScratch& S) {
  PrepArgs a{};
  a.L = L;
  a.S = S;
  a.lanes = team_lanes_small(L);
  a.cnt_b = S.cnt;
  a.idx_b = S.idx;
  return a;
}

int launch_prep_logprob(const TokenLayout& L, const TokenScratch& S, float* logp, float* lse, float* entropy, hipStream_t s) {
  ProfScope ps(PROF_PREP, s);
  PrepArgs a = prep_args(L, S);
  a.logp = logp;
  a.lse = lse;
  a.entropy = entropy;
  hipLaunchKernelGGL(k_prep_small<PREP_LOGPROB>, dim3(1), dim3(kPsThreads), 0, s, a);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_prep_backward(const TokenLayout& L, const TokenScratch& S, const float* logp, const CoefArgs& ca, float* coef,
                         hipStream_t s) {
  ProfScope ps(PROF_PREP, s);
  PrepArgs a = prep_args(L, S);
  a.logp = const_cast<float*>(logp);   // only read in this mode
  a.ca = ca;
  a.coef = coef;
  hipLaunchKernelGGL(k_prep_small<PREP_BACKWARD>, dim3(1), dim3(kPsThreads), 0, s, a);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_prep_backward_loss(const TokenLayout& L, const TokenScratch& S, const float* logp, const CoefArgs& ca, float* coef,
                              float* loss, uint8_t* clip_mask, int32_t* n_valid, hipStream_t s) {
  static_assert(16 * kPsThreads / 16 <= kOneResp && kPsThreads == kOneThreads, "what prep_is_small lets through");
  ProfScope ps(PROF_PREP, s);
  PrepArgs a = prep_args(L, S);
  a.logp = const_cast<float*>(logp);   // only read in this mode
  a.ca = ca;
  a.coef = coef;
  const SurrogateArgs sa{L, logp, ca.old_logp, ca.adv, ca.cc, ca.agg, clip_mask};
  hipLaunchKernelGGL(k_prep_backward_loss, dim3(2), dim3(kPsThreads), 0, s, a, sa, LossOut{loss, n_valid, nullptr, 0});
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_prep_step(const TokenLayout& L, const TokenScratch& S, const TokenScratch& SB, const TokenScratch& SF,
                     const float* adv, float* logp, float* lse, int32_t* gates, int n_gates, hipStream_t s) {
  ProfScope ps(PROF_PREP, s);
  PrepArgs a = prep_args(L, S);
  a.logp = logp;
  a.lse = lse;
  a.adv = adv;
  a.cnt_b = SB.cnt;
  a.idx_b = SB.idx;
  a.cnt_f = SF.cnt;
  a.idx_f = SF.idx;
  a.gates = gates;
  a.n_gates = n_gates;
  hipLaunchKernelGGL(k_prep_small<PREP_STEP>, dim3(1), dim3(kPsThreads), 0, s, a);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

}  // namespace atg

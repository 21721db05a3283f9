// bf16 contractions of the LM head (gfx950): log-probabilities, exponentials, logit gradient, dHidden, dW.
//
// All of them are persistent grids of one workgroup per compute unit over 256 x 256 output tiles (gemm_bf16.hpp), which the
// logits' last round cuts along the tokens; the logits of up to 192 tokens are streams over tiles of 128 vocabulary rows and 64,
// 128 or 192 tokens (gemm_stream.hpp).  The operand whose index is contiguous in the output is operand A: a lane then holds four
// consecutive outputs per accumulator block, and results leave the registers as 16-byte stores without passing through LDS.
#include <limits.h>

#include <type_traits>

#include "gemm_bf16.hpp"
#include "gemm_stream.hpp"
#include "head_bf16.hpp"
#include "head_common.hpp"
#include "split_k.hpp"
#include "tile_order.hpp"

namespace atg {

namespace {

// Short k loops (k = H) with a heavy epilogue: two wavefronts per SIMD, 128 vocabulary rows x 64 tokens each.  A token's
// 128 logits of a wavefront are one 256-byte run of the stored exponentials.
using GLogit = Grid16<2, 4>;
// Fewer tokens (balanced_tokens)
using GLogit224 = Grid16<4, 2, kTile16, 224>;
using GLogit192 = Grid16<4, 2, kTile16, 192>;
using GLogit160 = Grid16<4, 2, kTile16, 160>;
// At most a half and a quarter of a tile's tokens, for the last round of the persistent grid
using GLogit128 = Grid16<4, 2, kTile16, 128>;
using GLogit64 = Grid16<8, 1, kTile16, 64>;
// Launches of few tokens (narrow_launch), on tiles of 128 vocabulary rows: twice as many tiles share out better where there
// are few, and more steps fit the ring
template <int T>
using GNarrow = typename std::conditional<(T <= 128), Grid16<4, 2, kNarrowV, T>, Grid16<2, 4, kNarrowV, T>>::type;
constexpr int narrow_depth(int T) { return T <= 64 ? 6 : T <= 128 ? 4 : 3; }    // steps in the ring
constexpr int kFoldBytes = 4 * 256 * 3 * 4;     // [wavefronts along the vocabulary][tokens] x 3 behind the ring
using GDh = Grid16<2, 2>;   // long k loop (k = V): one wavefront per SIMD
using GDw = Grid16<4, 2>;

// Row permutation of operand A inside groups of 32: with tile row `row` holding output index a_index(row), the eight
// values of a lane's accumulator blocks 2 p and 2 p + 1 are eight consecutive outputs, and the four lane groups of a
// wavefront cover 32 consecutive ones (64 bytes of bf16 per store instruction and row).
__device__ __forceinline__ int a_index(int row) {
  return (row & ~31) | (((row >> 2) & 3) << 3) | (((row >> 4) & 1) << 2) | (row & 3);
}
// first of the eight outputs of the block pair p (relative to the wavefront's first row)
__device__ __forceinline__ int pair_first(int p, int lane) { return p * 32 + (lane >> 4) * 8; }

template <int IB>
__device__ __forceinline__ float pick(const floatx4 (&col)[IB], int i_sel, int r_sel) {
  float v = 0.f;
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) v = (i_sel == i && r_sel == r) ? col[i][r] : v;
  return v;
}

__device__ __forceinline__ float across_groups_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}
__device__ __forceinline__ float across_groups_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}

// A launch of logits tiles: A = W rows (v0 ..), B = gathered hidden rows (list positions t0 ..)
struct LogitIn {
  const bf16_t* hidden;
  const bf16_t* W;
  const int32_t* idx;      // of the launch's first list position
  const int32_t* token_id;
  int n, H, V;             // n: list positions of the launch, or of the part of it that a cut tile covers
  int pad_end;             // positions from n up to here are the launch's padding (from here on: not this tile's)
};

// What the epilogue needs to know of a lane's tokens, one per accumulator block column: fetched behind the k loop's last
// requests (list first, then what it points to), so it costs no registers in the loop and no wait
// (columns past the end of the list repeat its last row)
template <typename G>
struct TokenCols {
  int row[G::kJB], y[G::kJB];
  __device__ __forceinline__ void rows(const LogitIn& in, int t0, const Coord16<G>& co) {
#pragma unroll
    for (int j = 0; j < G::kJB; ++j) row[j] = in.idx[min(t0 + co.b_row(j), in.n - 1)];
  }
  __device__ __forceinline__ void targets(const LogitIn& in) {
#pragma unroll
    for (int j = 0; j < G::kJB; ++j) y[j] = in.token_id[row[j]];
  }
  __device__ __forceinline__ void settle() {
#pragma unroll
    for (int j = 0; j < G::kJB; ++j) asm volatile("" : "+v"(y[j]));
  }
};

// The tiles it = first, first + gridDim.x, ... < end of one shape; place(it, &v0, &t0) says where a tile lies.  The next
// tile's first two steps are requested in front of a tile's epilogue, whose LDS is the slot that they leave free, and what the epilogue
// has to look up is fetched beside the last two steps.  That takes 2 us of waiting from a tile, of 14 to 100 us, and gives less,
// since the clock falls as the matrix cores are busier: log-probabilities of 3000 rows at H = 1024, V = 32000 184 -> 178 us, a step
// of 8000 rows at H = 1024, V = 50000 2170 -> 2140, entropy of 4700 rows at H = 2048 4343 -> 4317; C2's step by less than its
// runs differ (393.6 and 391.2 ms).
// Off: offsets inside an operand panel
template <typename G, bool PERMUTED, typename Off, typename Place, typename Epilogue>
__device__ __forceinline__ void logit_tiles(const LogitIn& in, int first, int end, Place place, char* smem, Epilogue epi) {
  if (first >= end) return;
  const int nk = in.H / kStepK;
  const Off row_bytes = static_cast<Off>(in.H) * 2;
  RowPanel<G::kLoadsA, Off> pa;
  GatherPanel<G::kLoadsB> pb;
  int rows[G::kLoadsB];
  auto fetch_rows = [&](int t0) {
    const Coord16<G> co;
#pragma unroll
    for (int q = 0; q < G::kLoadsB; ++q) rows[q] = in.idx[min(t0 + pb.row(q, co.wave, co.lane), in.n - 1)];
  };
  auto aim = [&](int v0) {
    const Coord16<G> co;
    pa.init(reinterpret_cast<const char*>(in.W) + static_cast<size_t>(v0) * row_bytes, co.wave, co.lane, [&](int row) {
      return static_cast<Off>(min(PERMUTED ? a_index(row) : row, in.V - 1 - v0)) * row_bytes;
    });
    pb.init(co.wave, co.lane,
            [&](int q) { return reinterpret_cast<const char*>(in.hidden) + static_cast<size_t>(rows[q]) * row_bytes; });
  };
  floatx4 acc[G::kIB][G::kJB];
  auto g = make_gemm16<G>(acc, pa, pb, smem, Coord16<G>());
  int v0, t0;
  place(first, &v0, &t0);
  fetch_rows(t0);
  aim(v0);
  g.begin(nk);
  for (int it = first;;) {
    const int next = it + static_cast<int>(gridDim.x);
    int vn = 0, tn = 0;
    if (next < end) place(next, &vn, &tn);
    TokenCols<G> cols;
    typename Epilogue::template Fetched<G> more;
    g.run(nk, [&](int stage) {
      const Coord16<G> co;
      if (stage == 0) {
        if (next < end) fetch_rows(tn);
        cols.rows(in, t0, co);
      } else {
        cols.targets(in);
        epi.fetch(more, cols, in, t0, co);
      }
    });
    // here since the last step's barrier; a wait for them behind the requests would wait for those as well
    cols.settle();
    more.settle();
    if (next < end) {
      aim(vn);
      g.begin(nk);
    }
    epi.template finish<G>(acc, cols, more, v0, t0, in, smem + kRingFree);
    if (next >= end) break;
    it = next;
    v0 = vn;
    t0 = tn;
  }
}

// A launch of at most T tokens, as one stream of k-steps over this workgroup's vocabulary tiles.  Bound by memory: the weights
// pass once, for little arithmetic.  V = 151936, 256 x 256 tiles before: 8 tokens at H = 4096 396 -> 217 us (5.7 TB/s), 100
// tokens at H = 2048 199 -> 135 us (of these 240 -> 217 and 144 -> 135 by loads past the caches).  With 200 tokens the arithmetic is as long as the loads, and the
// tiles of 256 x 256 are as fast (390 us at H = 4096, 405 as a stream).
// ONCE: see read_once
template <int T, bool PERMUTED, bool ONCE, typename Epilogue>
__device__ __forceinline__ void logit_stream(const LogitIn& in, char* smem, Epilogue epi) {
  using G = GNarrow<T>;
  using PA = RowPanel<G::kLoadsA, uint32_t, ONCE>;
  using PB = GatherPanel<G::kLoadsB>;
  using S = Stream16<G, PA, PB, narrow_depth(T)>;
  static_assert(G::kThreads == GLogit::kThreads && S::kBytes + kFoldBytes <= kRingBytes, "fits the launch");
  const int nk = in.H / kStepK, grid = gridDim.x, first = logical_workgroup();
  if (first * kNarrowV >= in.V) return;
  const uint32_t row_bytes = static_cast<uint32_t>(in.H) * 2;
  PA pa;
  PB pb;
  TokenCols<G> cols;
  typename Epilogue::template Fetched<G> more;
  {
    const Coord16<G> co;
    cols.rows(in, 0, co);
    cols.targets(in);
    epi.fetch(more, cols, in, 0, co);
    // they have to be here before the stream starts: a wait for them behind it would wait for the stream as well
    cols.settle();
    more.settle();
    pb.init(co.wave, co.lane, [&](int q) {
      const int t = min(pb.row(q, co.wave, co.lane), in.n - 1);
      return reinterpret_cast<const char*>(in.hidden) + static_cast<size_t>(in.idx[t]) * row_bytes;
    });
  }
  auto aim = [&](int v0) {
    const Coord16<G> co;
    pa.init(reinterpret_cast<const char*>(in.W) + static_cast<size_t>(v0) * row_bytes, co.wave, co.lane, [&](int row) {
      return static_cast<uint32_t>(min(PERMUTED ? a_index(row) : row, in.V - 1 - v0)) * row_bytes;
    });
  };
  int v_req = first * kNarrowV, k_req = 0;      // of the step requested last
  auto next = [&] {                             // (behind the last tile: that one again)
    if (++k_req < nk) return;
    k_req = 0;
    if (v_req + grid * kNarrowV < in.V) v_req += grid * kNarrowV;
    aim(v_req);
#pragma unroll
    for (int q = 0; q < G::kLoadsB; ++q) pb.p[q] -= row_bytes;
  };
  floatx4 acc[G::kIB][G::kJB];
  S st(acc, pa, pb, smem, Coord16<G>());
  aim(v_req);
  st.begin(next);
  for (int v0 = first * kNarrowV; v0 < in.V; v0 += grid * kNarrowV) {
    st.clear();
    for (int k = 0; k < nk; ++k) st.step(next);
    epi.template finish<G>(acc, cols, more, v0, 0, in, smem + kRingBytes - kFoldBytes);
  }
  st.finish();
}

template <bool PERMUTED, bool ONCE, typename Epilogue>
__device__ __forceinline__ void logit_narrow(const LogitIn& in, char* smem, Epilogue epi) {
  if (in.n <= 64) logit_stream<64, PERMUTED, ONCE>(in, smem, epi);
  else if (in.n <= 128) logit_stream<128, PERMUTED, ONCE>(in, smem, epi);
  else logit_stream<192, PERMUTED, ONCE>(in, smem, epi);
}

// Tokens of a tile: as many tiles as 256 tokens each take, of equal size, in steps of 32 (from 1569 tokens on that is always 256).
// A last tile of 256 that is mostly padding costs its whole arithmetic.  Log-probabilities at V = 151936, all tiles of 256 before: 300
// tokens 272 -> 235 us at H = 2048 and 515 -> 432 at H = 4096, 600 379 -> 362, 1100 606 -> 572, entropy of 300 290 -> 250; 2048
// tokens and more are as they were.
__device__ __forceinline__ int balanced_tokens(int n) {
  const int tiles = (n + kTile16 - 1) / kTile16;
  return ((n + tiles - 1) / tiles + 31) / 32 * 32;
}

// All tiles of a launch, of G.  Those that do not fill a round of the grid are cut into halves or quarters of their tokens if there
// are workgroups for all of them: 594 tiles (the full vocabulary, up to 256 tokens) are two rounds and a half instead of three
// (197 tokens at H = 4096 372 -> 346 us with the call's other kernels, 400 at H = 2048, 4.6 rounds, 345 -> 328; with equal tiles and the
// ring of gemm_bf16.hpp 331 and 268).
template <typename G, bool PERMUTED, typename Off, typename Epilogue>
__device__ __forceinline__ void logit_rounds(const LogitIn& in, int n_vtiles, char* smem, Epilogue epi) {
  constexpr bool kCut = sizeof(Off) == 4;       // (not for vocabularies beyond 8.3 million)
  constexpr int T = G::kTileB;
  const TileOrder ord{n_vtiles, (in.n + T - 1) / T, 8};
  const int me = logical_workgroup(), grid = gridDim.x, rest = ord.total() % grid;
  const int cuts = !kCut || rest * 2 > grid ? 1 : rest * 4 > grid ? 2 : 4;
  const int whole = cuts == 1 ? ord.total() : ord.total() - rest;
  logit_tiles<G, PERMUTED, Off>(
      in, me, whole,
      [&](int it, int* v0, int* t0) {
        int vt, tt;
        ord.decode(it, &vt, &tt);
        *v0 = vt * kTile16;
        *t0 = tt * T;
      },
      smem, epi);
  if constexpr (kCut) {
    if (cuts == 1 || me >= rest * cuts) return;
    int vt, tt;
    ord.decode(whole + me / cuts, &vt, &tt);
    const int t = tt * T + me % cuts * (T / cuts);
    if (t >= in.n) return;
    LogitIn part = in;
    part.pad_end = t + T / cuts;
    part.n = min(in.n, part.pad_end);
    auto place = [&](int, int* v0, int* t0) {
      *v0 = vt * kTile16;
      *t0 = t;
    };
    lds_barrier();      // the whole tiles' epilogues are done with LDS
    if (cuts == 2) logit_tiles<GLogit128, PERMUTED, Off>(part, 0, 1, place, smem, epi);
    else logit_tiles<GLogit64, PERMUTED, Off>(part, 0, 1, place, smem, epi);
  }
}

template <bool PERMUTED, typename Off, typename Epilogue>
__device__ __forceinline__ void logit_launch(const LogitIn& in, int n_vtiles, char* smem, Epilogue epi) {
  constexpr bool kCut = sizeof(Off) == 4;       // (not for vocabularies beyond 8.3 million)
  if constexpr (kCut) {
    if (narrow_launch(in.n)) {
      if (read_once(in.n, in.V, in.H)) logit_narrow<PERMUTED, true>(in, smem, epi);
      else logit_narrow<PERMUTED, false>(in, smem, epi);
      return;
    }
  }
  if constexpr (kCut) {
    switch (balanced_tokens(in.n)) {
      case 160: return logit_rounds<GLogit160, PERMUTED, Off>(in, n_vtiles, smem, epi);
      case 192: return logit_rounds<GLogit192, PERMUTED, Off>(in, n_vtiles, smem, epi);
      case 224: return logit_rounds<GLogit224, PERMUTED, Off>(in, n_vtiles, smem, epi);
      default: return logit_rounds<GLogit, PERMUTED, Off>(in, n_vtiles, smem, epi);
    }
  } else {
    logit_rounds<GLogit, PERMUTED, Off>(in, n_vtiles, smem, epi);
  }
}

// Where the partial results of vocabulary tile v0 and token t of a launch are kept (see narrow_launch)
template <typename G>
__device__ __forceinline__ size_t part_index(int v0, int t, int TC) {
  return static_cast<size_t>(v0 / G::kTileA) * (G::kTileA == kNarrowV ? kNarrowStride : TC) + t;
}

// ------------------------------------------------------------------------------------------------
// forward: per (vocabulary tile, token) maximum and sum of exponentials, and the target logit
// ------------------------------------------------------------------------------------------------
// ENT: also part_u, the partial sums of 2^(z log2e - m) * z that the entropy monitor needs (H = lse - E_p[z])
template <bool ENT>
struct FwdEpilogue {
  float *part_m, *part_s, *part_u, *zy;
  int TC;

  template <typename G>
  struct Fetched {
    __device__ __forceinline__ void settle() {}
  };
  template <typename G>
  __device__ __forceinline__ void fetch(Fetched<G>&, const TokenCols<G>&, const LogitIn&, int, const Coord16<G>&) const {}

  template <typename G>
  __device__ __forceinline__ void finish(const floatx4 (&acc)[G::kIB][G::kJB], const TokenCols<G>& cols, const Fetched<G>&,
                                         int v0, int t0, const LogitIn& in, char* lds) const {
    constexpr int T = G::kTileB;
    float* red_m = reinterpret_cast<float*>(lds);          // [kWavesA][T]
    float* red_s = red_m + G::kWavesA * T;
    float* red_u = red_s + G::kWavesA * T;
    const Coord16<G> co;
    const int n = in.n;
    const int vbase = v0 + co.wm * G::kRowsA;
    const int vrem = in.V - vbase;                    // vocabulary rows of this wavefront that exist (may be <= 0)
    const int vlane = 4 * (co.lane >> 4);             // first row of this lane inside a block
#pragma unroll
    for (int j = 0; j < G::kJB; ++j) {
      const int tcol = t0 + co.b_row(j);
      const int rel = cols.y[j] - vbase;
      floatx4 col[G::kIB];
#pragma unroll
      for (int i = 0; i < G::kIB; ++i) col[i] = acc[i][j];
      if (vrem < G::kRowsA) {
#pragma unroll
        for (int i = 0; i < G::kIB; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) col[i][r] = (i * 16 + vlane + r < vrem) ? col[i][r] : -INFINITY;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < G::kIB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, col[i][r]);
      mx = across_groups_max(mx);
      const float m2 = (mx == -INFINITY) ? 0.f : mx * kLog2e;
      float sum = 0.f, usum = 0.f;
#pragma unroll
      for (int i = 0; i < G::kIB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float e = fast_exp2(fmaf(col[i][r], kLog2e, -m2));
          sum += e;
          if (ENT) usum += e > 0.f ? e * col[i][r] : 0.f;
        }
      sum = across_groups_sum(sum);
      if (ENT) usum = across_groups_sum(usum);
      if (co.lane < 16) {
        red_m[co.wm * T + co.b_row(j)] = (mx == -INFINITY) ? -INFINITY : m2;
        red_s[co.wm * T + co.b_row(j)] = sum;
        if (ENT) red_u[co.wm * T + co.b_row(j)] = usum;
      }
      // target logit: held by exactly one lane of one wavefront of one tile
      const bool hit = tcol < n && rel >= 0 && rel < G::kRowsA && ((rel >> 2) & 3) == (co.lane >> 4);
      if (__builtin_amdgcn_ballot_w64(hit) != 0ull) {
        const float zt = pick<G::kIB>(col, rel >> 4, rel & 3);
        if (hit) zy[tcol] = zt;
      }
    }
    // fold the wavefronts' shares of the tile: one (max, sum) per token and vocabulary tile.  The buffers are free again
    // behind the next step's barrier.
    lds_barrier();
    const int tl = co.wave * 64 + co.lane;
    if (tl < T && t0 + tl < n) {
      float M = -INFINITY;
#pragma unroll
      for (int q = 0; q < G::kWavesA; ++q) M = fmaxf(M, red_m[q * T + tl]);
      float S = 0.f, U = 0.f;
#pragma unroll
      for (int q = 0; q < G::kWavesA; ++q) {
        const float mq = red_m[q * T + tl];
        if (mq != -INFINITY) {
          const float sc = fast_exp2(mq - M);
          S += red_s[q * T + tl] * sc;
          if (ENT) U += red_u[q * T + tl] * sc;
        }
      }
      const size_t at = part_index<G>(v0, t0 + tl, TC);
      part_m[at] = M;
      part_s[at] = S;
      if (ENT) part_u[at] = U;
    }
  }
};

template <bool ENT, typename Off>
__global__ __launch_bounds__(GLogit::kThreads) void k_head_fwd(
    const bf16_t* __restrict__ hidden, const bf16_t* __restrict__ W, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ cnt, int c0, const int32_t* __restrict__ token_id, float* __restrict__ part_m,
    float* __restrict__ part_s, float* __restrict__ part_u, float* __restrict__ zy, int H, int V, int TC, int n_vtiles,
    const int32_t* __restrict__ gate) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  if (gate && *gate == 0) return;
  const int n = chunk_count(cnt, c0, TC);
  if (n <= 0) return;
  logit_launch<false, Off>(LogitIn{hidden, W, idx + c0, token_id, n, H, V, INT_MAX}, n_vtiles, smem,
                           FwdEpilogue<ENT>{part_m, part_s, part_u, zy, TC});
}

// Stores eight consecutive bf16 outputs of a lane.
__device__ __forceinline__ void store8(bf16_t* p, const float (&d)[8]) {
  *reinterpret_cast<uint4*>(p) = make_uint4(pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3]), pack_bf16x2(d[4], d[5]),
                                            pack_bf16x2(d[6], d[7]));
}

// ------------------------------------------------------------------------------------------------
// exponentials (one-pass forward + backward): E[j][v] = exp(z - c_j) for the tokens j of the launch (zero for the padding
// columns V .. Vp and for the rows that pad the last tile); part_s = sums over the vocabulary rows of each tile, at part_index();
// zy[j] = target logit
// ------------------------------------------------------------------------------------------------
struct FeEpilogue {
  const float* c2;
  bf16_t* E;
  float *part_s, *zy;
  int Vp, TC;

  template <typename G>
  struct Fetched {
    float nc2[G::kJB];
    __device__ __forceinline__ void settle() {
#pragma unroll
      for (int j = 0; j < G::kJB; ++j) asm volatile("" : "+v"(nc2[j]));
    }
  };
  template <typename G>
  __device__ __forceinline__ void fetch(Fetched<G>& f, const TokenCols<G>&, const LogitIn& in, int t0, const Coord16<G>& co) const {
#pragma unroll
    for (int j = 0; j < G::kJB; ++j) f.nc2[j] = -c2[min(t0 + co.b_row(j), in.n - 1)];
  }

  template <typename G>
  __device__ __forceinline__ void finish(const floatx4 (&acc)[G::kIB][G::kJB], const TokenCols<G>& cols, const Fetched<G>& f,
                                         int v0, int t0, const LogitIn& in, char* lds) const {
    constexpr int T = G::kTileB;
    float* red_s = reinterpret_cast<float*>(lds);   // [kWavesA][T]
    const Coord16<G> co;
    const int n = in.n, V = in.V;
    const int vbase = v0 + co.wm * G::kRowsA;
    // tiles that lie fully inside the vocabulary and the token list need no per-element range checks
    const bool interior = (v0 + G::kTileA <= V) && (t0 + T <= n);
#pragma unroll
    for (int j = 0; j < G::kJB; ++j) {
      const int tcol = t0 + co.b_row(j);
      const bool live = tcol < n;
      const int rel = cols.y[j] - vbase;
      const float nc2 = f.nc2[j];
      const bool hit = live && rel >= 0 && rel < G::kRowsA && ((rel >> 3) & 3) == (co.lane >> 4);
      if (__builtin_amdgcn_ballot_w64(hit) != 0ull) {
        floatx4 col[G::kIB];
#pragma unroll
        for (int i = 0; i < G::kIB; ++i) col[i] = acc[i][j];
        const float zt = pick<G::kIB>(col, ((rel >> 5) << 1) | ((rel >> 2) & 1), rel & 3);
        if (hit) zy[tcol] = zt;
      }
      bf16_t* row = E + static_cast<size_t>(tcol) * Vp + vbase;
      float sum = 0.f;
#pragma unroll
      for (int p = 0; p < G::kIB / 2; ++p) {
        const int vf = pair_first(p, co.lane);
        float d[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) d[e] = fast_exp2(fmaf(acc[2 * p + (e >> 2)][j][e & 3], kLog2e, nc2));
        if (!interior) {
#pragma unroll
          for (int e = 0; e < 8; ++e) d[e] = (vbase + vf + e < V && live) ? d[e] : 0.f;
        }
        sum += ((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7]));
        if (interior || (vbase + vf < Vp && tcol < in.pad_end)) store8(row + vf, d);
      }
      sum = across_groups_sum(sum);
      if (co.lane < 16) red_s[co.wm * T + co.b_row(j)] = sum;
    }
    lds_barrier();      // the sums are free again behind the next step's barrier
    const int tl = co.wave * 64 + co.lane;
    if (tl < T && t0 + tl < n) {
      float S = 0.f;
#pragma unroll
      for (int q = 0; q < G::kWavesA; ++q) S += red_s[q * T + tl];
      part_s[part_index<G>(v0, t0 + tl, TC)] = S;
    }
  }
};

template <typename Off>
__global__ __launch_bounds__(GLogit::kThreads) void k_head_fe(
    const bf16_t* __restrict__ hidden, const bf16_t* __restrict__ W, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ cnt, int c0, const int32_t* __restrict__ token_id, const float* __restrict__ c2,
    bf16_t* __restrict__ E, float* __restrict__ part_s, float* __restrict__ zy, int H, int V, int Vp, int TC, int n_vtiles) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int n = chunk_count(cnt, c0, TC);
  if (n <= 0) return;
  logit_launch<true, Off>(LogitIn{hidden, W, idx + c0, token_id, n, H, V, INT_MAX}, n_vtiles, smem,
                          FeEpilogue{c2, E, part_s, zy, Vp, TC});
}

// ------------------------------------------------------------------------------------------------
// logit gradient with the logits recomputed (two-call path, and the fallback of the one-pass step):
// dZ[t][v] = g_t ([v = y_t] - exp(z - lse_t)); without coefficients g = -1 (softmax - onehot)
// ------------------------------------------------------------------------------------------------
struct DzEpilogue {
  const float *lse, *coef;
  bf16_t* dZ;
  int Vp;

  template <typename G>
  struct Fetched {
    float g[G::kJB], l[G::kJB];
    __device__ __forceinline__ void settle() {
#pragma unroll
      for (int j = 0; j < G::kJB; ++j) asm volatile("" : "+v"(g[j]), "+v"(l[j]));
    }
  };
  template <typename G>
  __device__ __forceinline__ void fetch(Fetched<G>& f, const TokenCols<G>& cols, const LogitIn&, int, const Coord16<G>&) const {
#pragma unroll
    for (int j = 0; j < G::kJB; ++j) {
      f.g[j] = coef ? coef[cols.row[j]] : -1.f;
      f.l[j] = lse[cols.row[j]];
    }
  }

  template <typename G>
  __device__ __forceinline__ void finish(const floatx4 (&acc)[G::kIB][G::kJB], const TokenCols<G>& cols, const Fetched<G>& f,
                                         int v0, int t0, const LogitIn& in, char*) const {
    const Coord16<G> co;
    const int n = in.n, V = in.V;
    const int vbase = v0 + co.wm * G::kRowsA;
    const bool interior = (v0 + G::kTileA <= V) && (t0 + G::kTileB <= n);
#pragma unroll
    for (int j = 0; j < G::kJB; ++j) {
      const int tcol = t0 + co.b_row(j);
      const bool live = tcol < n;
      const int rel = cols.y[j] - vbase;
      const float g = f.g[j], nl2 = -f.l[j] * kLog2e;
      bf16_t* row = dZ + static_cast<size_t>(tcol) * Vp + vbase;
#pragma unroll
      for (int p = 0; p < G::kIB / 2; ++p) {
        const int vf = pair_first(p, co.lane);
        float d[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) d[e] = -g * fast_exp2(fmaf(acc[2 * p + (e >> 2)][j][e & 3], kLog2e, nl2));
        if (static_cast<unsigned>(rel - vf) < 8u) {      // the onehot term: one element in V per token
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (rel - vf == e) d[e] += g;
        }
        if (!interior) {
#pragma unroll
          for (int e = 0; e < 8; ++e) d[e] = (vbase + vf + e < V && live) ? d[e] : 0.f;
        }
        if (interior || (vbase + vf < Vp && tcol < in.pad_end)) store8(row + vf, d);
      }
    }
  }
};

template <typename Off>
__global__ __launch_bounds__(GLogit::kThreads) void k_head_dz(
    const bf16_t* __restrict__ hidden, const bf16_t* __restrict__ W, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ cnt, int c0, const int32_t* __restrict__ token_id, const float* __restrict__ lse,
    const float* __restrict__ coef, bf16_t* __restrict__ dZ, int H, int V, int Vp, int TC, int n_vtiles,
    const int32_t* __restrict__ gate) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  if (gate && *gate == 0) return;
  const int n = chunk_count(cnt, c0, TC);
  if (n <= 0) return;
  logit_launch<true, Off>(LogitIn{hidden, W, idx + c0, token_id, n, H, V, INT_MAX}, n_vtiles, smem, DzEpilogue{lse, coef, dZ, Vp});
}

// ---- partial tiles of a split contraction (split_k.hpp), in the accumulator layout of grid G -----------------------
template <typename G>
__device__ __forceinline__ size_t partial_at(int slot, int wave, int i, int j, int lane) {
  return static_cast<size_t>(slot) * (kTile16 * kTile16 / 4) + ((wave * G::kIB + i) * G::kJB + j) * 64 + lane;
}

template <typename G>
__device__ __forceinline__ void store_partial(floatx4* part, int slot, const floatx4 (&acc)[G::kIB][G::kJB], const Coord16<G>& co) {
#pragma unroll
  for (int j = 0; j < G::kJB; ++j)
#pragma unroll
    for (int i = 0; i < G::kIB; ++i) part[partial_at<G>(slot, co.wave, i, j, co.lane)] = acc[i][j];
}

// One wavefront's column block j of split tile q: the sum of its S parts.  unit = (q * wavefronts + wave) * kJB + j.
template <typename G>
__device__ __forceinline__ void load_partials(floatx4 (&col)[G::kIB], const floatx4* part, const SplitK& sp, int q, int wave,
                                              int j, int lane) {
#pragma unroll
  for (int i = 0; i < G::kIB; ++i) col[i] = part[partial_at<G>(q, wave, i, j, lane)];
  for (int s = 1; s < sp.S; ++s)
#pragma unroll
    for (int i = 0; i < G::kIB; ++i) col[i] += part[partial_at<G>(s * sp.rest + q, wave, i, j, lane)];
}

constexpr int kReduceBlocks = 2048, kReduceThreads = 256;

// ------------------------------------------------------------------------------------------------
// Wt[h][v] = W[v][h], zero for V <= v < Vp: tiles of 64 v x 128 h through LDS, turned by the transposing LDS read (four
// v of one h per lane and read).  Loads are 256-byte runs of W, stores 128-byte runs of Wt.  Bound by memory: 2.49 GB
// in 487 us at V = 151936, H = 4096 (963 us with 64 x 64 tiles and 2-byte accesses).
// ------------------------------------------------------------------------------------------------
constexpr int kTpThreads = 256, kTpV = 64, kTpH = 128;

__global__ __launch_bounds__(kTpThreads) void k_transpose_w(const bf16_t* __restrict__ W, int V, int Vp, int H,
                                                            bf16_t* __restrict__ Wt, const int32_t* __restrict__ cnt,
                                                            int min_rows) {
  __shared__ __attribute__((aligned(16))) char tile[kTpV * kTpH * 2];
  if (*cnt <= min_rows) return;       // dHidden reads W itself
  const int v0 = blockIdx.x * kTpV, h0 = blockIdx.y * kTpH;
  const int c = threadIdx.x & 15;     // 16-byte chunk of a row
#pragma unroll
  for (int p = 0; p < kTpV / 16; ++p) {
    const int k = p * 16 + (threadIdx.x >> 4), s = (k & 3) | (((k >> 3) & 1) << 2);
    uint4 x = make_uint4(0, 0, 0, 0);
    if (v0 + k < V && h0 + c * 8 < H) x = *reinterpret_cast<const uint4*>(W + static_cast<size_t>(v0 + k) * H + h0 + c * 8);
    *reinterpret_cast<uint4*>(tile + k * (kTpH * 2) + ((c ^ (2 * s)) & 15) * 16) = x;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, r = (lane & 15) >> 2, q = lane & 3;
  const int k = 8 * g + r, s = (k & 3) | (((k >> 3) & 1) << 2);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int hb = (wave + 4 * b) * 16, h = h0 + hb + (lane & 15);
    const int cc = hb / 8 + (q >> 1);
    const char* at = tile + k * (kTpH * 2) + ((cc ^ (2 * s)) & 15) * 16 + (q & 1) * 8;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const uint2 lo = lds_read_tr(at + half * 32 * (kTpH * 2)), hi = lds_read_tr(at + (half * 32 + 4) * (kTpH * 2));
      if (h < H)
        *reinterpret_cast<uint4*>(Wt + static_cast<size_t>(h) * Vp + v0 + half * 32 + g * 8) = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// dHidden: A = columns of W (h), B = dZ / E rows (tokens), k = vocabulary.
// For many rows W is transposed first and both operands are contiguous along k (1552 TFLOP/s); for few rows the contraction reads
// W as it stands, k-major (1486 on the same box), and the transposition is saved.  Per weight the transposition takes 0.8 ps (H =
// 4096) to 1.1 ps (H = 2048) of the chip, the slower loop 0.06 to 0.08 fs per row: the two meet between 10 000 and 18 000 rows of a
// head, and on either side of the line the wrong choice costs 1 % of this contraction at the most.
// ------------------------------------------------------------------------------------------------
constexpr int kUntransposedRows = 12288;

struct DhArgs {
  const bf16_t* dZ;
  const bf16_t* W;            // [V][H]
  const bf16_t* Wt;           // [H][Vp], read when the head has more than kUntransposedRows rows
  const int32_t* idx;
  const int32_t* cnt;
  int c0;
  bf16_t* d_hidden;
  int H, V, Vp, TC;
  const float* scale;         // row factors of the one-pass path, or null
  const int32_t* perm;        // after the rows were compacted: row j of dZ belongs to list position perm[j] ...
  const int32_t* live_cnt;    // ... and only the first *live_cnt rows take part
  floatx4* part;              // partial tiles
};

__device__ __forceinline__ int rows_of(const int32_t* live_cnt, const int32_t* cnt, int c0, int TC) {
  const int n = chunk_count(cnt, c0, TC);
  return live_cnt ? min(*live_cnt, n) : n;
}

// T: the launch works on transposed weights.  Lane outputs of a block column: with a_index() on the rows of Wt pairs of
// blocks are eight consecutive h; columns of W are taken as they are, four consecutive h per block.
template <bool T>
__device__ __forceinline__ void dh_store(const DhArgs& a, const floatx4 (&col)[GDh::kIB], int jt, int n, int hbase, int lane) {
  if (jt >= n) return;
  const int jl = a.perm ? a.perm[jt] : jt;
  const float sc = a.scale ? a.scale[jl] : 1.f;
  bf16_t* out = a.d_hidden + static_cast<size_t>(a.idx[a.c0 + jl]) * a.H + hbase;
  if (T) {
#pragma unroll
    for (int p = 0; p < GDh::kIB / 2; ++p) {
      const int hf = pair_first(p, lane);
      float d[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = col[2 * p + (e >> 2)][e & 3] * sc;
      if (hbase + hf < a.H) store8(out + hf, d);
    }
  } else {
#pragma unroll
    for (int i = 0; i < GDh::kIB; ++i) {
      const int hf = i * 16 + 4 * (lane >> 4);
      const floatx4 d = col[i] * sc;
      if (hbase + hf < a.H) *reinterpret_cast<uint2*>(out + hf) = make_uint2(pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3]));
    }
  }
}

__device__ __forceinline__ TileOrder dh_order(int n, int H) {
  return TileOrder{(n + kTile16 - 1) / kTile16, (H + kTile16 - 1) / kTile16, 8};
}

template <bool T, typename Off, bool ONCE>
__device__ __forceinline__ void dh_tiles(const DhArgs& a, int n) {
  using G = GDh;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const TileOrder ord = dh_order(n, a.H);
  const int nk_all = a.Vp / kStepK;
  const SplitK sp = plan_split(ord.total(), nk_all, gridDim.x);
  const Off row_bytes = static_cast<Off>(a.Vp) * 2;
  const int items = sp.full + sp.rest * sp.S;

  for (int it = logical_workgroup(); it < items; it += gridDim.x) {
    const int part = it < sp.full ? 0 : (it - sp.full) / sp.rest;
    const int tile = it < sp.full ? it : it - part * sp.rest;
    int tt, ht;
    ord.decode(tile, &tt, &ht);
    const int t0 = tt * kTile16, h0 = ht * kTile16;
    const bool split = it >= sp.full && sp.S > 1;
    const int k0 = split ? part * sp.chunk : 0;
    const int nk = split ? min(sp.chunk, nk_all - k0) : nk_all;
    floatx4 acc[G::kIB][G::kJB];
    {
      const Coord16<G> co;
      RowPanel<G::kLoadsB, Off> pb;
      const size_t kb = static_cast<size_t>(k0) * kStepK * 2;
      pb.init(reinterpret_cast<const char*>(a.dZ) + static_cast<size_t>(t0) * row_bytes + kb, co.wave, co.lane,
              [&](int row) { return static_cast<Off>(row) * row_bytes; });
      if constexpr (T) {
        RowPanel<G::kLoadsA, Off> pa;
        pa.init(reinterpret_cast<const char*>(a.Wt) + static_cast<size_t>(h0) * row_bytes + kb, co.wave, co.lane,
                [&](int row) { return static_cast<Off>(min(a_index(row), a.H - 1 - h0)) * row_bytes; });
        gemm16<G>(acc, pa, pb, nk, smem, co);
      } else {
        KMajorTailPanel<G::kLoadsA, Off, ONCE> pa;
        pa.init(reinterpret_cast<const char*>(a.W + static_cast<size_t>(k0) * kStepK * a.H + h0), co.wave, co.lane,
                static_cast<size_t>(a.H) * 2, min(31, (a.H - h0) / 8 - 1), a.V - k0 * kStepK);
        gemm16<G>(acc, pa, pb, nk, smem, co);
      }
    }
    const Coord16<G> co;
    if (split) {
      store_partial<G>(a.part, it - sp.full, acc, co);
    } else {
#pragma unroll
      for (int j = 0; j < G::kJB; ++j) {
        floatx4 col[G::kIB];
#pragma unroll
        for (int i = 0; i < G::kIB; ++i) col[i] = acc[i][j];
        dh_store<T>(a, col, t0 + co.b_row(j), n, h0 + co.wm * G::kRowsA, co.lane);
      }
    }
  }
}

template <bool T, typename Off>
__global__ __launch_bounds__(GDh::kThreads) void k_head_dh(DhArgs a) {
  if ((*a.cnt > kUntransposedRows) != T) return;
  const int n = rows_of(a.perm ? a.live_cnt : nullptr, a.cnt, a.c0, a.TC);
  if (n <= 0) return;
  if constexpr (!T && sizeof(Off) == 4) {
    if (read_once(n, a.V, a.H)) {
      dh_tiles<T, Off, true>(a, n);
      return;
    }
  }
  dh_tiles<T, Off, false>(a, n);
}

// adds the parts of the split tiles and finishes them; `grid` = workgroups of the contraction
__global__ __launch_bounds__(kReduceThreads) void k_head_dh_reduce(DhArgs a, int grid) {
  using G = GDh;
  const int n = rows_of(a.perm ? a.live_cnt : nullptr, a.cnt, a.c0, a.TC);
  if (n <= 0) return;
  const TileOrder ord = dh_order(n, a.H);
  const SplitK sp = plan_split(ord.total(), a.Vp / kStepK, grid);
  if (sp.S <= 1) return;
  const bool transposed = *a.cnt > kUntransposedRows;
  constexpr int kWaves = G::kThreads / 64;
  const int lane = threadIdx.x & 63;
  const int units = sp.rest * kWaves * G::kJB;
  for (int u = (blockIdx.x * kReduceThreads + threadIdx.x) >> 6; u < units; u += (gridDim.x * kReduceThreads) >> 6) {
    const int j = u % G::kJB, wave = u / G::kJB % kWaves, q = u / (G::kJB * kWaves);
    int tt, ht;
    ord.decode(sp.full + q, &tt, &ht);
    floatx4 col[G::kIB];
    load_partials<G>(col, a.part, sp, q, wave, j, lane);
    const int jt = tt * kTile16 + (wave % G::kWavesB) * G::kRowsB + j * 16 + (lane & 15);
    const int hbase = ht * kTile16 + (wave / G::kWavesB) * G::kRowsA;
    if (transposed) dh_store<true>(a, col, jt, n, hbase, lane);
    else dh_store<false>(a, col, jt, n, hbase, lane);
  }
}

// ------------------------------------------------------------------------------------------------
// dW[v][h] (+)= sum_t dZ[t][v] * hG[t][h]: A = hG columns (h), B = dZ columns (v), both k-major, k = tokens
// ------------------------------------------------------------------------------------------------
struct DwArgs {
  const bf16_t* dZ;
  const bf16_t* hG;
  const int32_t* cnt;
  int c0;
  float* dW;
  int H, V, Vp, TC, n_vtiles, accumulate, first_chunk;
  const int32_t* live_cnt;    // or null: the rows were compacted, only the first *live_cnt take part
  floatx4* part;              // partial tiles
};

// A wavefront's sub-tile, NJ block columns at a time; v0, h0: of the tile.  ADD: the values to add are requested for all NJ
// columns before the first is stored.  Without ADD nothing is read, and nothing may wait: neither the choice between the two nor
// the check of the vocabulary's end is made between the stores, since a register that a load may be on its way to makes
// them wait for everything in flight.
template <typename G, int NJ, bool ADD>
__device__ __forceinline__ void dw_store_tile(const DwArgs& a, const floatx4 (&acc)[G::kIB][G::kJB], int v0, int h0,
                                              const Coord16<G>& co) {
  const int hb = h0 + co.wm * G::kRowsA;
  auto at = [&](int j) {
    return reinterpret_cast<f32x4_any*>(a.dW + static_cast<size_t>(v0 + co.b_row(j)) * a.H + hb + 4 * (co.lane >> 4));
  };
  if (hb + G::kRowsA <= a.H && v0 + G::kTileB <= a.V) {
#pragma unroll
    for (int j0 = 0; j0 < G::kJB; j0 += NJ) {
      floatx4 x[NJ][G::kIB];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < G::kIB; ++i) x[j][i] = ADD ? at(j0 + j)[i * 4] + acc[i][j0 + j] : acc[i][j0 + j];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < G::kIB; ++i) at(j0 + j)[i * 4] = x[j][i];
    }
  } else {
#pragma unroll
    for (int j = 0; j < G::kJB; ++j)
#pragma unroll
      for (int i = 0; i < G::kIB; ++i)      // a whole block of 16 columns exists or does not (H % 64 == 0)
        if (v0 + co.b_row(j) < a.V && hb + i * 16 < a.H) at(j)[i * 4] = ADD ? at(j)[i * 4] + acc[i][j] : acc[i][j];
  }
}

// bands of 32 / (tiles along H) vocabulary tiles: the 32 workgroups that share an XCD's L2 then cover every
// H-tile of the same few vocabulary tiles, and each panel of the large operand (the 10 GB of dZ rows)
// is fetched by one XCD only (measured 2.4 % faster than bands of 8)
__device__ __forceinline__ TileOrder dw_order(int n_vtiles, int H) {
  const int n_htiles = (H + kTile16 - 1) / kTile16;
  return TileOrder{n_vtiles, n_htiles, max(1, 32 / n_htiles)};
}

// k-steps of n rows.  The rows of the last step that do not exist are zero in hG and finite in dZ.  (In whole tiles of 256 rows
// before: 64 tokens at H = 2048 362 -> 250 us.)
__device__ __forceinline__ int dw_steps(int n) { return (n + kStepK - 1) / kStepK; }

template <typename Off>
__global__ __launch_bounds__(GDw::kThreads) void k_head_dw(DwArgs a) {
  using G = GDw;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int n = rows_of(a.live_cnt, a.cnt, a.c0, a.TC);
  if (n <= 0 && !(a.first_chunk && !a.accumulate)) return;
  const TileOrder ord = dw_order(a.n_vtiles, a.H);
  const int nk_all = dw_steps(n);
  const SplitK sp = plan_split(ord.total(), nk_all, gridDim.x);
  const int items = sp.full + sp.rest * sp.S;

  for (int it = logical_workgroup(); it < items; it += gridDim.x) {
    const int part = it < sp.full ? 0 : (it - sp.full) / sp.rest;
    const int tile = it < sp.full ? it : it - part * sp.rest;
    int vt, ht;
    ord.decode(tile, &vt, &ht);
    const int v0 = vt * kTile16, h0 = ht * kTile16;
    const bool split = it >= sp.full && sp.S > 1;
    const int k0 = split ? part * sp.chunk : 0;
    const int nk = split ? min(sp.chunk, nk_all - k0) : nk_all;
    floatx4 acc[G::kIB][G::kJB];
    {
      const Coord16<G> co;
      KMajorPanel<G::kLoadsA, Off> pa;
      KMajorPanel<G::kLoadsB, Off> pb;
      pa.init(reinterpret_cast<const char*>(a.hG + static_cast<size_t>(k0) * kStepK * a.H + h0), co.wave, co.lane,
              static_cast<size_t>(a.H) * 2, min(31, (a.H - h0) / 8 - 1));
      pb.init(reinterpret_cast<const char*>(a.dZ + static_cast<size_t>(k0) * kStepK * a.Vp + v0), co.wave, co.lane,
              static_cast<size_t>(a.Vp) * 2, min(31, (a.Vp - v0) / 8 - 1));
      gemm16<G>(acc, pa, pb, nk, smem, co);
    }
    const Coord16<G> co;
    constexpr int kCols = sizeof(Off) == 4 ? 4 : 1;      // (64-bit offsets leave no registers for more)
    if (split) store_partial<G>(a.part, it - sp.full, acc, co);
    else if (a.accumulate) dw_store_tile<G, kCols, true>(a, acc, v0, h0, co);
    else dw_store_tile<G, kCols, false>(a, acc, v0, h0, co);
  }
}

__global__ __launch_bounds__(kReduceThreads) void k_head_dw_reduce(DwArgs a, int grid) {
  using G = GDw;
  const int n = rows_of(a.live_cnt, a.cnt, a.c0, a.TC);
  if (n <= 0) return;
  const TileOrder ord = dw_order(a.n_vtiles, a.H);
  const SplitK sp = plan_split(ord.total(), dw_steps(n), grid);
  if (sp.S <= 1) return;
  constexpr int kWaves = G::kThreads / 64;
  const int lane = threadIdx.x & 63;
  const int units = sp.rest * kWaves * G::kJB;
  for (int u = (blockIdx.x * kReduceThreads + threadIdx.x) >> 6; u < units; u += (gridDim.x * kReduceThreads) >> 6) {
    const int j = u % G::kJB, wave = u / G::kJB % kWaves, q = u / (G::kJB * kWaves);
    int vt, ht;
    ord.decode(sp.full + q, &vt, &ht);
    floatx4 col[G::kIB];
    load_partials<G>(col, a.part, sp, q, wave, j, lane);
    const int v = vt * kTile16 + (wave % G::kWavesB) * G::kRowsB + j * 16 + (lane & 15);
    const int hb = ht * kTile16 + (wave / G::kWavesB) * G::kRowsA;
    f32x4_any* out = reinterpret_cast<f32x4_any*>(a.dW + static_cast<size_t>(v) * a.H + hb + 4 * (lane >> 4));
    if (v >= a.V) continue;
#pragma unroll
    for (int i = 0; i < G::kIB; ++i)
      if (a.accumulate && hb + i * 16 < a.H) col[i] += out[i * 4];
#pragma unroll
    for (int i = 0; i < G::kIB; ++i)
      if (hb + i * 16 < a.H) out[i * 4] = col[i];
  }
}

}  // namespace

// ================================================================================================
// launchers
// ================================================================================================
namespace {

// 256 rows of W, Wt or dZ span 4 GiB or more (a vocabulary or a hidden size beyond 8.3 million): 64-bit offsets in the panels
bool wide_rows(const HeadGeom& g) { return static_cast<int64_t>(g.H > g.Vp ? g.H : g.Vp) * 2 * kTile16 >= int64_t{1} << 32; }

}  // namespace


int launch_fwd_bf16(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                    float* part_m, float* part_s, float* part_u, float* zy, hipStream_t s, const int32_t* gate) {
  auto k = wide_rows(g) ? (part_u ? k_head_fwd<true, uint64_t> : k_head_fwd<false, uint64_t>)
                        : (part_u ? k_head_fwd<true, uint32_t> : k_head_fwd<false, uint32_t>);
  ATG_TRY(allow_big_lds(k, kRingBytes));
  hipLaunchKernelGGL(k, dim3(gemm_grid()), dim3(GLogit::kThreads), kRingBytes, s, static_cast<const bf16_t*>(hidden),
                     static_cast<const bf16_t*>(W), ch.idx, ch.cnt, ch.c0, token_id, part_m, part_s, part_u, zy, g.H, g.V,
                     g.TC, g.n_vtiles, gate);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_fe_bf16(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                   const float* c2, void* E, float* part_s, float* zy, hipStream_t s) {
  auto k = wide_rows(g) ? k_head_fe<uint64_t> : k_head_fe<uint32_t>;
  ATG_TRY(allow_big_lds(k, kRingBytes));
  hipLaunchKernelGGL(k, dim3(gemm_grid()), dim3(GLogit::kThreads), kRingBytes, s, static_cast<const bf16_t*>(hidden),
                     static_cast<const bf16_t*>(W), ch.idx, ch.cnt, ch.c0, token_id, c2, static_cast<bf16_t*>(E), part_s,
                     zy, g.H, g.V, g.Vp, g.TC, g.n_vtiles);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_dz_bf16(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                   const float* lse, const float* coef, void* dZ, hipStream_t s, const int32_t* gate) {
  auto k = wide_rows(g) ? k_head_dz<uint64_t> : k_head_dz<uint32_t>;
  ATG_TRY(allow_big_lds(k, kRingBytes));
  hipLaunchKernelGGL(k, dim3(gemm_grid()), dim3(GLogit::kThreads), kRingBytes, s, static_cast<const bf16_t*>(hidden),
                     static_cast<const bf16_t*>(W), ch.idx, ch.cnt, ch.c0, token_id, lse, coef, static_cast<bf16_t*>(dZ),
                     g.H, g.V, g.Vp, g.TC, g.n_vtiles, gate);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

bool narrow_launches_bf16(const HeadGeom& g) { return !wide_rows(g); }

bool transposes_w_bf16(int64_t n_tok) { return n_tok > kUntransposedRows; }

int launch_transpose_w_bf16(const HeadGeom& g, const void* W, void* Wt, const int32_t* cnt, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(ceil_div(g.Vp, kTpV)), static_cast<unsigned>(ceil_div(g.H, kTpH)));
  hipLaunchKernelGGL(k_transpose_w, grid, dim3(kTpThreads), 0, s, static_cast<const bf16_t*>(W), g.V, g.Vp, g.H,
                     static_cast<bf16_t*>(Wt), cnt, kUntransposedRows);
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_dh_bf16(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* W, const void* Wt, void* d_hidden,
                   void* part, hipStream_t s, const float* scale, const int32_t* perm, const int32_t* live_cnt) {
  const DhArgs a{static_cast<const bf16_t*>(dZ), static_cast<const bf16_t*>(W), static_cast<const bf16_t*>(Wt), ch.idx,
                 ch.cnt, ch.c0, static_cast<bf16_t*>(d_hidden), g.H, g.V, g.Vp, g.TC, scale, perm, live_cnt,
                 static_cast<floatx4*>(part)};
  // which of the two has work is only known on the device, unless the list is too short or the chunk too far behind
  if (Wt) {
    auto k = wide_rows(g) ? k_head_dh<true, uint64_t> : k_head_dh<true, uint32_t>;
    ATG_TRY(allow_big_lds(k, kRingBytes));
    hipLaunchKernelGGL(k, dim3(gemm_grid()), dim3(GDh::kThreads), kRingBytes, s, a);
    ATG_LAUNCH_CHECK();
  }
  if (ch.c0 < kUntransposedRows) {
    auto k = wide_rows(g) ? k_head_dh<false, uint64_t> : k_head_dh<false, uint32_t>;
    ATG_TRY(allow_big_lds(k, kRingBytes));
    hipLaunchKernelGGL(k, dim3(gemm_grid()), dim3(GDh::kThreads), kRingBytes, s, a);
    ATG_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(k_head_dh_reduce, dim3(kReduceBlocks), dim3(kReduceThreads), 0, s, a, gemm_grid());
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

int launch_dw_bf16(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* hG, float* dW, void* part,
                   int accumulate, int first_chunk, hipStream_t s, const int32_t* live_cnt) {
  const DwArgs a{static_cast<const bf16_t*>(dZ), static_cast<const bf16_t*>(hG), ch.cnt, ch.c0, dW, g.H, g.V, g.Vp, g.TC,
                 g.n_vtiles, accumulate, first_chunk, live_cnt, static_cast<floatx4*>(part)};
  auto k = wide_rows(g) ? k_head_dw<uint64_t> : k_head_dw<uint32_t>;
  ATG_TRY(allow_big_lds(k, kRingBytes));
  hipLaunchKernelGGL(k, dim3(gemm_grid()), dim3(GDw::kThreads), kRingBytes, s, a);
  ATG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_head_dw_reduce, dim3(kReduceBlocks), dim3(kReduceThreads), 0, s, a, gemm_grid());
  ATG_LAUNCH_CHECK();
  return AT_GRPO_OK;
}

}  // namespace atg

// Workgroup-tile contraction of bf16 operands on the gfx950 matrix cores.
//
// One workgroup produces a 256 x 256 fp32 tile (or a part of one, see Grid16)
//   C[a, b] = sum_k A[a, k] * B[b, k]
// where each operand may be stored with its rows contiguous along k or k-major (rows of k, contiguous along
// a or b).  Its wavefronts share the tile as a Grid16 (below).  k is consumed in steps of 64.
//
// MFMA shape.  v_mfma_f32_16x16x32_bf16, not 32x32x16: both deliver the same peak, but these kernels are bound by
// power, and per multiply-add the 16x16x32 form moves half as many accumulator words through the register file.
// On 256 x 256 tiles 32x32x16 gave 1360 TFLOP/s at 1.59 GHz (k = 2048, the logits) and 1310 at 1.44-1.54 (k = 151936,
// dHidden); 16x16x32 gave 1427-1473 at 1.74-1.82 and 1477-1523 at 1.68-1.74 (five runs on four boxes), and with the ring as it is
// now 1550 at 1.84 and 1552 at 1.77 (1422 on dW's shape, 1339-1410 before).
//
// Data path: global -> LDS with direct-to-LDS loads (global_load_lds_dwordx4, 16 bytes per lane) into a ring of five
// 32 KiB slots (one operand panel each: all 160 KiB of a compute unit); LDS -> registers with ds_read_b128 (operands
// contiguous along k) or the transposing ds_read_b64_tr_b16 (k-major operands), fragments fetched one 32-wide sub-step
// ahead of the MFMAs that consume them.  The direct loads go through inline asm: the compiler would otherwise make
// every later LDS read wait for all outstanding direct loads.  Their completion is enforced by hand with s_waitcnt vmcnt
// in front of the one workgroup barrier per k-step.  No value that the k loop uses may come from a load the compiler
// has to wait for inside the loop (a spilled register, say): such a wait would drain the direct loads too.  (In the assembly, what
// the kernels of head_bf16.hip spill lies outside their k loops, except four words a step of dW with 64-bit offsets.)
//
// Instruction order: a wavefront that issues a burst of LDS reads or direct loads keeps its SIMD's matrix pipe idle for
// the length of the burst.  The loop body is therefore written out as a fixed sequence, pinned with scheduling barriers,
// in which an MFMA is followed by at most one fragment read and one direct load.  Addresses cost no vector instructions
// in the loop: global addresses are a scalar base plus a lane offset that does not change, LDS addresses a lane offset
// per slot plus an immediate.
//
// Accumulator layout (per lane, block (i, j), register r = 0..3):
//   A row of the tile = wm * kRowsA + i * 16 + 4 * (lane / 16) + r
//   B row of the tile = wn * kRowsB + j * 16 + lane % 16
// i.e. four consecutive A rows per lane: A is the operand whose index is contiguous in the output.
#pragma once

#include "common.hpp"

namespace atg {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16v8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16v4 __attribute__((__vector_size__(4 * sizeof(__bf16))));

constexpr int kTile16 = 256;                      // rows of each operand per tile
constexpr int kStepK = 64;                        // k per step
constexpr int kRingSlots = 5;
constexpr int kRingSlot = kTile16 * kStepK * 2;   // 32 KiB: one operand panel of one step
constexpr int kRingBytes = kRingSlots * kRingSlot;
constexpr int kRingA = 3 * kRingSlot;             // the first three slots are A's, the others B's
constexpr int kRingFree = 2 * kRingSlot;          // the slot that a tile's first two steps leave to the epilogue in front of it

// How the wavefronts of a workgroup share the TA x TB tile: WA x WB of them, each owning (TA / WA) x (TB / WB).
//   Grid16<4, 2> / <2, 4>  8 wavefronts, two per SIMD (128 accumulator registers): one covers part of the other's
//                          per-tile prologue and epilogue; used where the k loop is short (k = H)
//   Grid16<2, 2>           4 wavefronts, one per SIMD (256 accumulator registers): a third fewer LDS reads per MFMA and
//                          half as many wavefronts at each barrier; 2 % faster on the long k loop of dHidden
// Tiles of fewer than 256 rows of an operand still take a whole ring slot per panel.
template <int WA, int WB, int TA = kTile16, int TB = kTile16>
struct Grid16 {
  static constexpr int kWavesA = WA, kWavesB = WB, kThreads = WA * WB * 64;
  static constexpr int kTileA = TA, kTileB = TB;
  static constexpr int kRowsA = TA / WA, kRowsB = TB / WB;             // rows of a wavefront's sub-tile
  static constexpr int kIB = kRowsA / 16, kJB = kRowsB / 16;           // accumulator blocks of a wavefront
  static constexpr int kLoadsA = TA / 8 / (WA * WB);                   // direct loads per step and wavefront
  static constexpr int kLoadsB = (TB / 8 + WA * WB - 1) / (WA * WB);   // (TB = 160 or 224 on 8 wavefronts: rows past the tile's, unused)
  static constexpr int kMm = kIB * kJB, kRd = kIB + kJB;               // MFMAs and fragment reads per sub-step
  // a fragment read follows every kRdEvery-th MFMA: the last one must be early enough to land before the sub-step ends
  // (4 wavefronts, same box: every 3rd 1494 TFLOP/s at k = 151936 and 1414 with a k-major operand, every 4th 1472 and 1377)
  static constexpr int kRdEvery = (kMm / kRd >= 4) ? kMm / kRd - 1 : kMm / kRd;
  // When the loads of Gemm16 are issued: a step's B loads behind the first kSpanB MFMAs of its sub-step, the first kFirstA of its A
  // loads behind the others there, and the rest in the next sub-step.  With two wavefronts per SIMD, B within a quarter, as it has the
  // least time to land, and A in two halves; with one, evenly.  Ms a call at V = 151936 under full load, B over a quarter with half of
  // A / over a quarter without A / evenly without A: dW of 250000 rows at H = 2048 106.1, 109.2, 109.5, exponentials 110.1, 109.8,
  // 110.2, dHidden 101.0, 100.1, 99.4; dHidden of 37000 at H = 4096 on three heads 32.9, 33.0, 32.8.  In short bursts, where the clock
  // is higher, the exponentials of 20000 rows take 8.94, 8.95 and 9.70 ms.
  static constexpr int kSpanB = WA * WB == 4 ? kMm : kMm / 4;
  static constexpr int kFirstA = WA * WB == 4 ? 0 : kLoadsA / 2;
  static_assert(kRowsA % 16 == 0 && kRowsB % 16 == 0 && kLoadsA >= 1 && kLoadsB >= 1, "whole blocks, whole loads");
  static_assert(kLoadsB <= kSpanB && kFirstA <= kMm - kSpanB && kLoadsA - kFirstA <= kMm, "at most one load behind an MFMA");
  static_assert(kRdEvery >= 1 && (kRd - 1) * kRdEvery < kMm, "every fragment is read inside its sub-step");
};

__device__ __forceinline__ uint32_t lds_addr32(const char* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)p));
}

// the same pointer, known to the compiler to be uniform
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u >> 32));
  return reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | lo);
}

// 16 bytes per lane, global -> LDS at (wave-uniform) lds + lane * 16; global address = scalar base + lane offset
__device__ __forceinline__ void direct_load_s(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds) : "memory");
}
// the same with a 64-bit address per lane
__device__ __forceinline__ void direct_load_v(const char* p, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(p), "s"(lds) : "memory");
}

// direct_load_s for lines that nothing reads again while the caches hold them
__device__ __forceinline__ void direct_load_once(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" : : "v"(off), "s"(base), "s"(lds) : "memory");
}

// from base + off: with 32-bit offsets the base stays scalar; operands whose panel spans 4 GiB or more take 64-bit ones
template <bool ONCE = false>
__device__ __forceinline__ void direct_load(const char* base, uint32_t off, uint32_t lds) {
  if (ONCE) direct_load_once(base, off, lds);
  else direct_load_s(base, off, lds);
}
template <bool ONCE = false>
__device__ __forceinline__ void direct_load(const char* base, uint64_t off, uint32_t lds) {
  static_assert(!ONCE, "few tokens of a vocabulary beyond 8.3 million: in whole tiles, by the usual loads");
  direct_load_v(base + off, lds);
}

#define ATG_PIN16() __builtin_amdgcn_sched_barrier(0)

// LDS-only workgroup barrier: waits for this wavefront's LDS operations, not for its outstanding global stores
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);   // vmcnt and expcnt at their maxima, lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
}

// s_waitcnt vmcnt(N) lgkmcnt(0)
template <int N>
__device__ __forceinline__ void wait_loads_but() {
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 0xF) | ((N >> 4) << 14));
}

// ---- operands --------------------------------------------------------------------------------------
// A panel in LDS is 32 KiB.  Operand contiguous along k: 256 rows of 128 bytes, the 16-byte chunk c of row r stored at
// chunk c ^ ((r >> 1) & 7).  k-major operand: 64 k-rows of 512 bytes, chunk c (of 32) of k-row k stored at
// (c & 16) | ((c ^ 2 s) & 15), s = (k & 3) | ((k >> 3) & 1) << 2.  Both make the fragment reads free of bank
// conflicts.  The swizzle is applied on the global side of the direct loads, whose LDS side is lane * 16.

// Off: uint32_t where 256 rows of the operand (64 k-rows of a k-major one) lie within 4 GiB, else uint64_t (see wide_rows)

// NL: direct loads of a wavefront per step (kLoadsA or kLoadsB of the grid); ONCE: nothing reads the panel again (direct_load_once)

// rows contiguous along k
template <int NL, typename Off = uint32_t, bool ONCE = false>
struct RowPanel {
  static constexpr bool kKMajor = false;
  const char* base;
  Off off[NL];
  // row_off(row): byte offset of tile row `row` from b
  template <typename F>
  __device__ __forceinline__ void init(const char* b, int wave, int lane, F row_off) {
    base = uniform_ptr(b);
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int row = (wave * NL + q) * 8 + (lane >> 3);
      off[q] = row_off(row) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
  }
  __device__ __forceinline__ void load(int q, uint32_t lds) { direct_load<ONCE>(base, off[q], lds); }
  __device__ __forceinline__ void advance() { base += kStepK * 2; }
};

// rows contiguous along k at arbitrary addresses (gathered rows)
template <int NL>
struct GatherPanel {
  static constexpr bool kKMajor = false;
  const char* p[NL];
  // the tile row that load q fetches for this lane
  static __device__ __forceinline__ int row(int q, int wave, int lane) { return (wave * NL + q) * 8 + (lane >> 3); }
  // row_ptr(q): address of tile row row(q)
  template <typename F>
  __device__ __forceinline__ void init(int wave, int lane, F row_ptr) {
#pragma unroll
    for (int q = 0; q < NL; ++q) p[q] = row_ptr(q) + (((lane & 7) ^ ((row(q, wave, lane) >> 1) & 7)) << 4);
  }
  __device__ __forceinline__ void load(int q, uint32_t lds) { direct_load_v(p[q], lds); }
  __device__ __forceinline__ void advance() {
#pragma unroll
    for (int q = 0; q < NL; ++q) p[q] += kStepK * 2;
  }
};

// k-major: k-row k at base + k * ld, 512 bytes of columns per row
template <int NL, typename Off = uint32_t>
struct KMajorPanel {
  static constexpr bool kKMajor = true;
  const char* base;
  Off off[NL];
  size_t step;
  // cmax: last 16-byte chunk (0..31) that may be read (chunks past it are fetched from it; the caller masks them)
  __device__ __forceinline__ void init(const char* b, int wave, int lane, size_t ld, int cmax) {
    base = uniform_ptr(b);
    step = ld * kStepK;
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int k = (wave * NL + q) * 2 + (lane >> 5);
      const int P = lane & 31, s = (k & 3) | (((k >> 3) & 1) << 2);
      const int C = (P & 16) | ((P ^ (2 * s)) & 15);
      off[q] = static_cast<Off>(k * ld) + min(C, cmax) * 16;
    }
  }
  __device__ __forceinline__ void load(int q, uint32_t lds) { direct_load(base, off[q], lds); }
  __device__ __forceinline__ void advance() { base += step; }
};

// k-major with a number of k-rows that need not be a multiple of 64: rows past the last are fetched from the last one (the
// other operand is zero there)
template <int NL, typename Off = uint32_t, bool ONCE = false>
struct KMajorTailPanel {
  static constexpr bool kKMajor = true;
  const char* base;
  Off off[NL];
  size_t ld;
  int rows, wave, lane, cmax;     // k-rows left from `base` on
  __device__ __forceinline__ void init(const char* b, int wave_, int lane_, size_t ld_, int cmax_, int rows_) {
    base = uniform_ptr(b);
    ld = ld_;
    rows = rows_;
    wave = wave_;
    lane = lane_;
    cmax = cmax_;
    offsets();
  }
  __device__ __forceinline__ void offsets() {
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int k = (wave * NL + q) * 2 + (lane >> 5);
      const int P = lane & 31, s = (k & 3) | (((k >> 3) & 1) << 2);
      const int C = (P & 16) | ((P ^ (2 * s)) & 15);
      off[q] = static_cast<Off>(max(min(k, rows - 1), 0) * ld) + min(C, cmax) * 16;
    }
  }
  __device__ __forceinline__ void load(int q, uint32_t lds) { direct_load<ONCE>(base, off[q], lds); }
  __device__ __forceinline__ void advance() {
    base += ld * kStepK;
    rows -= kStepK;
    if (rows < kStepK) offsets();
  }
};

// Transposing read: inside each group of 16 lanes, lane 4 r + q names 4 consecutive columns of row r, and lane i receives
// column i of the four rows.
__device__ __forceinline__ uint2 lds_read_tr(const char* p) {
  const bf16v4 v = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
      (__attribute__((address_space(3))) bf16v4*)(__attribute__((address_space(3))) const char*)p);
  return __builtin_bit_cast(uint2, v);
}

// Fragment reads of one operand: NB blocks of 16 rows starting at tile row `row0`.
template <int NB, bool KM>
struct FragReader;

template <int NB>
struct FragReader<NB, false> {
  int at[2], cur[2];
  __device__ __forceinline__ void init(int row0, int lane) {
    const int r = lane & 15;
    at[0] = (row0 + r) * (kStepK * 2) + ((((lane >> 4)) ^ ((r >> 1) & 7)) << 4);
    at[1] = at[0] ^ 64;                           // k + 32: chunk index ^ 4
  }
  __device__ __forceinline__ void slot(int byte) {
    cur[0] = at[0] + byte;
    cur[1] = at[1] + byte;
  }
  __device__ __forceinline__ uint4 read(const char* smem, int ks, int blk) const {
    return *reinterpret_cast<const uint4*>(smem + cur[ks] + blk * 16 * (kStepK * 2));
  }
};

template <int NB>
struct FragReader<NB, true> {
  int at[NB], cur[NB];
  __device__ __forceinline__ void init(int col0, int lane) {
    // 16 lanes read 4 k-rows x 16 columns: lane 4 r + q the 4 columns q of k-row r; lane i receives column i
    const int g = lane >> 4, r = (lane & 15) >> 2, q = lane & 3;
    const int k = 8 * g + r, s = (k & 3) | (((k >> 3) & 1) << 2);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int c = (col0 + b * 16) / 8 + (q >> 1);
      at[b] = k * (kTile16 * 2) + ((c & 16) | ((c ^ (2 * s)) & 15)) * 16 + (q & 1) * 8;
    }
  }
  __device__ __forceinline__ void slot(int byte) {
#pragma unroll
    for (int b = 0; b < NB; ++b) cur[b] = at[b] + byte;
  }
  __device__ __forceinline__ uint4 read(const char* smem, int ks, int blk) const {
    const char* p = smem + cur[blk] + ks * 32 * (kTile16 * 2);
    const uint2 lo = lds_read_tr(p), hi = lds_read_tr(p + 4 * (kTile16 * 2));
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
  }
};

// index of the MFMA after which load k of `cnt` is issued within one sub-step: evenly spread
__device__ __forceinline__ constexpr int load_after(int k, int cnt, int mm) { return ((2 * k + 1) * mm) / (2 * cnt); }
// the load issued after MFMA n, or -1
__device__ __forceinline__ constexpr int load_behind(int n, int cnt, int mm) {
  const int k = (2 * n * cnt + mm - 1) / (2 * mm);
  return k < cnt && load_after(k, cnt, mm) == n ? k : -1;
}

// acc += a b, with the accumulator tied to its registers: the builtin leaves the compiler free to give the result other
// registers than the addend, and with 256 accumulator registers per lane it then moves hundreds of them per k-step.  The
// compiler does not see the instruction's latency, so mfma_settle() has to stand between the last one and the first
// other use of an accumulator.  Between two MFMAs on one accumulator stand the kMm - 1 others of a sub-step: 19 and more on whole
// tiles (31 on those of 256 tokens), 15 and 7 on halves and quarters, of 16 cycles each, against the one whose result has to be there.
template <typename G>
__device__ __forceinline__ void mfma_in_place(floatx4& acc, bf16v8 a, bf16v8 b) {
  static_assert(G::kMm >= 8, "others between two MFMAs on one accumulator");
  if constexpr (G::kMm * 4 > 128)
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
  else
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
template <typename G>
__device__ __forceinline__ void mfma_settle(floatx4 (&acc)[G::kIB][G::kJB]) {
  asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
  for (int i = 0; i < G::kIB; ++i)
#pragma unroll
    for (int j = 0; j < G::kJB; ++j) {
      if constexpr (G::kMm * 4 > 128) asm volatile("" : "+a"(acc[i][j]));
      else asm volatile("" : "+v"(acc[i][j]));
    }
}

// LDS ring: three slots for the A panels and two for the B panels of consecutive k-steps: A of step kt in slot kt % 3, B in slot
// 3 + kt % 2.  What step kt leaves free at its barrier is requested again from there on, B of step kt+2 first: it has up to a whole
// step to land, A of step kt+3 up to two (the A panels are the weights, the B panels what more workgroups share).  With both
// operands taking turns in the five slots (A of step kt+2 requested in front of that barrier, B behind it) steps of 20000 rows took
// 27.8 ms at H = 2048 and 54.8 at H = 4096, now 26.1 and 51.8, and log-probabilities of 300 rows 235 -> 224 and 432 -> 405 us, of 8192
// rows 3670 -> 3560.  Where the launches go on for long, power is the bound and the gain smaller: 250000 rows 329 -> 325 ms,
// 37000 at H = 4096 on three heads 99.9 -> 98.4.  (Three slots for dW's B, the rows of dZ, instead: dW of 20000 rows 8.6 -> 9.0 ms.)
// Per k-step:
//   sub-step 0   MFMAs on the first 32 of k; fragments of the second 32; requests the other A loads of step kt+2
//   wait until all but those A loads have landed; workgroup barrier (one per k-step)
//   sub-step 1   MFMAs on the second 32; first fragments of step kt+1; requests B of step kt+2 and the first kFirstA loads of A of
//                step kt+3, into the slots that step kt has just left
// A slot is only overwritten after the barrier that follows its last read.
template <typename G, typename PA, typename PB>
struct Gemm16 {
  floatx4 (&acc)[G::kIB][G::kJB];
  PA& pa;
  PB& pb;
  const char* smem;
  uint32_t lds_a, lds_b;      // where this wavefront's part of a panel lies in the first slot of its operand
  FragReader<G::kIB, PA::kKMajor> ra;
  FragReader<G::kJB, PB::kKMajor> rb;
  uint4 fa[2][G::kIB], fb[2][G::kJB];
  int sa, sb;                 // byte offsets of the slots of the step being consumed

  __device__ __forceinline__ static int behind_a(int s) { return s == 2 * kRingSlot ? 0 : s + kRingSlot; }
  __device__ __forceinline__ static int behind_b(int s) { return s ^ kRingSlot; }
  __device__ __forceinline__ void mm(int f, int n) {
    const int i = n / G::kJB, j = n % G::kJB;
    mfma_in_place<G>(acc[i][j], __builtin_bit_cast(bf16v8, fa[f][i]), __builtin_bit_cast(bf16v8, fb[f][j]));
  }
  // fragment n of sub-step ks, in the order the MFMAs first need it: A block 0, the B blocks, the other A blocks
  __device__ __forceinline__ void rd(int ks, int f, int n) {
    if (n == 0) fa[f][0] = ra.read(smem, ks, 0);
    else if (n <= G::kJB) fb[f][n - 1] = rb.read(smem, ks, n - 1);
    else fa[f][n - G::kJB] = ra.read(smem, ks, n - G::kJB);
  }
  __device__ __forceinline__ void ld_a(int slot, int q) { pa.load(q, lds_a + slot + q * 1024); }
  __device__ __forceinline__ void ld_b(int slot, int q) { pb.load(q, lds_b + slot + q * 1024); }
  __device__ __forceinline__ void aim_reads(int a, int b) {
    ra.slot(a);
    rb.slot(kRingA + b);
  }

  // REQUEST: step kt+2 exists; MORE: step kt+3 does; NEXT: step kt+1 does
  template <bool REQUEST, bool MORE, bool NEXT>
  __device__ __forceinline__ void step() {
    constexpr int kMm = G::kMm, kRd = G::kRd, kEv = G::kRdEvery, kSpan = G::kSpanB;
    constexpr int kFirst = G::kFirstA, kSecond = G::kLoadsA - G::kFirstA, kRest = kMm > kSpan ? kMm - kSpan : 1;
    const int na = behind_a(sa), nb = behind_b(sb), nna = behind_a(na);
#pragma unroll
    for (int n = 0; n < kMm; ++n) {
      mm(0, n);
      ATG_PIN16();
      if (n % kEv == 0 && n / kEv < kRd) {
        rd(1, 1, n / kEv);
        ATG_PIN16();
      }
      if (REQUEST && load_behind(n, kSecond, kMm) >= 0) {
        ld_a(nna, kFirst + load_behind(n, kSecond, kMm));
        ATG_PIN16();
      }
    }
    if (REQUEST) {
      pa.advance();
      wait_loads_but<G::kLoadsA>();
    } else {
      wait_loads_but<0>();
    }
    __builtin_amdgcn_s_barrier();
    ATG_PIN16();
    if (NEXT) aim_reads(na, nb);
#pragma unroll
    for (int n = 0; n < kMm; ++n) {
      mm(1, n);
      ATG_PIN16();
      if (NEXT && n % kEv == 0 && n / kEv < kRd) {
        rd(0, 0, n / kEv);
        ATG_PIN16();
      }
      if (REQUEST && n < kSpan && load_behind(n, G::kLoadsB, kSpan) >= 0) {
        ld_b(sb, load_behind(n, G::kLoadsB, kSpan));
        ATG_PIN16();
      }
      if (MORE && kFirst > 0 && n >= kSpan && load_behind(n - kSpan, kFirst, kRest) >= 0) {
        ld_a(sa, load_behind(n - kSpan, kFirst, kRest));
        ATG_PIN16();
      }
    }
    if (REQUEST) pb.advance();
    sa = na;
    sb = nb;
  }

  __device__ __forceinline__ void request_step(int a, int b) {
#pragma unroll
    for (int q = 0; q < G::kLoadsA; ++q) ld_a(a, q);
    pa.advance();
#pragma unroll
    for (int q = 0; q < G::kLoadsB; ++q) ld_b(b, q);
    pb.advance();
  }

  // Requests the first two of nk steps, into all slots but kRingFree.  The last reads of a tile's panels lie in front of its final
  // step's barrier, so the next tile's may be requested as soon as run() is through: they travel while the results leave.
  __device__ __forceinline__ void begin(int nk) {
    if (nk > 0) request_step(0, 0);
    if (nk > 1) request_step(kRingSlot, kRingSlot);
  }

  // acc = A B^T over nk >= 0 steps, of which begin() has requested the first two.  Every thread of the workgroup calls it.
  // fetch(0) and fetch(1) stand in front of the last step but one and the last: what a caller loads there costs no registers
  // in the loop and no wait behind it.
  template <typename F>
  __device__ __forceinline__ void run(int nk, F fetch) {
#pragma unroll
    for (int i = 0; i < G::kIB; ++i)
#pragma unroll
      for (int j = 0; j < G::kJB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
    if (nk > 1) wait_loads_but<G::kLoadsA + G::kLoadsB>();
    else wait_loads_but<0>();
    __builtin_amdgcn_s_barrier();
    sa = sb = 0;
    aim_reads(0, 0);
#pragma unroll
    for (int n = 0; n < G::kRd; ++n) rd(0, 0, n);
    if (nk > 2) {
#pragma unroll
      for (int q = 0; q < G::kFirstA; ++q) ld_a(kRingFree, q);
    }
    int kt = 0;
    for (; kt + 3 < nk; ++kt) step<true, true, true>();
    if (kt + 2 < nk) {
      step<true, false, true>();
      ++kt;
    }
    fetch(0);
    if (kt + 1 < nk) step<false, false, true>();
    fetch(1);
    if (nk > 0) step<false, false, false>();
    mfma_settle<G>(acc);
  }
};

// The thread's coordinates, recomputed where they are needed: what the compiler derives from an opaque thread index cannot
// be hoisted out of the loop over tiles, where it would occupy registers through the k loop and be spilled.
template <typename G>
struct Coord16 {
  int lane, wave, wm, wn;
  __device__ __forceinline__ Coord16() {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    wm = wave / G::kWavesB;
    wn = wave % G::kWavesB;
  }
  __device__ __forceinline__ int a_row(int i) const { return wm * G::kRowsA + i * 16 + 4 * (lane >> 4); }   // + r
  __device__ __forceinline__ int b_row(int j) const { return wn * G::kRowsB + j * 16 + (lane & 15); }
};

template <typename G, typename PA, typename PB>
__device__ __forceinline__ Gemm16<G, PA, PB> make_gemm16(floatx4 (&acc)[G::kIB][G::kJB], PA& pa, PB& pb, char* smem,
                                                         const Coord16<G>& co) {
  const uint32_t lds = lds_addr32(smem);
  Gemm16<G, PA, PB> g{acc, pa, pb, smem, static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(lds + co.wave * G::kLoadsA * 1024)),
                      static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(lds + kRingA + co.wave * G::kLoadsB * 1024)), {}, {}, {}, {}, 0, 0};
  g.ra.init(co.wm * G::kRowsA, co.lane);
  g.rb.init(co.wn * G::kRowsB, co.lane);
  return g;
}

// one tile on its own: acc = A B^T over nk steps of 64 (nk may be 0)
template <typename G, typename PA, typename PB>
__device__ __forceinline__ void gemm16(floatx4 (&acc)[G::kIB][G::kJB], PA& pa, PB& pb, int nk, char* smem,
                                       const Coord16<G>& co) {
  auto g = make_gemm16<G>(acc, pa, pb, smem, co);
  g.begin(nk);
  g.run(nk, [](int) {});
}

}  // namespace atg

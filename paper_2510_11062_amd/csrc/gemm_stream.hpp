// Contraction of bf16 operands as a stream of k-steps (gfx950), for tiles with little arithmetic per byte.
//
// Same operands, swizzles, fragments and accumulators as gemm_bf16.hpp, another ring: D slots that hold both panels of one
// k-step of a TA x TB tile each, one barrier per step, and D - 1 steps in flight.  Steps follow one another across
// tiles: the loads run D - 1 steps ahead of the arithmetic whatever tile they belong to, so that memory is never left alone
// at the end of a tile.  Step s:
//   MFMAs on its first half, fragments of its second half
//   wait until step s + 1 has landed; barrier: every wavefront has read what it needs of step s
//   MFMAs on its second half; first fragments of step s + 1; requests step s + D into the slot that step s leaves
// There is no branch around an MFMA: behind its last step a stream goes on requesting (next_panels() says what), so that the
// counts of loads in flight are constants, and finish() waits for what was requested in vain.
#pragma once

#include "gemm_bf16.hpp"

namespace atg {

template <typename G, typename PA, typename PB, int D>
struct Stream16 {
  static_assert(!PA::kKMajor && !PB::kKMajor, "rows along k");
  static_assert(D >= 3, "the step in front of the one being consumed has landed, at least one more is under way");
  static constexpr int kPanelA = G::kTileA * kStepK * 2, kSlot = (G::kTileA + G::kTileB) * kStepK * 2, kBytes = D * kSlot;
  static constexpr int kLa = G::kLoadsA, kLb = G::kLoadsB, kL = kLa + kLb;
  static_assert((D - 1) * kL < 64, "the counter of loads in flight");

  floatx4 (&acc)[G::kIB][G::kJB];
  PA& pa;
  PB& pb;
  const char* smem;
  uint32_t lds;               // of the ring
  uint32_t wave_a, wave_b;    // where this wavefront's part of a panel lies
  int slot, fill;             // byte offsets of the slots of the step consumed and of the one requested next
  FragReader<G::kIB, false> ra;
  FragReader<G::kJB, false> rb;
  uint4 fa[2][G::kIB], fb[2][G::kJB];

  __device__ __forceinline__ Stream16(floatx4 (&acc_)[G::kIB][G::kJB], PA& pa_, PB& pb_, char* smem_, const Coord16<G>& co)
      : acc(acc_), pa(pa_), pb(pb_), smem(smem_) {
    lds = lds_addr32(smem_);
    wave_a = __builtin_amdgcn_readfirstlane(co.wave * kLa * 1024);
    wave_b = __builtin_amdgcn_readfirstlane(kPanelA + co.wave * kLb * 1024);
    ra.init(co.wm * G::kRowsA, co.lane);
    rb.init(co.wn * G::kRowsB, co.lane);
  }

  __device__ __forceinline__ static int behind(int s) { return s + kSlot == kBytes ? 0 : s + kSlot; }
  __device__ __forceinline__ void mm(int f, int n) {
    const int i = n / G::kJB, j = n % G::kJB;
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16v8, fa[f][i]), __builtin_bit_cast(bf16v8, fb[f][j]),
                                                        acc[i][j], 0, 0, 0);
  }
  __device__ __forceinline__ void rd(int ks, int f, int n) {
    if (n == 0) fa[f][0] = ra.read(smem, ks, 0);
    else if (n <= G::kJB) fb[f][n - 1] = rb.read(smem, ks, n - 1);
    else fa[f][n - G::kJB] = ra.read(smem, ks, n - G::kJB);
  }
  __device__ __forceinline__ void aim_reads(int s) {
    ra.slot(s);
    rb.slot(s + kPanelA);
  }
  __device__ __forceinline__ void load(int k) {
    if (k < kLa) pa.load(k, lds + fill + wave_a + k * 1024);
    else pb.load(k - kLa, lds + fill + wave_b + (k - kLa) * 1024);
  }
  // behind the loads of a step
  __device__ __forceinline__ void requested() {
    pa.advance();
    pb.advance();
    fill = behind(fill);
  }
  // MFMAs on fragment set f; reads of the fragments of half ks into set 1 - f; the loads of a step with LOAD
  template <bool LOAD>
  __device__ __forceinline__ void half(int f, int ks) {
#pragma unroll
    for (int n = 0; n < G::kMm; ++n) {
      mm(f, n);
      ATG_PIN16();
      if (n % G::kRdEvery == 0 && n / G::kRdEvery < G::kRd) {
        rd(ks, 1 - f, n / G::kRdEvery);
        ATG_PIN16();
      }
      if (LOAD) {
#pragma unroll
        for (int k = 0; k < kL; ++k)
          if (load_after(k, kL, G::kMm) == n) {
            load(k);
            ATG_PIN16();
          }
      }
    }
  }

  // Starts a stream, the panels aimed at its first step.  No wavefront may still need the ring.
  // next_panels(): called in front of every request but the first, aims the panels anew where a tile ends.
  template <typename Next>
  __device__ __forceinline__ void begin(Next next_panels) {
    slot = fill = 0;
#pragma unroll 1
    for (int i = 0; i < D; ++i) {
      if (i > 0) next_panels();
#pragma unroll
      for (int k = 0; k < kL; ++k) load(k);
      requested();
    }
    wait_loads_but<(D - 1) * kL>();
    __builtin_amdgcn_s_barrier();
    ATG_PIN16();
    aim_reads(0);
#pragma unroll
    for (int n = 0; n < G::kRd; ++n) rd(0, 0, n);
  }

  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < G::kIB; ++i)
#pragma unroll
      for (int j = 0; j < G::kJB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
  }

  template <typename Next>
  __device__ __forceinline__ void step(Next next_panels) {
    half<false>(0, 1);
    wait_loads_but<(D - 2) * kL>();
    __builtin_amdgcn_s_barrier();
    ATG_PIN16();
    slot = behind(slot);
    aim_reads(slot);
    next_panels();
    half<true>(1, 0);
    requested();
  }

  // Every load into LDS has landed: LDS may be used for something else, or be given back.
  __device__ __forceinline__ void finish() {
    wait_loads_but<0>();
    __builtin_amdgcn_s_barrier();
  }
};

}  // namespace atg

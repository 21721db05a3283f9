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

template <typename K>
int allow_big_lds(K kernel, int bytes) {
  ATG_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
  return AT_GRPO_OK;
}

// persistent grid: one workgroup per compute unit
inline int gemm_grid() {
  const int cus = device_cu_count();
  return cus > 0 ? cus : 256;
}

}  // namespace atg

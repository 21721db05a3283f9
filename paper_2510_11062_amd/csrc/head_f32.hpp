// Launchers of the fp32 head contractions (see head_kernels.hpp for the meaning of the arguments).
#pragma once

#include "head_kernels.hpp"

namespace atg {

constexpr int kVocabTileF32 = 64;    // vocabulary rows per partial of the log-probability kernel
// room for the parts of contractions split along k
size_t partial_bytes_f32(const HeadGeom& g);

int launch_fwd_f32(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                   float* part_m, float* part_s, float* part_u, float* zy, hipStream_t s);
int launch_lse_combine_f32(const HeadGeom& g, const HeadChunk& ch, const float* part_m, const float* part_s, const float* part_u,
                           const float* zy, float* logp, float* lse, float* entropy, hipStream_t s);
int launch_dz_f32(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                  const float* lse, const float* coef, void* dZ, void* clear, int64_t clear_bytes, hipStream_t s);
// dHidden and dW
int launch_grads_f32(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* W, const void* hidden, void* d_hidden,
                     float* dW, void* part, int accumulate, int first_chunk, hipStream_t s);

}  // namespace atg

// Launchers of the bf16 head contractions (see head_kernels.hpp for the meaning of the arguments).  `part`: room for
// the partial tiles of a split contraction, head_partial_bytes() of it.
#pragma once

#include "head_kernels.hpp"

namespace atg {

int launch_fwd_bf16(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                    float* part_m, float* part_s, float* part_u, float* zy, hipStream_t s, const int32_t* gate);
int launch_fe_bf16(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                   const float* c2, void* E, float* part_s, float* zy, hipStream_t s);
int launch_dz_bf16(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W, const int32_t* token_id,
                   const float* lse, const float* coef, void* dZ, hipStream_t s, const int32_t* gate);
// do logits launches of few tokens follow narrow_launch()?
bool narrow_launches_bf16(const HeadGeom& g);
// Wt = W transposed, unless the head's list is short enough for dHidden to read W itself (then Wt is not touched; with
// transposes_w_bf16(rows of the batch) == false no list can be long enough and Wt may be null everywhere).
bool transposes_w_bf16(int64_t n_tok);
int launch_transpose_w_bf16(const HeadGeom& g, const void* W, void* Wt, const int32_t* cnt, hipStream_t s);
int launch_dh_bf16(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* W, const void* Wt, void* d_hidden,
                   void* part, hipStream_t s, const float* scale, const int32_t* perm, const int32_t* live_cnt);
int launch_dw_bf16(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* hG, float* dW, void* part,
                   int accumulate, int first_chunk, hipStream_t s, const int32_t* live_cnt);

}  // namespace atg

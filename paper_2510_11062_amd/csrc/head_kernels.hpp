// Launchers of the LM-head kernels: forward contraction with online-softmax partials, the
// partial combine, and the three backward contractions.  All take device-side token counts, so
// no launch depends on a host read-back.
#pragma once

#include "common.hpp"

namespace atg {

// Geometry of one head pass over a super-chunk of at most TC compacted tokens.
struct HeadGeom {
  int dtype;        // at_grpo_dtype
  int H, V;
  int Vp;           // V rounded up to 64 (k padding of the dZ / W^T buffers)
  int TC;           // tokens per super-chunk (multiple of 256)
  int vtile;        // vocabulary rows per partial of the log-probability kernels
  int n_vtiles;     // ceil(V / vtile)
  int esize;        // bytes per element of hidden / W / dZ
};

struct HeadChunk {
  const int32_t* idx;   // compacted token rows of this head (device), whole list
  const int32_t* cnt;   // number of entries in idx (device scalar)
  int32_t c0;           // first list position of this super-chunk
};

// part_m / part_s: per-(vocabulary tile, token) running max (log2 domain) and sum, [n_vtiles][TC], in bf16 launches of few
// tokens [ceil(V / kNarrowV)][kNarrowStride] (see narrow_launch; logit_part_floats() is room for both); zy: [TC] target
// logit.  hidden / W are the caller's tensors.
// part_u: null, or partial sums for the entropy monitor, laid out the same (selects the kernel variant).
int launch_head_fwd(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W,
                    const int32_t* token_id, float* part_m, float* part_s, float* part_u, float* zy,
                    hipStream_t s, const int32_t* gate = nullptr);

// logp[row], lse[row] for the rows of this super-chunk (lse may be null).
// With part_u, also entropy[row] = lse - E_p[z].  bf16 with `scale` (and ca): also scale[j] = -g_j, the factor of rows whose E
// becomes softmax - onehot.
struct CoefArgs;
int launch_lse_combine(const HeadGeom& g, const HeadChunk& ch, const float* part_m,
                       const float* part_s, const float* part_u, const float* zy, float* logp,
                       float* lse, float* entropy, hipStream_t s, const int32_t* gate = nullptr, int head = 0,
                       const CoefArgs* ca = nullptr, float* scale = nullptr);

// bf16: Wt[H][Vp] = W[V][H]^T, zero in the k padding.  A head with few rows (*cnt of its list) is left untransposed, and
// needs_transposed_w() == false for a batch of n_tok rows says that no copy is ever read (Wt may then be null).
bool needs_transposed_w(const HeadGeom& g, int64_t n_tok);
int launch_transpose_w(const HeadGeom& g, const void* W, void* Wt, const int32_t* cnt, hipStream_t s);

// vocabulary rows per partial (HeadGeom::vtile)
int head_vocab_tile(int dtype);

// bf16 (fp32 reads the rows where they lie; hG is null and nothing happens): hG[TC][H] = the gathered hidden rows of this
// super-chunk, zero rows up to the next multiple of 256.  With `scale`, row j is multiplied by scale[j] (j counted from the
// start of the super-chunk).  With `perm`, row j is list position perm[j] (and its factor), for j < *live_cnt; zero rows
// behind.
int launch_gather_hidden(const HeadGeom& g, const HeadChunk& ch, const void* hidden,
                         void* hG, hipStream_t s, const float* scale = nullptr,
                         const int32_t* perm = nullptr, const int32_t* live_cnt = nullptr,
                         void* E = nullptr);

// dZ[TC][Vp] for this super-chunk (element type of hidden).  fp32: the launch also sets clear_bytes (a multiple of 16) of
// `clear` to zero, whatever the list holds.
int launch_head_dz(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W,
                   const int32_t* token_id, const float* lse, const float* coef, void* dZ,
                   hipStream_t s, const int32_t* gate = nullptr, void* clear = nullptr, int64_t clear_bytes = 0);

// Scratch for the partial tiles of launch_head_dh / launch_head_dw over g.TC rows.
size_t head_partial_bytes(const HeadGeom& g);

// ---- forward and backward from one pass over the logits (bf16) ---------------------------------------
// A `gate` argument of the launchers above and below is a device word: with a non-null gate the kernel
// returns at once while the word is 0 (coef == null in launch_head_dz: dZ = softmax - onehot).

// c2[j] = log2(e) * z[j][y_j], the reference of the exponentials, for the tokens of the launch.
int launch_ref_logit(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W,
                     const int32_t* token_id, float* c2, hipStream_t s);

// E[j][v] = exp(z[j][v] - c_j) (bf16, [TC][Vp]); part_s partial row sums, laid out as above; zy[TC] target logit.
int launch_head_fe(const HeadGeom& g, const HeadChunk& ch, const void* hidden, const void* W,
                   const int32_t* token_id, const float* c2, void* E, float* part_s, float* zy, hipStream_t s);

// logp / lse of the rows; scale[j] = -g_j / S_j; E[j][y_j] = e_y - S_j; raises *gate when a row's sum is
// out of range (that row gets scale 0), unless the row has no advantage: it then goes to later[(*n_later)++], in any order.
int launch_fe_combine(const HeadGeom& g, const HeadChunk& ch, int head, const float* part_s, const float* c2,
                      const float* zy, const int32_t* token_id, const CoefArgs& ca, float* logp, float* lse,
                      float* scale, void* E, int32_t* gate, int32_t* later, int32_t* n_later, hipStream_t s);

// bf16: d_hidden[row] = dZ[j] . W for the rows of this super-chunk.
// With `scale`, row j of the result is multiplied by scale[j] (j counted from ch.c0).  With `perm` (after
// launch_compact_rows), the first *live_cnt rows of dZ are contracted and row j goes to list position perm[j].
// `part`: head_partial_bytes() of scratch (partial results of contractions split along k).
int launch_head_dh(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* W, const void* Wt,
                   void* d_hidden, void* part, hipStream_t s, const float* scale = nullptr, const int32_t* perm = nullptr,
                   const int32_t* live_cnt = nullptr);

// Takes the rows with scale[j] == 0 out of a super-chunk of E (bf16, TC <= 32768): rows from the tail are
// copied into their places, so that rows 0 .. *live_cnt - 1 all have a non-zero factor; perm[j] = the list
// position (counted from ch.c0) whose row now sits at j.  holes / movers: scratch of TC entries each;
// *pair_cnt = rows moved.  Deterministic.
int launch_compact_rows(const HeadGeom& g, const HeadChunk& ch, const float* scale, void* E, int32_t* perm,
                        int32_t* holes, int32_t* movers, int32_t* live_cnt, int32_t* pair_cnt, hipStream_t s);

// bf16: dW[V][H] (+)= dZ^T . hidden rows.  first_chunk: runs even for an empty list so that dW is defined.
// With `live_cnt`: only the first *live_cnt rows of the chunk are contracted.
int launch_head_dw(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* hG, float* dW, void* part, int accumulate, int first_chunk, hipStream_t s, const int32_t* live_cnt = nullptr);

// fp32: both of them, in one launch.
int launch_head_grads(const HeadGeom& g, const HeadChunk& ch, const void* dZ, const void* W, const void* hidden, void* d_hidden,
                      float* dW, void* part, int accumulate, int first_chunk, hipStream_t s);

}  // namespace atg

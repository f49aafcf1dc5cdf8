// The encoder layer of modules.py in float32 as runs of kernel launches: what _native.so calls instead of one library
// product, copy or layer at a time.  All pointers are device pointers, all tensors contiguous.
#pragma once

#include <stdint.h>

#include "../../include/tempo.h"

#ifdef __cplusplus
extern "C" {
#endif

// tokens T = batch * seq; heads of d = hidden / heads columns.
typedef struct {
  int64_t batch, seq, hidden, heads, ffn;
  float eps1, eps2, p;
  uint64_t seed, offset;
  tempo_gelu_kind kind;
  const float *wqkv, *bqkv, *wproj, *bproj, *w1, *b1, *w2, *b2;  // Linear: [out, in] and [out]
  const float *gamma1, *beta1, *gamma2, *beta2;
  const float* x;          // [T, hidden]; in the backward null, as all else, where the gradients wanted do not need it
  const int32_t* key_len;  // [batch] or null
  // written by the forward, read by the backward
  float *qkv, *probs, *ctxt, *y1, *rstd1, *h, *y2, *rstd2;
  uint32_t *keep, *side;   // keep bits [batch, heads, seq, seq] (null in the backward: drawn again); GELU's mask [T, ffn]
} tempo_encoder;

// Whether the products of a layer of this size are faster as these kernels than as library calls.
TEMPO_API int tempo_encoder_takes(const tempo_encoder* e);

// out: scratch as large as probs.
TEMPO_API tempo_status tempo_encoder_fwd(const tempo_encoder* e, float* out, void* hip_stream);

// The gradients of a layer; null: not computed.  Those of a LayerNorm are written together.
typedef struct {
  float *dx, *dwqkv, *dbqkv, *dwproj, *dbproj, *dw1, *db1, *dw2, *db2;
  float *dgamma1, *dbeta1, *dgamma2, *dbeta2;
} tempo_encoder_grads;

// From dy to the gradient of the second LayerNorm's input, ds2, and to that of the first one's output, dy1 (both
// [T, hidden]; dy1 null: not computed).  dh: scratch [T, ffn].
TEMPO_API tempo_status tempo_encoder_bwd_ffn(const tempo_encoder* e, const tempo_encoder_grads* g, const float* dy,
                                             float* ds2, float* dh, float* dy1, void* workspace, size_t workspace_bytes,
                                             void* hip_stream);
// From dy1 to the gradient of the first LayerNorm's input, ds1; [T, hidden].
TEMPO_API tempo_status tempo_encoder_bwd_norm(const tempo_encoder* e, const tempo_encoder_grads* g, const float* dy1,
                                              float* ds1, void* workspace, size_t workspace_bytes, void* hip_stream);
// From ds1 to the gradients of the attention block and dx.  dctxt [T, hidden], dqkv [T, 3 hidden], dout and out as
// large as probs: scratch (dctxt null: only the output projection's).
TEMPO_API tempo_status tempo_encoder_bwd_attention(const tempo_encoder* e, const tempo_encoder_grads* g,
                                                   const float* ds1, float* dctxt, float* dqkv, float* dout, float* out,
                                                   void* hip_stream);

#ifdef __cplusplus
}
#endif

// Host-side entry points shared between the translation units of libdetinfer (not exported).
#pragma once

#include "common.h"

namespace det {

// det_attn_decode with the sequence length taken as seqlens[b] + len_offset (the decoder layer
// passes its `positions` array with len_offset = 1: the new token sits at row positions[b]).
// slots: cache slot of each row (nullptr: row b uses slot b).
// qscales: nullptr for the bf16 output [B, Hq*D]; else `out` receives the int8 codes and qscales the
// scales of the output's 8-bit block quantization, as det_quant_act_q8 lays them out for (B, Hq*D).
int attn_decode_impl(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens,
                     const int32_t* slots, int len_offset, void* out, void* ws, size_t ws_bytes, int B, int Hq, int Hkv, int D,
                     int Lmax, float scale, hipStream_t s, void* qscales = nullptr);

// The same on rows that name their slots (attn_rows.hip): arguments checked by the caller.  ws_o: the chunk outputs of the
// workspace, [R, Hq, ncmax, D].  attn_walk_workgroups: the (row tile, KV head) workgroups such a launch has.
long long attn_walk_workgroups(int R, int G, int Hkv);
int attn_walk(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens, const int32_t* slots,
              int len_offset, void* out, float* qscales, float* ws_o, int R, int Hq, int Hkv, int Lmax, int ncmax, float scale,
              hipStream_t s);

// SwiGLU projection with quantized output (qgemm.hip), where it fits: aligned buffers as the layer lays them out.
bool qgemm_swiglu_quant_fits(int M, int F, int K);
int qgemm_swiglu_quant(const void* codes, const void* scales, const void* packed_gate_up, void* codes_out, void* scales_out, int M,
                       int F, int K, void* stream);

// RMSNorm, quantization and projection of raw rows x [M, K] in one launch (qgemm.hip), where it fits (N columns).
bool qgemm_norm_fits(int M, int N, int K);
int qgemm_norm_qkv_rope_append(const void* x, const void* w_norm, float eps, const void* packed_qkv, void* qbuf, void* kcache,
                               void* vcache, const int32_t* positions, const int32_t* slots, const float* rope_cos,
                               const float* rope_sin, int M, int Hq, int Hkv, int D, int Lmax, int K, void* stream);
bool qgemm_norm_swiglu_quant_fits(int M, int F, int K);
int qgemm_norm_swiglu_quant(const void* x, const void* w_norm, float eps, const void* packed_gate_up, void* codes_out,
                            void* scales_out, int M, int F, int K, void* stream);
int qgemm_norm_swiglu(const void* x, const void* w_norm, float eps, const void* packed_gate_up, void* Y, int ldy, int M, int F, int K,
                      void* stream);

}  // namespace det

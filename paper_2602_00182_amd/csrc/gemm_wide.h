// The wide-tile form of the bf16 GEMM (gemm_wide.hip), chosen by gemm.hip.
#pragma once

#include "common.h"

namespace det {

struct gemm_wide_args {
    const void* A;
    int lda;
    const void* Bp;
    int cb;  // column blocks per slab of the packing
    void* C;
    int ldc;
    const void* R;
    int ldr;
    int M, N, K;
    int out_f32;
    gemm_rope_args ra;
};

// Row blocks a wave should have (a tile is 32 times as many rows high), 0 where the other tiles are the better ones.
int gemm_wide_rows(int M, int N, int K, int cb);
int gemm_wide(int epi, int rbw, const gemm_wide_args& a, hipStream_t s);

}  // namespace det

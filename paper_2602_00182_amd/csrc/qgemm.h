// Shared by the forms of the block-quantized GEMM (qgemm.hip, qgemm_few.hip, qgemm_mid.hip).
#pragma once

#include "common.h"
#include "geometry.h"

namespace det {

typedef int v4i __attribute__((ext_vector_type(4)));

// The codes q of a column block's 64 k, stored as q + 8, two a byte, become 16*q as signed bytes (the nibble in the upper half
// of a byte, its top bit flipped), and the matrix core sums 16*p*q from the bits of 786432, a float whose last place is worth
// 1/16: read as a float the sum is 786432 + P, exactly (|P| <= 64 * 128 * 8), and one subtraction gives P.  Neither the +8 (which
// took a matrix instruction more for every row block, or six vector instructions more a column block) nor the conversion to
// floating point, which issues at half the rate of a subtraction, costs anything of its own.  us before and after: 1962 rows
// 2048 x 11264 113 -> 102, 5632 x 2048 58 -> 52, 14336 x 4096 266 -> 245, 4096 x 28672 521 -> 465; 24 rows of 4096 x 28672
// 22.7 -> 20.6, 128 rows of 14336 x 4096 77 -> 73, one row of 4096 x 28672 16.2 -> 15.2.
constexpr v4i kProductStart = {0x49400000, 0x49400000, 0x49400000, 0x49400000};
__device__ __forceinline__ float product(int sum) { return __int_as_float(sum) - 786432.0f; }
__device__ __forceinline__ v4i code_bytes(const uint2& c)
{
    auto hi = [](uint32_t x) { return (int)((x & 0xF0F0F0F0u) ^ 0x80808080u); };
    return v4i{hi(c.x << 4), hi(c.x), hi(c.y << 4), hi(c.y)};
}

// Counters in LDS by which the waves of a workgroup tell each other what is done.  LDS serves a wave's instructions in order.
// Written as instructions: a volatile access of the C language goes by way of flat addresses, whose wait takes in every load under
// way (14336 x 4096 with it and without, us: qgemm_mid.hip, 8 rows, 22.4 and 14.1; qgemm_few.hip, one row, 11.2 and 10.9).
__device__ __forceinline__ uint32_t lds_address(const int* p) { return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) int*)p; }
__device__ __forceinline__ void publish(int* counter, int value)
{
    if ((threadIdx.x & 63) == 0) asm volatile("ds_write_b32 %0, %1" ::"v"(lds_address(counter)), "v"(value) : "memory");
}
__device__ __forceinline__ int lds_look(const int* counter)
{
    int v;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(lds_address(counter)) : "memory");
    return v;
}
// Waits until lane i < n finds counters[i] at its `need` or above.
__device__ __forceinline__ void await(const int* counters, int n, int need)
{
    const int lane = threadIdx.x & 63;
    for (;;) {
        const int have = lds_look(&counters[lane < n ? lane : 0]);
        if (__ballot(lane < n && have < need) == 0) break;
        __builtin_amdgcn_s_sleep(1);
    }
}

// Epilogues for waves that read what they need besides the sums before these are there: kEpiResidual from the residual's four
// values, kEpiRopeAppend from the pairs' cosines and sines.  The same operations as gemm_epilogue_store and
// gemm_epilogue_rope_append, which stay in one piece: made of these parts they compile to other code for the kernels that read at
// the end (the wide bf16 tiles 7 % more instructions).  us whole and cut up: one row of 4096 x 4096 with the residual 7.89 and 8.01 on one card, level
// on others, 55 rows of 5632 x 2048 10.16 and 9.97; with the rotation 55 rows of hidden 4096 14.6 and 14.8, 128 rows 19.8 and 19.4, of hidden 2048 9.33
// and 9.56; else level.
__device__ __forceinline__ uint2 gemm_residual(const float (&v)[4], const uint2& rv)
{
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = bf16_to_f32(f32_to_bf16_rne(v[e]));
    y[0] = y[0] + bf16lo_to_f32(rv.x);
    y[1] = y[1] + bf16hi_to_f32(rv.x);
    y[2] = y[2] + bf16lo_to_f32(rv.y);
    y[3] = y[3] + bf16hi_to_f32(rv.y);
    return make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
}

struct rope_factors {
    float2 c, s;
};
__device__ __forceinline__ rope_factors gemm_rope_factors(const gemm_rope_args& ra, int p, int n)
{
    rope_factors f{make_float2(0.f, 0.f), make_float2(0.f, 0.f)};
    if ((n >> 7) < ra.Hq + ra.Hkv) {  // value heads are copied
        const size_t at = (size_t)p * 64 + ((n & 127) >> 1);
        f.c = *reinterpret_cast<const float2*>(ra.cos_t + at);
        f.s = *reinterpret_cast<const float2*>(ra.sin_t + at);
    }
    return f;
}
__device__ __forceinline__ void gemm_rope_append(const float (&v)[4], const gemm_rope_args& ra, size_t row, int p, int slot, int n,
                                                 const rope_factors& f)
{
    constexpr int D = 128, half = 64;
    const int head = n >> 7, i0 = (n & (D - 1)) >> 1;
    uint16_t x[4], lo0, hi0, lo1, hi1;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = f32_to_bf16_rne(v[e]);
    uint16_t* dst;
    if (head < ra.Hq + ra.Hkv) {
        rope_pair(x[0], x[1], f.c.x, f.s.x, lo0, hi0);
        rope_pair(x[2], x[3], f.c.y, f.s.y, lo1, hi1);
        dst = head < ra.Hq ? ra.qbuf + (row * ra.Hq + head) * D
                           : ra.kcache + (((size_t)slot * ra.Hkv + (head - ra.Hq)) * ra.Lmax + p) * D;
    } else {
        lo0 = x[0], hi0 = x[1], lo1 = x[2], hi1 = x[3];
        dst = ra.vcache + (((size_t)slot * ra.Hkv + (head - ra.Hq - ra.Hkv)) * ra.Lmax + p) * D;
    }
    *reinterpret_cast<uint32_t*>(dst + i0) = lo0 | ((uint32_t)lo1 << 16);
    *reinterpret_cast<uint32_t*>(dst + half + i0) = hi0 | ((uint32_t)hi1 << 16);
}

// Bytes of a stage (64 k) of a packed slab of 16*cb columns: codes, then scales.
__host__ __device__ constexpr int qstage_w_bytes(int cb) { return 544 * cb; }

// Launches of a few rows (qgemm_few.hip).  x != nullptr: the rows are raw activations [M, K] (bf16), which the kernel normalizes
// (RMSNorm with w_norm, eps) and quantizes itself (kEpiSwiglu and kEpiRopeAppend only); codes and scales are then not used.
struct qgemm_few_args {
    const void *codes, *scales, *wp;
    void* C;
    int ldc;
    const void* R;
    int ldr, M, N, K, out_f32;
    gemm_rope_args ra;
    const void *x, *w_norm;
    float eps;
};
constexpr int kFewRows = DET_QGEMM_FEW_ROWS;
bool qgemm_few_fits(int M, int cb, int K, bool norm);
void qgemm_few(int epi, int cb, const qgemm_few_args& a, hipStream_t s);
// Launches of more, in tiles of at most 48 rows (qgemm_mid.hip); x is not taken.
bool qgemm_mid_fits(int M, int cb, int rows);
void qgemm_mid(int epi, int cb, const qgemm_few_args& a, int rows, hipStream_t s);

}  // namespace det

// What the attention kernels do between the lanes of a wave: a lane holds scores of the pair (row, head) lane % 16, so the
// four lanes lr, lr + 16, lr + 32, lr + 48 share a pair.
#pragma once

#include "common.h"

namespace det {

typedef short short4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t fbits(float v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ float bitsf(uint32_t v) { return __builtin_bit_cast(float, v); }

// the value of a variable that is the same in every lane, for the scalar unit
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Rows of sixteen lanes 0..3.  add32(a, b): rows 0, 1 get a[row] + a[row+2], rows 2, 3 get b[row-2] + b[row].
// add16(a, b): rows 0, 2 get a[row] + a[row+1], rows 1, 3 get b[row-1] + b[row].
__device__ __forceinline__ float add32(float a, float b)
{
    const uint2v r = __builtin_amdgcn_permlane32_swap(fbits(a), fbits(b), false, false);
    return bitsf(r[0]) + bitsf(r[1]);
}
__device__ __forceinline__ float add16(float a, float b)
{
    const uint2v r = __builtin_amdgcn_permlane16_swap(fbits(a), fbits(b), false, false);
    return bitsf(r[0]) + bitsf(r[1]);
}
// Within the rows of sixteen lanes: the value of lane (l + N) % 16; and `mine` in the lanes below N and from N + 4 (N + 8 for
// <8> of eight lanes) on, the value lane l - N has of `from` in lanes N ..
template <int N>
__device__ __forceinline__ float row_ror(float v)
{
    return bitsf((uint32_t)__builtin_amdgcn_update_dpp(0, (int)fbits(v), 0x120 + N, 0xF, 0xF, true));
}
template <int N>
__device__ __forceinline__ float lanes_from(float mine, float from)
{
    return bitsf((uint32_t)__builtin_amdgcn_update_dpp((int)fbits(mine), (int)fbits(from), 0x110 + N, 0xF, 0xF & ~((1 << (N / 4)) - 1), false));
}
// maximum over the four lanes that hold one pair (lr, lr+16, lr+32, lr+48), in all four
__device__ __forceinline__ float max_rows(float v)
{
    uint2v r = __builtin_amdgcn_permlane32_swap(fbits(v), fbits(v), false, false);
    v = fmaxf(bitsf(r[0]), bitsf(r[1]));
    r = __builtin_amdgcn_permlane16_swap(fbits(v), fbits(v), false, false);
    return fmaxf(bitsf(r[0]), bitsf(r[1]));
}

// maximum over the wave, in every lane
__device__ __forceinline__ float max_lanes(float v)
{
    v = fmaxf(v, row_ror<8>(v));
    v = fmaxf(v, row_ror<4>(v));
    v = fmaxf(v, row_ror<2>(v));
    v = fmaxf(v, row_ror<1>(v));
    return max_rows(v);
}

// Where the pieces of a K row lie (piece p at p ^ k_swizzle): row 4q + r of an operand block.  A read of sixteen bytes a lane is
// served in quarters of lanes 0-3, 12-15 and, of the next sixteen, 4-11 (the other way round in the second), which ask for
// pieces four apart: with the row's own number as the swizzle the two halves met in the same banks.
__device__ __forceinline__ int k_swizzle(int q, int r) { return r | (((0x78 >> (2 * q)) & 3) << 2); }

// det_expf for arguments that are never positive (a score minus the maximum of its chunk): the same operations
// without the overflow test.  NaN stays NaN (the integer conversion of NaN is 0 in hardware; written as the
// instruction because the C conversion is undefined there).
__device__ __forceinline__ float exp_nonpos(float x)
{
    const float n = __builtin_rintf(x * 0x1.715476p+0f);
    float r = __builtin_fmaf(n, -0x1.62e4p-1f, x);
    r = __builtin_fmaf(n, -0x1.7f7d1cp-20f, r);
    float p = 0x1.a01a02p-13f;
    p = __builtin_fmaf(p, r, 0x1.6c16c2p-10f);
    p = __builtin_fmaf(p, r, 0x1.111112p-7f);
    p = __builtin_fmaf(p, r, 0x1.555556p-5f);
    p = __builtin_fmaf(p, r, 0x1.555556p-3f);
    p = __builtin_fmaf(p, r, 0.5f);
    p = __builtin_fmaf(p, r, 1.0f);
    p = __builtin_fmaf(p, r, 1.0f);
    int ni;
    asm("v_cvt_i32_f32 %0, %1" : "=v"(ni) : "v"(n));
    const float y = bitsf(fbits(p) + ((uint32_t)ni << 23));
    return x < -87.0f ? 0.0f : y;
}

// e >= 0 (or NaN) of eight tokens as three bf16 operands that sum to it exactly, by truncation
__device__ __forceinline__ void split_pieces(const float (&e)[8], bf16x8 (&piece)[3])
{
    uint32_t w[3][8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        w[0][k] = fbits(e[k]) & 0xFFFF0000u;
        const float r1 = e[k] - bitsf(w[0][k]);
        w[1][k] = fbits(r1) & 0xFFFF0000u;
        w[2][k] = fbits(r1 - bitsf(w[1][k]));  // at most 8 significant bits: exact in bf16
    }
#pragma unroll
    for (int y = 0; y < 3; ++y)  // the upper halves, in order
        piece[y] = __builtin_bit_cast(bf16x8, make_uint4(__builtin_amdgcn_perm(w[y][1], w[y][0], 0x07060302u),
                                                         __builtin_amdgcn_perm(w[y][3], w[y][2], 0x07060302u),
                                                         __builtin_amdgcn_perm(w[y][5], w[y][4], 0x07060302u),
                                                         __builtin_amdgcn_perm(w[y][7], w[y][6], 0x07060302u)));
}

}  // namespace det

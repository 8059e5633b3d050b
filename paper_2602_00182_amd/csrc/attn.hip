// Single-query attention over a KV cache in fixed 256-token chunks, and the softmax statistics it
// is built on.  Every reduction has a written order (the paper's section 6.5, invariants 2 and 3):
// scores on the matrix cores with one accumulator chain over the head dimension, chunk sums
// through the 256-leaf tree, chunk partials combined in ascending chunk order.  A chunk's
// arithmetic depends on nothing but that sequence's own cache rows and length.
#include <math.h>

#include <atomic>
#include <type_traits>

#include "attn_lane.h"
#include "attn_rows.h"
#include "geometry.h"
#include "internal.h"
#include "stream.h"

namespace det {

constexpr int kChunk = 256;
constexpr int kD = 128;
constexpr int kHalfTok = 128;  // tokens of the half chunk whose V^T sits in LDS at a time

// Softmax statistics of one 256-token chunk of one row, computed by ONE wavefront.  Lane 16r + i holds the
// scores of the tokens 64r + 16k + i, k = 0..3, of the chunk (s[k], valid[k]; chunk_token(lane, k)): the sixteen
// lanes of a row hold one group of 64 leaves of the 256-leaf tree, so the tree's strides 32 and 16 pair values
// of one lane, its strides 8, 4, 2, 1 are shifts inside a row of sixteen lanes (a modifier of the adding
// instruction), and only the four group sums cross rows, through scalar registers.
//   m_c = max of the valid scores (-inf if there is none);
//   e   = det_expf(s - m_c) for a valid token, 0 otherwise;
//   l_c = the 256-leaf sum of e: inside each group of 64 leaves, leaf j takes leaf j+off for off = 32, 16, .., 1,
//         and the four group sums q0..q3 combine as (q0+q2)+(q1+q3).
// m_c and l_c are returned in every lane.  No LDS, no barrier: the waves of a workgroup run it independently
// on different rows.  attn_tile and det_softmax_f32 call it.  attn_chunk_kernel below and attn_walk_kernel (attn_rows.hip) compute
// the same statistics, in the same order, from other lane layouts (add32, add16 and exp_nonpos of attn_lane.h); the tests hold
// their bytes to attn_tile's (test_gpu_attn_decode_forms.py, test_gpu_attn_walk.py, test_gpu_attn_few.py).
__device__ __forceinline__ int chunk_token(int lane, int k) { return ((lane >> 4) << 6) + (k << 4) + (lane & 15); }
__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ void chunk_stats(const float (&s)[4], const bool (&valid)[4], float& m_c, float (&e)[4],
                                            float& l_c)
{
    float sv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) sv[k] = valid[k] ? s[k] : -INFINITY;
    float m = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));  // max is exact: any order
    m = fmaxf(m, lane_plus<8>(m));  // (a lane past its row's end reads 0 here and holds nothing of use afterwards:
    m = fmaxf(m, lane_plus<4>(m));  //  lane 0 of a row only ever takes lanes inside the row)
    m = fmaxf(m, lane_plus<2>(m));
    m = fmaxf(m, lane_plus<1>(m));
    m = fmaxf(fmaxf(lane_value(m, 0), lane_value(m, 16)), fmaxf(lane_value(m, 32), lane_value(m, 48)));
    m_c = m;
#pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = valid[k] ? det_expf(sv[k] - m) : 0.0f;
    const float a = e[0] + e[2];  // stride 32: leaf j takes leaf j + 32, j = i and j = 16 + i
    const float b = e[1] + e[3];
    float t = a + b;              // stride 16
    t = t + lane_plus<8>(t);
    t = t + lane_plus<4>(t);
    t = t + lane_plus<2>(t);
    t = t + lane_plus<1>(t);
    const float qa = lane_value(t, 0) + lane_value(t, 32);
    const float qb = lane_value(t, 16) + lane_value(t, 48);
    l_c = qa + qb;
}

// Combination of chunk statistics in ascending chunk order:
//   m = max_c m_c;  w_c = det_expf(m_c - m);  L = fold_c (L + w_c*l_c) from +0.
__device__ __forceinline__ float combine_max(const float* mc, int nc)
{
    float m = mc[0];
    for (int c = 1; c < nc; ++c) m = fmaxf(m, mc[c]);
    return m;
}

// ------------------------------------------------------------------ attention, pass 1

// One workgroup: one 256-token chunk of one cache slot's K/V, for up to RT query rows (tokens) times G
// query heads that share the KV head ("pairs"): the rows of one prompt share each chunk of K and V (causal prefill: row i of a
// prompt has length p + i), in calls too small for attn_rows.hip and for the rows it leaves.  (Rows that share nothing have
// attn_chunk_kernel.)  Grid (chunk, head group, row tile); 256 threads.
//
// The arithmetic of one (row, head, chunk) is the same whatever else sits in the workgroup:
//   scores: wave w takes tokens 64w..64w+63 of the chunk as four 16-token blocks; the K rows are the row
//           operand of v_mfma_f32_16x16x32_bf16 and sixteen pairs' query vectors its column operand; four
//           steps cover the 128 head dimensions in ascending order (step i takes d = 32g + 8i + e for lane
//           group g), one accumulator chain per (token, pair), then one multiply by the scale.
//   stats : chunk_stats, one wave per pair, a token valid iff it lies below that row's length.
//   PV    : on the matrix cores as well.  e_j (fp32, >= 0) is cut into three bf16 pieces by truncation,
//           e = hi + mid + lo exactly, so every product piece * v is exact in fp32; one accumulator chain
//           per (pair, d) runs over the chunk's eight 32-token steps in ascending order, each step adding
//           the hi, then the mid, then the lo products (V^T is the row operand, the pieces the column
//           operand).  Tokens at or past the row's length have e = 0 and add +0.
// Rows of a tile that name different slots are handled one slot after the other (same arithmetic, no
// sharing).  V rows at or past the longest length of such a group are never read (zeros instead), K rows
// likewise.  A V row between two lengths of a group meets e = 0 in the shorter ones, which keeps a finite
// value out of their sums but not an infinity or a NaN (0 * inf = NaN): where a group of several lengths ends
// with a NaN, its rows are taken again one by one (the look for it costs 0.3 to 0.7 us a launch: sixteen rows at the end of
// 300 tokens, 32/8 heads 20.5 -> 20.7 us, 100 rows of one prompt, 16/16 heads 10.0 -> 10.4).  So what the cache holds at and
// past a row's length cannot reach that row's output.

// Index (in uint4 = eight tokens of one head dimension) into the transposed V half tile: 128 rows (d) of 16
// pieces (128 tokens), the pieces of a row rotated by d + d/8 so that both the transposing writes (rows 8
// apart, same piece) and the operand reads (sixteen consecutive rows, same piece) spread over the banks.
__device__ __forceinline__ int vt_index(int d, int piece) { return d * 16 + ((piece + d + (d >> 3)) & 15); }
// Index (in floats) of token tok in pair p's score row: the row's 16-byte pieces are rotated by p, so that
// sixteen pairs reading or writing the same tokens hit different banks.
__device__ __forceinline__ int sc_index(int p, int tok)
{
    return p * kChunk + ((((tok >> 2) + p) & 63) << 2) + (tok & 3);
}

template <int I>
__device__ __forceinline__ uint32_t u4_word(const uint4& v)
{
    return I == 0 ? v.x : (I == 1 ? v.y : (I == 2 ? v.z : v.w));
}

// The workgroup's part: chunk c, head group hgrp, row tile `tile`; len and slot (LDS, complete) hold the tile's rows'
// lengths (0 or less: not this call's) and slots.
template <int G, int RT, bool DIRECT>
__device__ __forceinline__ void attn_tile(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kcache,
                                          const uint16_t* __restrict__ vcache, float* __restrict__ ws_m,
                                          float* __restrict__ ws_l, float* __restrict__ ws_o, uint16_t* __restrict__ out,
                                          int Hq, int Hkv, int Lmax, int ncmax, float scale, int c, int hgrp, int tile,
                                          const int* len, const int* slot)
{
    constexpr int NP = G * RT;             // pairs (row, head) of the workgroup
    constexpr int CBK = (NP + 15) / 16;    // blocks of sixteen pairs
    constexpr int DPW = 2 * CBK;           // (pair block, 16-wide d block) units of one wave in PV: 8*CBK/4
    static_assert((G & (G - 1)) == 0 && CBK <= 4, "pair layout");
    __shared__ __align__(16) float sc[NP * kChunk];  // scores, then e_j
    __shared__ uint4 vt[128 * 16];                   // V^T of half a chunk: [d][token], 32 KB
    __shared__ float mc_s[NP], lc_s[NP];             // the pairs' chunk statistics (DIRECT only)
    __shared__ int s_nan;                            // some sum of the group is a NaN
    const int kvh = (hgrp * G) / (Hq / Hkv);
    const int t0 = c * kChunk;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, lr = lane & 15;

    bool any = false;
#pragma unroll
    for (int ri = 0; ri < RT; ++ri) any = any || len[ri] > t0;
    if (!any) return;  // uniform over the workgroup

    auto row_len = [&](int ri) { return uni(len[ri]); };
    auto row_slot = [&](int ri) { return uni(slot[ri]); };
    uint32_t done = 0, alone = 0;  // rows computed, and rows that are groups of their own
    bool first_group = true;
#pragma unroll 1
    for (int first = 0; first < RT; ++first) {
        if (((done >> first) & 1u) || row_len(first) <= t0) continue;
        const int group_slot = row_slot(first);
        uint32_t mask = 0;
        int minlen = 0x7FFFFFFF, maxlen = 0;
#pragma unroll
        for (int ri = 0; ri < RT; ++ri) {
            const int l = row_len(ri);
            if (l > t0 && row_slot(ri) == group_slot && (ri == first || !((alone >> first | alone >> ri) & 1u))) {
                mask |= 1u << ri;
                minlen = l < minlen ? l : minlen;
                maxlen = l > maxlen ? l : maxlen;
            }
        }
        done |= mask;
        if (!first_group) __syncthreads();  // the previous group's LDS contents are no longer read
        first_group = false;
        // tokens of this chunk at or past the shortest length and below the longest (uniform over the workgroup)
        const bool window = minlen < maxlen && minlen < t0 + kChunk;
        if (window && tid == 0) s_nan = 0;  // (set below, barriers later)

        const size_t kv_base = ((size_t)group_slot * Hkv + kvh) * (size_t)Lmax * kD;
        const uint16_t* kp = kcache + kv_base;
        const uint16_t* vp = vcache + kv_base;

        // ---- V: half a chunk at a time through registers into the transposed LDS tile.  A thread owns the
        // 8 x 8 block (tokens 8*oc .. +7 of the half) x (d = 8*o .. +7): eight 16-byte loads, one per token.
        const int o = lane & 15, oc = 4 * wave + (lane >> 4);
        uint4 vr[8];
        auto load_v = [&](int hf) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int tok = t0 + kHalfTok * hf + 8 * oc + j;
                vr[j] = make_uint4(0, 0, 0, 0);
                if (tok < maxlen) vr[j] = *reinterpret_cast<const uint4*>(vp + (size_t)tok * kD + 8 * o);
            }
        };
        auto store_vt = [&]() {
            auto row = [&](auto e_tag) {
                constexpr int E = decltype(e_tag)::value;
                uint32_t w[4];
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const uint32_t a = u4_word<E / 2>(vr[2 * jj]), b = u4_word<E / 2>(vr[2 * jj + 1]);
                    w[jj] = (E & 1) ? ((a >> 16) | (b & 0xFFFF0000u)) : ((a & 0xFFFFu) | (b << 16));
                }
                vt[vt_index(8 * o + E, oc)] = make_uint4(w[0], w[1], w[2], w[3]);
            };
            row(std::integral_constant<int, 0>{});
            row(std::integral_constant<int, 1>{});
            row(std::integral_constant<int, 2>{});
            row(std::integral_constant<int, 3>{});
            row(std::integral_constant<int, 4>{});
            row(std::integral_constant<int, 5>{});
            row(std::integral_constant<int, 6>{});
            row(std::integral_constant<int, 7>{});
        };
        load_v(0);  // travels while the scores are computed

        // ---- scores
        {
            uint4 qf[CBK][4];
#pragma unroll
            for (int cb = 0; cb < CBK; ++cb) {
                const int p = 16 * cb + lr;
                const int ri = p / G, h = p % G;
#pragma unroll
                for (int i = 0; i < 4; ++i) qf[cb][i] = make_uint4(0, 0, 0, 0);
                if (p < NP && ((mask >> ri) & 1u)) {
                    const uint4* qp = reinterpret_cast<const uint4*>(
                        q + ((size_t)(tile * RT + ri) * Hq + (size_t)hgrp * G + h) * kD + 32 * g);
#pragma unroll
                    for (int i = 0; i < 4; ++i) qf[cb][i] = qp[i];
                }
            }
#pragma unroll
            for (int tb = 0; tb < 4; ++tb) {
                const int tok = t0 + 64 * wave + 16 * tb + lr;
                uint4 kf[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) kf[i] = make_uint4(0, 0, 0, 0);
                if (tok < maxlen) {
                    const uint4* kr = reinterpret_cast<const uint4*>(kp + (size_t)tok * kD + 32 * g);
#pragma unroll
                    for (int i = 0; i < 4; ++i) kf[i] = kr[i];
                }
#pragma unroll
                for (int cb = 0; cb < CBK; ++cb) {
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[i]),
                                                                      __builtin_bit_cast(bf16x8, qf[cb][i]), acc, 0, 0, 0);
                    // lane holds S[token = 16tb + 4g + v][pair = 16cb + lr]
                    const int p = 16 * cb + lr;
                    if (p < NP)
                        *reinterpret_cast<float4*>(&sc[sc_index(p, 64 * wave + 16 * tb + 4 * g)]) =
                            make_float4(acc[0] * scale, acc[1] * scale, acc[2] * scale, acc[3] * scale);
                }
            }
        }
        store_vt();  // first half of V; nobody reads vt before the barriers below
        load_v(1);   // second half travels during the statistics and the first half of PV
        __syncthreads();

        // ---- statistics: wave w takes pairs w, w+4, ..; no barrier inside
#pragma unroll
        for (int pi = 0; pi < (NP + 3) / 4; ++pi) {
            const int p = 4 * pi + wave;
            if (p < NP) {  // uniform over the wave
                const int ri = p / G;
                const bool in_group = (mask >> ri) & 1u;
                const int l = len[ri];
                float sv[4], e[4], m_c, l_c;
                bool vd[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    vd[k] = in_group && t0 + chunk_token(lane, k) < l;
                    sv[k] = sc[sc_index(p, chunk_token(lane, k))];
                }
                chunk_stats(sv, vd, m_c, e, l_c);
#pragma unroll
                for (int k = 0; k < 4; ++k) sc[sc_index(p, chunk_token(lane, k))] = e[k];
                if (lane == 0 && in_group) {
                    const size_t part = ((size_t)(tile * RT + ri) * Hq + (size_t)hgrp * G + p % G) * ncmax + c;
                    ws_m[part] = m_c;
                    ws_l[part] = l_c;
                    if constexpr (DIRECT) {
                        mc_s[p] = m_c;
                        lc_s[p] = l_c;
                    }
                }
            }
        }
        __syncthreads();

        // ---- PV.  Wave w owns pair block pb and the 16-wide d blocks db0 .. db0+DPW-1.
        const int pb = CBK == 1 ? 0 : (CBK == 2 ? wave >> 1 : wave);
        const int db0 = CBK == 1 ? 2 * wave : (CBK == 2 ? 4 * (wave & 1) : 0);
        const int pp = 16 * pb + lr;  // this lane's pair as the column of the operand and of the output
        f32x4 acc[DPW];
#pragma unroll
        for (int u = 0; u < DPW; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto pv_half = [&](int hf) {
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                const int tk = kHalfTok * hf + 32 * s4 + 8 * g;  // this lane's eight tokens of the step
                float ev[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) ev[k] = 0.0f;
                if (pp < NP) {
                    const float4 a = *reinterpret_cast<const float4*>(&sc[sc_index(pp, tk)]);
                    const float4 b = *reinterpret_cast<const float4*>(&sc[sc_index(pp, tk + 4)]);
                    ev[0] = a.x, ev[1] = a.y, ev[2] = a.z, ev[3] = a.w;
                    ev[4] = b.x, ev[5] = b.y, ev[6] = b.z, ev[7] = b.w;
                }
                uint32_t hi[8], mid[8], lo[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    hi[k] = __float_as_uint(ev[k]) & 0xFFFF0000u;
                    const float r1 = ev[k] - __uint_as_float(hi[k]);
                    mid[k] = __float_as_uint(r1) & 0xFFFF0000u;
                    lo[k] = __float_as_uint(r1 - __uint_as_float(mid[k]));  // at most 8 significant bits: exact in bf16
                }
                auto pack = [](const uint32_t (&x)[8]) {
                    return __builtin_bit_cast(bf16x8, make_uint4((x[0] >> 16) | (x[1] & 0xFFFF0000u), (x[2] >> 16) | (x[3] & 0xFFFF0000u),
                                                                 (x[4] >> 16) | (x[5] & 0xFFFF0000u), (x[6] >> 16) | (x[7] & 0xFFFF0000u)));
                };
                const bf16x8 phi = pack(hi), pmid = pack(mid), plo = pack(lo);
#pragma unroll
                for (int u = 0; u < DPW; ++u) {
                    const bf16x8 vf = __builtin_bit_cast(bf16x8, vt[vt_index(16 * (db0 + u) + lr, 4 * s4 + g)]);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, phi, acc[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pmid, acc[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, plo, acc[u], 0, 0, 0);
                }
            }
        };
        pv_half(0);
        __syncthreads();  // every wave is done with the first half of V^T
        store_vt();
        __syncthreads();
        pv_half(1);
        if (window) {
            f32x4 t = acc[0];  // a NaN stays one (so does inf - inf, at the cost of a needless repetition)
#pragma unroll
            for (int u = 1; u < DPW; ++u) t += acc[u];
            const float nan = (t[0] + t[1]) + (t[2] + t[3]);
            if (nan != nan && pp < NP && ((mask >> (pp / G)) & 1u)) s_nan = 1;
            __syncthreads();
            if (s_nan) {  // again, one by one
                alone |= mask;
                done &= ~mask;
                --first;
                continue;
            }
        }

        // lane holds O[d = 16*(db0+u) + 4g + v][pair pp]
        bool mine = false;
        int my_row = 0, my_len = 0;
#pragma unroll
        for (int ri = 0; ri < RT; ++ri)
            if (pp < NP && pp / G == ri && ((mask >> ri) & 1u)) {
                mine = true;
                my_row = tile * RT + ri;
                my_len = len[ri];
            }
        if (DIRECT && mine && my_len <= kChunk) {
            // The row has this one chunk: what the second pass would compute from the single partial, computed
            // here with the same operations (m = m_c; w = det_expf(m_c - m); L = 0 + w*l_c; O = 0 + w*O_c;
            // out = bf16(O / L)), and the partial output is not written.
            const float w = det_expf(mc_s[pp] - mc_s[pp]);
            const float wl = w * lc_s[pp];
            const float L = 0.0f + wl;
            uint16_t* orow = out + ((size_t)my_row * Hq + (size_t)hgrp * G + pp % G) * kD + 4 * g;
#pragma unroll
            for (int u = 0; u < DPW; ++u) {
                float y[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float wo = w * acc[u][v];
                    const float O = 0.0f + wo;
                    y[v] = O / L;
                }
                *reinterpret_cast<uint2*>(orow + 16 * (db0 + u)) = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
            }
        } else if (mine) {
            const size_t part = ((size_t)my_row * Hq + (size_t)hgrp * G + pp % G) * ncmax + c;
            float* op = ws_o + part * kD + 4 * g;
#pragma unroll
            for (int u = 0; u < DPW; ++u) {
                float2* dst = reinterpret_cast<float2*>(op + 16 * (db0 + u));  // 8-byte stores: ws_o is only that aligned
                dst[0] = make_float2(acc[u][0], acc[u][1]);
                dst[1] = make_float2(acc[u][2], acc[u][3]);
            }
        }
    }
}

template <int G, int RT, bool DIRECT>
__global__ __launch_bounds__(256, 2) void attn_tile_kernel(const uint16_t* __restrict__ q,
                                                        const uint16_t* __restrict__ kcache,
                                                        const uint16_t* __restrict__ vcache,
                                                        const int32_t* __restrict__ seqlens,
                                                        const int32_t* __restrict__ slots,
                                                        float* __restrict__ ws_m, float* __restrict__ ws_l,
                                                        float* __restrict__ ws_o, uint16_t* __restrict__ out, int R,
                                                        int Hq, int Hkv, int Lmax, int ncmax, float scale,
                                                        int len_offset)
{
    const int hgrp = blockIdx.y, tile = blockIdx.z, tid = threadIdx.x;
    const int c = blockIdx.x;
    // the tile's rows: length (0: no such row) and slot
    __shared__ int len[RT], slot[RT];
    if (tid < RT) {
        const int r = tile * RT + tid;
        int l = 0, sl = -1;
        if (r < R) {
            l = seqlens[r] + len_offset;
            l = l > Lmax ? Lmax : l;
            sl = slots ? slots[r] : r;
        }
        len[tid] = l;
        slot[tid] = sl;
    }
    __syncthreads();
    if constexpr (DIRECT) {
        // rows without any token get zeros, from the workgroups of chunk 0 (there is no second pass to do it)
        if (c == 0) {
#pragma unroll
            for (int ri = 0; ri < RT; ++ri) {
                const int r = tile * RT + ri;
                if (r < R && len[ri] <= 0)
                    for (int i = tid; i < G * kD; i += 256) out[((size_t)r * Hq + (size_t)hgrp * G) * kD + i] = 0;
            }
        }
    }
    attn_tile<G, RT, DIRECT>(q, kcache, vcache, ws_m, ws_l, ws_o, out, Hq, Hkv, Lmax, ncmax, scale, c, hgrp, tile, len, slot);
}

// The chunk of workgroup (x, stream) of attn_chunk_kernel, a stream being one (row, KV head), counted in grid
// order.  Workgroups go round-robin over the eight XCDs, and inside one over its compute units: where the number of chunks has
// factors of two, chunk x of every stream would fall to the same places, and those that always get the first chunks, which more
// rows reach, work while the others wait (16 chunks, 48 rows of 200 to 4096 tokens: the first XCD 1.37 times the mean).  So the
// chunks of a group as long as that power of two change places from stream to stream, by the leading bits of the stream's
// number times the golden ratio, whose values are even over any run of streams; a stream stays in eight-chunk order or nearly so.
// us without, and with (in attn_tile_kernel with one row a workgroup, which had these launches before): 48 rows of 200 to 4096
// tokens, 32/8 heads 110.8 -> 89.1 (the bytes at the rate of a copy 80), of 100 to 2000,
// 16/16 heads 103 -> 84.5, 32 rows of 1001, 32/8 heads 43 -> 34.  Over 800 launches (2 to 32 chunks, 8 to 64 rows, 2 to 16 KV heads;
// lengths equal, all half, of the upper half and of twenty to one) 4.5 % less time, equal lengths level, 15 launches slower by more
// than 1.5 %, at most 4.  Heads in front of chunks in the grid, an earlier order for the same reason, took 3 % less, 86 launches
// slower, up to 17 % (9 chunks, 16 rows of 1151 tokens, 16/4 heads 17.8 -> 20.5, now 17.4).  An odd number of chunks spreads by
// itself.  Above 32 the chunks stay where they are: as even already (level over 60 launches).
__device__ __forceinline__ int attn_chunk_of(int x, int stream, int ncmax)
{
    const int group = ncmax <= DET_ATTN_TURN_CHUNKS ? ncmax & -ncmax : 1;
    return x ^ (int)__umulhi((uint32_t)stream * 0x9E3779B9u, (uint32_t)group);
}

// Pass 1 for rows that share nothing (one row a workgroup: decode), one chunk for the G heads of a KV head.  The order of
// every operation is attn_tile's; what differs is where things are.  A wave's share of the chunk is 64 tokens up to the weights, then
// 32 dimensions.  K comes as whole rows by LDS-DMA and V in whole rows through registers, all in one round trip; a wave reads
// its K operands from its own part of the buffer and leaves its V there (transposed by the LDS read), so that two workgroups fit
// a compute unit.  Loaded as the operand lies in registers, sixteen rows an instruction, K took the memory pipe twice as long (one
// workgroup of a launch of 4096 tokens, 32/8 heads: 3.4 of 7.5 us until everything had landed).
// A wave has at most eight pairs where the operand has sixteen columns, and alone on its SIMD it issues a vector instruction
// every 5.6 clocks: so the scores are dealt out over all lanes before the exponentials (2600 clocks before, 800 now), and the
// three pieces of e are cut once, not by each wave for its dimensions (second product 4300 -> 1300).
// Two barriers: the waves' maxima, then e and V.  What bounds the small launches is this chain of one memory round trip and
// two barriers, the large ones memory: 64 rows of 4096 tokens, 32/8 heads 5.4 TB/s.
// Against the form before (both passes, us): one sequence of 4096 tokens, 32/8 heads 12.0 -> 9.9, of 512, 16/4 heads 10.5 -> 8.2; 24 of
// 30 to 536, 16/4 14.6 -> 11.6; 64 of 300, 16/4 8.6 -> 6.7; against attn_tile_kernel with one row a workgroup, which took launches of
// more than 512 workgroups: 48 of 200 to 4096, 32/8 93.2 -> 89.1; 32 of 1024 to 2048 45.5 -> 41.2; 64 of 100 to 4096 114.5 -> 107.4;
// 128 of 300 to 2048 122.9 -> 113.7; 64 of 4096 203 -> 198; 48 of 200 to 4096, 16/16 163 -> 155; none of 50 launches slower.
template <int G, bool DIRECT>
__global__ __launch_bounds__(256, 2) void attn_chunk_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kcache,
                                                           const uint16_t* __restrict__ vcache,
                                                           const int32_t* __restrict__ seqlens,
                                                           const int32_t* __restrict__ slots, float* __restrict__ ws_m,
                                                           float* __restrict__ ws_l, float* __restrict__ ws_o,
                                                           uint16_t* __restrict__ out, int Hq, int Hkv, int Lmax, int ncmax,
                                                           float scale, int len_offset)
{
    constexpr int GP = G < 4 ? 4 : G;     // pairs a row of sixteen lanes is dealt out for
    constexpr int NX = GP;                // scores a lane goes on with (of sixteen it gets from the products)
    constexpr int kPieceRow = 2 * kChunk + 64;  // bytes of a pair's pieces, so that the pairs' rows lie in different banks
    __shared__ uint4 vbuf[kChunk * 16];  // K of the chunk, then V, [token][piece], swizzled as in attn_rows.hip
    __shared__ uint4 pieces[3][GP][kPieceRow / 16];  // e's three bf16 pieces, [piece][pair][token]
    __shared__ float wave_m[4][16], wave_l[4][16];
    const int hgrp = blockIdx.y, r = blockIdx.z;
    const int c = attn_chunk_of(blockIdx.x, hgrp + (int)gridDim.y * r, ncmax);
    const int kvh = (hgrp * G) / (Hq / Hkv);
    const int t0 = c * kChunk;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, lr = lane & 15;
    uint4 qf[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) qf[i] = make_uint4(0, 0, 0, 0);
    if (lr < G) {
        const uint4* qp = reinterpret_cast<const uint4*>(q + ((size_t)r * Hq + (size_t)hgrp * G + lr) * kD + 32 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i) qf[i] = qp[i];
    }
    const int len = __builtin_amdgcn_readfirstlane(attn_row_len(seqlens, r, len_offset, Lmax));
    uint16_t* orow = DIRECT ? out + ((size_t)r * Hq + (size_t)hgrp * G) * kD : nullptr;
    if (DIRECT && c == 0 && len <= 0) {  // a row without any token: zeros (there is no second pass to write them)
        for (int i = tid; i < G * kD; i += 256) orow[i] = 0;
    }
    if (len <= t0) return;
    const int slot = slots ? __builtin_amdgcn_readfirstlane(slots[r]) : r;
    const int held = min(kChunk, len - t0);  // tokens of the chunk
    const size_t kv_base = (((size_t)slot * Hkv + kvh) * (size_t)Lmax + t0) * kD;

    uint4 vr[16];
    {
        typedef __attribute__((address_space(3))) uint32_t lds_u32;
        typedef __attribute__((address_space(1))) const uint32_t glob_u32;
        const char* kp = reinterpret_cast<const char*>(kcache + kv_base);
        const uint4* vp = reinterpret_cast<const uint4*>(vcache + kv_base);
#pragma unroll
        for (int b = 0; b < 16; ++b) {
            const uint32_t off = (uint32_t)min(64 * wave + 4 * b + g, held - 1) * 256u + 16u * (uint32_t)(lr ^ k_swizzle((b >> 1) & 3, g));
            __builtin_amdgcn_global_load_lds((glob_u32*)(kp + off), (lds_u32*)(vbuf + wave * 1024 + b * 64), 16, 0, 0);
        }
        asm volatile("" ::: "memory");  // the wait below counts on this order: loads return in order
#pragma unroll
        for (int b = 0; b < 16; ++b) {
            vr[b] = vp[min(64 * wave + 4 * b + g, held - 1) * 16 + lr];
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x4F70);  // vmcnt(16): all but V
        __builtin_amdgcn_sched_barrier(0);
    }
    uint4 kf[2][2][4];  // row lr of operand block (st, b): token 32st + 8(lr/4) + 4b + lr%4 of the wave's
    {
        const char* base = reinterpret_cast<const char*>(vbuf) + wave * 16384 + (8 * (lr >> 2) + (lr & 3)) * 256;
        const int kz = k_swizzle(lr >> 2, lr & 3);
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    kf[st][b][i] = *reinterpret_cast<const uint4*>(base + st * 8192 + b * 1024 + (((4 * g + i) ^ kz) << 4));
    }

    // ---- scores.  The products leave the sixteen tokens 32 st + 8 g + k (st = 0, 1, k = 0 .. 7) of pair lr in lane (g, lr), lr < G,
    // and nothing of use in the other lanes, so they are dealt out: lane (g, lr) goes on with the NX scores x = NX*(lr / GP) ..
    // of pair lr % GP, x = 8 st + k, in the order of the tokens.
    float s[NX];
    {
        float all[16];
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[st][b][i]),
                                                                  __builtin_bit_cast(bf16x8, qf[i]), acc, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) all[8 * st + 4 * b + v] = acc[v];
            }
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            s[x] = all[x];
            if constexpr (GP == 4) {
                s[x] = lanes_from<4>(s[x], all[4 + x]);
                s[x] = lanes_from<8>(s[x], all[8 + x]);
                s[x] = lanes_from<12>(s[x], all[12 + x]);
            } else {
                s[x] = lanes_from<8>(s[x], all[8 + x]);
            }
        }
    }
    const int share = lr / GP;                                                               // which of a pair's scores
    const int first = GP == 4 ? 32 * (share >> 1) + 8 * g + 4 * (share & 1) : 32 * share + 8 * g;  // their first token of the wave's 64
    float m_c = -INFINITY;
#pragma unroll
    for (int x = 0; x < NX; ++x) {
        s[x] = 64 * wave + first + x < held ? s[x] * scale : -INFINITY;
        m_c = fmaxf(m_c, s[x]);
    }
    if constexpr (GP == 4) m_c = fmaxf(m_c, row_ror<4>(m_c));
    m_c = fmaxf(m_c, row_ror<8>(m_c));
    m_c = max_rows(m_c);
    if (g == 0) wave_m[wave][lr] = m_c;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    m_c = fmaxf(fmaxf(wave_m[0][lr], wave_m[1][lr]), fmaxf(wave_m[2][lr], wave_m[3][lr]));

    // ---- e and this wave's 64 leaves of the tree, leaf 32 st + 8 g + k: stride 32 pairs the halves of the row of lanes, 16 and 8 the rows
    {
#pragma unroll
        for (int x = 0; x < NX; ++x) s[x] = exp_nonpos(s[x] - m_c);
        float a[NX];
#pragma unroll
        for (int x = 0; x < NX; ++x) a[x] = s[x] + row_ror<8>(s[x]);
        const float r0 = add32(a[0], a[1]), r1 = add32(a[2], a[3]);
        float t4 = add16(r0, r1);  // rows hold k = 0 2 1 3, and below 4 6 5 7
        if constexpr (GP == 4)
            t4 = t4 + row_ror<4>(t4);  // stride 4: the neighbouring quarters of the row of lanes
        else
            t4 = t4 + add16(add32(a[NX - 4], a[NX - 3]), add32(a[NX - 2], a[NX - 1]));
        const float t2 = add16(t4, t4);
        const float t1 = add32(t2, t2);
        if (g == 0) wave_l[wave][lr] = t1;
        // the three pieces (split_pieces: truncation, exact), once for all waves
        uint32_t w[3][NX];
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            w[0][x] = fbits(s[x]) & 0xFFFF0000u;
            const float rest = s[x] - bitsf(w[0][x]);
            w[1][x] = fbits(rest) & 0xFFFF0000u;
            w[2][x] = fbits(rest - bitsf(w[1][x]));
        }
#pragma unroll
        for (int y = 0; y < 3; ++y) {
            uint32_t* to = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(pieces[y][lr % GP]) + 2 * (64 * wave + first));
            const uint2 lo = make_uint2(__builtin_amdgcn_perm(w[y][1], w[y][0], 0x07060302u), __builtin_amdgcn_perm(w[y][3], w[y][2], 0x07060302u));
            if constexpr (NX == 4) {
                *reinterpret_cast<uint2*>(to) = lo;
            } else {
                *reinterpret_cast<uint4*>(to) = make_uint4(lo.x, lo.y, __builtin_amdgcn_perm(w[y][NX - 3], w[y][NX - 4], 0x07060302u),
                                                           __builtin_amdgcn_perm(w[y][NX - 1], w[y][NX - 2], 0x07060302u));
            }
        }
    }
#pragma unroll
    for (int b = 0; b < 16; ++b) {
        const int tok = 64 * wave + 4 * b + g;  // token % 4 = g, token / 8 % 2 = b / 2 % 2
        if (tok >= held) vr[b] = make_uint4(0, 0, 0, 0);
        vbuf[tok * 16 + ((((lr >> 1) ^ (g | (((b >> 1) & 1) << 2))) << 1) | (lr & 1))] = vr[b];
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const float l_c = (wave_l[0][lr] + wave_l[2][lr]) + (wave_l[1][lr] + wave_l[3][lr]);

    // ---- weighted sums: wave w owns d = 32w .. 32w+31, all tokens in ascending steps (steps past the length would add zeros)
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    typedef __attribute__((address_space(3))) short4v lds_short4;
    const uint32_t vbase = (uint32_t)(uintptr_t)(lds_char_t*)vbuf + (uint32_t)(8 * g + (lr >> 2)) * 256u + 8u * (uint32_t)(lr & 3);
    const uint32_t f = (uint32_t)((lr >> 2) | ((g & 1) << 2));
    auto pv_step = [&](int st) {
        bf16x8 piece[3];
#pragma unroll
        for (int y = 0; y < 3; ++y) piece[y] = __builtin_bit_cast(bf16x8, pieces[y][lr % GP][4 * st + g]);  // (columns from G on are not used)
        bf16x8 vf[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t at = vbase + (uint32_t)st * 8192u + (((uint32_t)(2 * wave + u) ^ f) << 5);
            typedef short short8v __attribute__((ext_vector_type(8)));
            const short4v v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)at);
            const short4v v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)(at + 1024u));
            vf[u] = __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
        }
#pragma unroll
        for (int y = 0; y < 3; ++y)
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[u], piece[y], acc[u], 0, 0, 0);
    };
    if (held > kChunk - 32) {
#pragma unroll
        for (int st = 0; st < 8; ++st) pv_step(st);
    } else {
        for (int st = 0; 32 * st < held; ++st) pv_step(st);
    }

    // lane holds O[d = 32w + 16u + 4g + v][pair lr]
    if (lr >= G) return;
    if (DIRECT && len <= kChunk) {
        // the row's only chunk: what the second pass would compute from the single partial, with its operations
        const float w = det_expf(m_c - m_c);
        const float wl = w * l_c;
        const float L = 0.0f + wl;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float y[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float wo = w * acc[u][v];
                const float O = 0.0f + wo;
                y[v] = O / L;
            }
            *reinterpret_cast<uint2*>(orow + lr * kD + 32 * wave + 16 * u + 4 * g) =
                make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
        }
    }
    const size_t part = ((size_t)r * Hq + (size_t)hgrp * G + lr) * ncmax + c;
    if (wave == 0 && g == 0) {
        ws_m[part] = m_c;
        ws_l[part] = l_c;
    }
    if (DIRECT && len <= kChunk) return;
    float* op = ws_o + part * kD + 32 * wave + 4 * g;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        float2* dst = reinterpret_cast<float2*>(op + 16 * u);  // 8-byte stores: ws_o is only that aligned
        dst[0] = make_float2(acc[u][0], acc[u][1]);
        dst[1] = make_float2(acc[u][2], acc[u][3]);
    }
}

// The rows of a slot-naming call that a walking launch leaves (attn_rows.h), as a bit per row in LDS; returns the words in use.
// All of the workgroup's threads call it.
constexpr int kLeftWords = 1024;  // 65535 rows
template <int G>
__device__ __forceinline__ int find_left_rows(const int32_t* __restrict__ seqlens, const int32_t* __restrict__ slots,
                                              int len_offset, int Lmax, int R, int Hkv, uint64_t* left, int* scratch)
{
    int limit = kWalkChunks;
    if (Lmax > kWalkChunks * kChunk)
        limit = attn_walk_limit(seqlens, len_offset, Lmax, R, (R + kWalkPairs / G - 1) / (kWalkPairs / G), kWalkPairs / G, Hkv, scratch);
    attn_for_row_words<kWalkPairs / G>(seqlens, slots, len_offset, Lmax, R, limit, [&](int w, const attn_row_classes& k) {
        if ((threadIdx.x & 63) == 0) left[w] = k.deep;
    });
    const int words = (R + 63) >> 6;
    __syncthreads();
    return words;
}

// Pass 1 for those rows, eight to a workgroup as in attn_tile_kernel: items are (chunk, KV head, eight rows), dealt
// round-robin over the grid, so that the rows that walk cost no workgroups.  (Dealt in runs of four, a few long rows kept few
// workgroups busy: 32 sequences of 1000 to 4000 tokens beside a prompt of 497, 32/8 heads 449 us for the call, 230 so.)
template <int G, bool DIRECT>
__global__ __launch_bounds__(256, 2) void attn_left_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kcache,
                                                          const uint16_t* __restrict__ vcache,
                                                          const int32_t* __restrict__ seqlens,
                                                          const int32_t* __restrict__ slots, float* __restrict__ ws_m,
                                                          float* __restrict__ ws_l, float* __restrict__ ws_o,
                                                          uint16_t* __restrict__ out, int R, int Hq, int Hkv, int Lmax,
                                                          int ncmax, float scale, int len_offset)
{
    constexpr int RT = 8;
    __shared__ uint64_t left[kLeftWords];
    __shared__ int len[RT], slot[RT], scratch;
    const int words = find_left_rows<G>(seqlens, slots, len_offset, Lmax, R, Hkv, left, &scratch);
    const int per_tile = Hkv * ncmax;
    int next = (int)blockIdx.x;  // this workgroup's next item, counted from the current tile's first
#pragma unroll 1
    for (int w = 0; w < words; ++w) {
        const uint64_t word = left[w];
        if (word == 0) continue;
#pragma unroll 1
        for (int y = 0; y < 8; ++y) {
            const uint32_t rows = (uint32_t)(word >> (8 * y)) & 255u;
            if (rows == 0) continue;
            const int tile = 8 * w + y;
            if (next < per_tile) {
                __syncthreads();  // the previous tile's lengths are no longer read
                if (threadIdx.x < RT) {
                    const int r = tile * RT + (int)threadIdx.x;
                    const bool in = (rows >> threadIdx.x) & 1u;
                    len[threadIdx.x] = in ? attn_row_len(seqlens, r, len_offset, Lmax) : 0;
                    slot[threadIdx.x] = in ? slots[r] : -1;
                }
                __syncthreads();
            }
#pragma unroll 1
            for (; next < per_tile; next += (int)gridDim.x) {
                attn_tile<G, RT, DIRECT>(q, kcache, vcache, ws_m, ws_l, ws_o, out, Hq, Hkv, Lmax, ncmax, scale, next / Hkv,
                                         next % Hkv, tile, len, slot);
                __syncthreads();  // its LDS contents are no longer read
            }
            next -= per_tile;
        }
    }
}

// ------------------------------------------------------------------ attention, pass 2

// Grid (query head, sequence); 128 threads, thread = d.  The arithmetic is the ascending-chunk fold
// of the canonical order; only the data movement is parallel.  What bounds it is its chain of memory round trips: the
// length, beside it the statistics, then the first eight chunks' sums, asked for in front of everything that needs the
// statistics; the next eight while these are folded.  Each of the two waves has the statistics of 64 chunks in its lanes (the
// maximum is exact, so order free; the weights w_c = det_expf(m_c - m) one chunk a lane) and hands them out as scalars, without LDS
// and barriers.  Both passes, us, with the statistics through LDS, twice from memory, in front of the sums, and now: one
// sequence of 512 tokens, 16/4 heads 7.9 -> 7.0, of 4096, 32/8 9.8 -> 9.3; 24 of 30 to 536, 16/4 11.5 -> 10.6, of 100 to 1024 14.5 -> 13.0;
// 32 of 1024 to 2048, 32/8 42.9 -> 40.6; 48 of 200 to 4096 87.3 -> 84.9; two of 32768 level.
// QUANT: instead of the bf16 output row the kernel writes its 8-bit block quantization (the bytes
// det_quant_act_q8 makes of it): a wave's 64 values are one block, so the block maximum is a wave
// reduction; `out` is then the int8 code array [B, Hq*128] and `scales` the block-major scale array
// with row stride ldd.
template <bool QUANT>
__device__ __forceinline__ void attn_combine(int h, int b, int len, const float* __restrict__ ws_m,
                                             const float* __restrict__ ws_l, const float* __restrict__ ws_o,
                                             void* __restrict__ out, int Hq, int ncmax, float* __restrict__ scales, int ldd,
                                             int first_pass_wrote_short_rows)
{
    const int d = threadIdx.x;
    const size_t o_idx = ((size_t)b * Hq + h) * kD + d;
    auto store = [&](uint16_t y) {
        if constexpr (!QUANT) {
            static_cast<uint16_t*>(out)[o_idx] = y;
        } else {
            const float a = bf16_to_f32(y);
            const float amax = max_lanes(fabsf(a));
            const float df = amax / 127.0f;
            int v = 0;
            if (df != 0.0f) {
                const float r = rintf(a / df);
                v = r < -127.0f ? -127 : (r > 127.0f ? 127 : (int)r);
            }
            static_cast<int8_t*>(out)[o_idx] = (int8_t)v;
            if ((d & 63) == 0) scales[(size_t)(2 * h + (d >> 6)) * ldd + b] = df;
        }
    };
    const int lane = d & 63;
    const size_t part = ((size_t)b * Hq + h) * ncmax;
    float mc = lane < ncmax ? ws_m[part + lane] : 0.0f, lc = lane < ncmax ? ws_l[part + lane] : 0.0f;  // (what is past the length is not used)
    if (first_pass_wrote_short_rows && len <= kChunk) return;  // rows of at most one chunk are complete (uniform)
    if (len <= 0) {  // uniform over the workgroup
        store(0);
        return;
    }
    const int nc = (len + kChunk - 1) / kChunk;
    const float* op = ws_o + part * kD + d;
    constexpr int W = 8;
    float o[W];
#pragma unroll
    for (int u = 0; u < W; ++u) o[u] = op[(size_t)min(u, nc - 1) * kD];
    float m = lane < nc ? mc : -INFINITY;
    for (int c = lane + kWave; c < nc; c += kWave) m = fmaxf(m, ws_m[part + c]);
    m = max_lanes(m);

    float L = 0.0f, O = 0.0f;
    for (int c0 = 0; c0 < nc; c0 += kWave) {
        const int n = min(kWave, nc - c0);
        if (c0 > 0) {
            mc = lane < n ? ws_m[part + c0 + lane] : 0.0f;
            lc = lane < n ? ws_l[part + c0 + lane] : 0.0f;
        }
        const float w = det_expf(mc - m);
        const float wl = w * lc;
        auto fold = [&](int c, float oc) __attribute__((always_inline)) {
            L = L + bitsf((uint32_t)__builtin_amdgcn_readlane((int)fbits(wl), c));
            const float wo = bitsf((uint32_t)__builtin_amdgcn_readlane((int)fbits(w), c)) * oc;
            O = O + wo;
        };
        for (int c = 0; c < n; c += W) {
            float next[W];
            const bool more = c0 + c + W < nc;
            if (more) {
#pragma unroll
                for (int u = 0; u < W; ++u) next[u] = op[(size_t)min(c0 + c + W + u, nc - 1) * kD];
            }
            if (c + W <= n) {
#pragma unroll
                for (int u = 0; u < W; ++u) fold(c + u, o[u]);
            } else {
#pragma unroll
                for (int u = 0; u < W - 1; ++u)
                    if (c + u < n) fold(c + u, o[u]);
            }
            if (more) {
#pragma unroll
                for (int u = 0; u < W; ++u) o[u] = next[u];
            }
        }
    }
    store(f32_to_bf16_rne(O / L));
}

template <bool QUANT>
__global__ __launch_bounds__(128) void attn_combine_kernel(const int32_t* __restrict__ seqlens,
                                                           const float* __restrict__ ws_m,
                                                           const float* __restrict__ ws_l,
                                                           const float* __restrict__ ws_o,
                                                           void* __restrict__ out, int Hq, int Lmax,
                                                           int ncmax, int len_offset, float* __restrict__ scales,
                                                           int ldd, int first_pass_wrote_short_rows)
{
    const int b = blockIdx.y;
    attn_combine<QUANT>(blockIdx.x, b, attn_row_len(seqlens, b, len_offset, Lmax), ws_m, ws_l, ws_o, out, Hq, ncmax, scales,
                        ldd, first_pass_wrote_short_rows);
}

// Pass 2 for those rows, (row, head) items dealt round-robin over the grid.  A workgroup finds its next item's row by
// counting the rows of whole words (looking at the rows one by one took 80 us for 961 of them).
template <int G, bool QUANT>
__global__ __launch_bounds__(128) void attn_left_combine_kernel(const int32_t* __restrict__ seqlens,
                                                                const int32_t* __restrict__ slots,
                                                                const float* __restrict__ ws_m,
                                                                const float* __restrict__ ws_l,
                                                                const float* __restrict__ ws_o, void* __restrict__ out,
                                                                int R, int Hq, int Hkv, int Lmax, int ncmax, int len_offset,
                                                                float* __restrict__ scales, int ldd)
{
    __shared__ uint64_t left[kLeftWords];
    __shared__ int scratch;
    const int words = find_left_rows<G>(seqlens, slots, len_offset, Lmax, R, Hkv, left, &scratch);
    const int lane = (int)threadIdx.x & 63;
    int word = 0, before = 0;  // the word of the current item's row, and the rows of the words before it
#pragma unroll 1
    for (int item = (int)blockIdx.x;; item += (int)gridDim.x) {
        const int row = item / Hq;  // counted over those rows
        for (; word < words; ++word) {
            const int n = __builtin_popcountll(left[word]);
            if (row < before + n) break;
            before += n;
        }
        if (word >= words) return;
        const uint64_t bits = left[word];
        const bool it = ((bits >> lane) & 1ull) && __builtin_popcountll(bits & ((1ull << lane) - 1ull)) == row - before;
        const int b = 64 * word + __builtin_ctzll(__ballot(it));
        __syncthreads();  // the previous item's weights are no longer read
        attn_combine<QUANT>(item % Hq, b, attn_row_len(seqlens, b, len_offset, Lmax), ws_m, ws_l, ws_o, out, Hq, ncmax, scales,
                            ldd, QUANT ? 0 : 1);
    }
}

// ------------------------------------------------------------------ softmax on given scores

constexpr int kMaxChunksHook = 1024;

// One workgroup per row; wave w computes the statistics of chunks w, w+4, .. (chunk_stats), then the chunks
// are combined in ascending order; p holds e_j until the final rescale.
__global__ __launch_bounds__(256) void softmax_kernel(const float* __restrict__ s,
                                                      const int32_t* __restrict__ lens,
                                                      float* __restrict__ p, float* __restrict__ m_out,
                                                      float* __restrict__ l_out, int Lmax)
{
    __shared__ float mc[kMaxChunksHook];
    __shared__ float lc[kMaxChunksHook];
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int len = lens[r];
    len = len > Lmax ? Lmax : len;
    if (len <= 0) {
        if (tid == 0) {
            m_out[r] = -INFINITY;
            l_out[r] = 0.0f;
        }
        return;
    }
    const float* sr = s + (size_t)r * Lmax;
    float* pr = p + (size_t)r * Lmax;
    const int nc = (len + kChunk - 1) / kChunk;
    for (int c = wave; c < nc; c += 4) {
        float sv[4], e[4], m_c, l_c;
        bool vd[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = c * kChunk + chunk_token(lane, k);
            vd[k] = j < len;
            sv[k] = vd[k] ? sr[j] : 0.0f;
        }
        chunk_stats(sv, vd, m_c, e, l_c);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (vd[k]) pr[c * kChunk + chunk_token(lane, k)] = e[k];
        if (lane == 0) {
            mc[c] = m_c;
            lc[c] = l_c;
        }
    }
    __syncthreads();  // also orders this workgroup's writes of e_j before the reads below
    const float m = combine_max(mc, nc);
    float L = 0.0f;
    for (int c = 0; c < nc; ++c) {
        const float w = det_expf(mc[c] - m);
        const float wl = w * lc[c];
        L = L + wl;
    }
    for (int c = 0; c < nc; ++c) {
        const int j = c * kChunk + tid;
        if (j < len) {
            const float w = det_expf(mc[c] - m);
            const float we = w * pr[j];
            pr[j] = we / L;
        }
    }
    if (tid == 0) {
        m_out[r] = m;
        l_out[r] = L;
    }
}

// The rows of a walking launch that it leaves (attn_rows.h).
template <int G>
static void launch_left(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens, const int32_t* slots,
                        int len_offset, void* out, float* ws_m, float* ws_l, float* ws_o, float* qscales, int R, int Hq,
                        int Hkv, int Lmax, int ncmax, float scale, hipStream_t s)
{
    const uint16_t *qq = static_cast<const uint16_t*>(q), *kk = static_cast<const uint16_t*>(kcache),
                   *vv = static_cast<const uint16_t*>(vcache);
    const dim3 grid(G == 8 ? 256 : 512), grid2(1024);  // pass 1: what is resident at a time (G = 8 needs 104 KB of LDS)
    if (qscales) {
        hipLaunchKernelGGL((attn_left_kernel<G, false>), grid, dim3(256), 0, s, qq, kk, vv, seqlens, slots, ws_m, ws_l, ws_o,
                           nullptr, R, Hq, Hkv, Lmax, ncmax, scale, len_offset);
        hipLaunchKernelGGL((attn_left_combine_kernel<G, true>), grid2, dim3(128), 0, s, seqlens, slots, ws_m, ws_l, ws_o,
                           out, R, Hq, Hkv, Lmax, ncmax, len_offset, qscales, (R + 3) & ~3);
    } else {
        hipLaunchKernelGGL((attn_left_kernel<G, true>), grid, dim3(256), 0, s, qq, kk, vv, seqlens, slots, ws_m, ws_l, ws_o,
                           static_cast<uint16_t*>(out), R, Hq, Hkv, Lmax, ncmax, scale, len_offset);
        if (ncmax > 1)  // else every row is complete
            hipLaunchKernelGGL((attn_left_combine_kernel<G, false>), grid2, dim3(128), 0, s, seqlens, slots, ws_m, ws_l, ws_o,
                               out, R, Hq, Hkv, Lmax, ncmax, len_offset, nullptr, 0);
    }
}
static int attn_left(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens, const int32_t* slots,
                     int len_offset, void* out, float* ws_m, float* ws_l, float* ws_o, float* qscales, int R, int Hq, int Hkv,
                     int Lmax, int ncmax, float scale, hipStream_t s)
{
#define DET_LAUNCH_LEFT(GG)                                                                                              \
    launch_left<GG>(q, kcache, vcache, seqlens, slots, len_offset, out, ws_m, ws_l, ws_o, qscales, R, Hq, Hkv, Lmax, ncmax, \
                    scale, s)
    switch (Hq / Hkv) {
        case 1: DET_LAUNCH_LEFT(1); break;
        case 2: DET_LAUNCH_LEFT(2); break;
        case 4: DET_LAUNCH_LEFT(4); break;
        default: DET_LAUNCH_LEFT(8); break;
    }
#undef DET_LAUNCH_LEFT
    return check_launch();
}

// Rows that name their slots walk their chunks inside one workgroup (attn_rows.hip) where that gives every compute
// unit one.  Below, the chunks of a row in workgroups of their own are the better split: sixteen rows at the end
// of 4000 tokens take 23 us that way and 176 walking, 256 such rows (128 workgroups) 165 and 180, 512 rows (256
// workgroups) 309 and 178; 1000 rows of one prompt (504) 170 and 60.
constexpr long long kWalkWorkgroups = DET_ATTN_WALK_WGS;

static size_t attn_ws_floats(int B, int Hq, int Lmax)
{
    const size_t nc = (size_t)(Lmax + kChunk - 1) / kChunk;
    return (size_t)B * Hq * nc * (2 + kD);
}

// Chunk partials for det_attn_decode_static: a fixed array in the code object instead of a buffer the
// caller brings.  Every device the library runs on holds its own copy at its own address; in host code
// the name `scratch` is only a handle for hipGetSymbolAddress, never a pointer to pass to a kernel.
static __device__ __align__(256) unsigned char scratch[DET_ATTN_STATIC_WS_BYTES];

constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

// Address of the current device's copy of `scratch`, looked up on the first call on that device.
static int static_scratch_ptr(void** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_last_hip_error((int)e);
        return DET_EHIP;
    }
    if (dev < 0 || dev >= kMaxDevices) return DET_ESHAPE;
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_last_hip_error((int)e);
            return DET_EHIP;
        }
        g_scratch_ptr[dev].store(p, std::memory_order_release);  // two racing first calls store the same address
    }
    *out = p;
    return DET_OK;
}

}  // namespace det

using namespace det;

extern "C" size_t det_attn_decode_workspace_bytes(int B, int Hq, int D, int Lmax)
{
    if (B < 1 || Hq < 1 || D != kD || Lmax < 1) return 0;
    return attn_ws_floats(B, Hq, Lmax) * sizeof(float);
}

int det::attn_decode_impl(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens,
                          const int32_t* slots, int len_offset, void* out, void* ws, size_t ws_bytes, int B, int Hq, int Hkv, int D,
                          int Lmax, float scale, hipStream_t s, void* qscales)
{
    if (!q || !kcache || !vcache || !seqlens || !out || !ws || B < 1 || Hq < 1 || Hkv < 1 || Lmax < 1)
        return DET_EINVAL;
    if (D != kD || Hq % Hkv != 0) return DET_ESHAPE;
    const int G = Hq / Hkv;
    if (G != 1 && G != 2 && G != 4 && G != 8) return DET_ESHAPE;
    if (B > 65535 || Hkv > 65535 || Hq > 65535) return DET_ESHAPE;
    if (!aligned16(q) || !aligned16(kcache) || !aligned16(vcache) || !aligned16(out) || !aligned16(ws))
        return DET_EALIGN;
    if (ws_bytes < det_attn_decode_workspace_bytes(B, Hq, D, Lmax)) return DET_EWORKSPACE;
    const int ncmax = (Lmax + kChunk - 1) / kChunk;
    const size_t n = (size_t)B * Hq * ncmax;
    float* ws_m = static_cast<float*>(ws);
    float* ws_l = ws_m + n;
    float* ws_o = ws_l + n;
    // Launch geometry (which workgroup computes a (row, head, chunk); never its arithmetic):
    //   * rows that name their slots (prefill: consecutive rows of a prompt share a slot) walk their chunks in
    //     one workgroup where there are enough of them (kWalkWorkgroups); fewer, but sixteen or more, go eight to
    //     a workgroup per chunk, so that they share each chunk of K and V;
    //   * other rows take attn_chunk_kernel.
    const bool tiled = slots != nullptr && B >= DET_ATTN_NAMED_ROWS;
    if (tiled && attn_walk_workgroups(B, G, Hkv) >= kWalkWorkgroups) {
        if (qscales && !aligned16(qscales)) return DET_EALIGN;
        const int rc = attn_walk(q, kcache, vcache, seqlens, slots, len_offset, out, static_cast<float*>(qscales), ws_o, B, Hq,
                                 Hkv, Lmax, ncmax, scale, s);
        if (rc != DET_OK || ncmax <= kWalkChunks) return rc;  // no row can be left
        return attn_left(q, kcache, vcache, seqlens, slots, len_offset, out, ws_m, ws_l, ws_o, static_cast<float*>(qscales), B,
                         Hq, Hkv, Lmax, ncmax, scale, s);
    }
    const int RT = tiled ? 8 : 1;
    const dim3 grid(ncmax, Hkv, (B + RT - 1) / RT);
    const uint16_t* qq = static_cast<const uint16_t*>(q);
    const uint16_t* kk = static_cast<const uint16_t*>(kcache);
    const uint16_t* vv = static_cast<const uint16_t*>(vcache);
    // Without the quantizing second pass, the first pass itself finishes every row of at most one chunk.
    const bool direct = qscales == nullptr;
    uint16_t* out16 = static_cast<uint16_t*>(out);
#define DET_LAUNCH_TILE(GG, RTV, DIR)                                                                                   \
    hipLaunchKernelGGL((attn_tile_kernel<GG, RTV, DIR>), grid, dim3(256), 0, s, qq, kk, vv, seqlens, slots, ws_m, ws_l, \
                       ws_o, out16, B, Hq, Hkv, Lmax, ncmax, scale, len_offset)
#define DET_LAUNCH_CHUNK(GG, DIR)                                                                                       \
    hipLaunchKernelGGL((attn_chunk_kernel<GG, DIR>), grid, dim3(256), 0, s, qq, kk, vv, seqlens, slots, ws_m, ws_l, ws_o, \
                       out16, Hq, Hkv, Lmax, ncmax, scale, len_offset)
#define DET_LAUNCH_ATTN(GG)                   \
    do {                                      \
        if (tiled && direct)                  \
            DET_LAUNCH_TILE(GG, 8, true);     \
        else if (tiled)                       \
            DET_LAUNCH_TILE(GG, 8, false);    \
        else if (direct)                      \
            DET_LAUNCH_CHUNK(GG, true);       \
        else                                  \
            DET_LAUNCH_CHUNK(GG, false);      \
    } while (0)
    switch (G) {
        case 1: DET_LAUNCH_ATTN(1); break;
        case 2: DET_LAUNCH_ATTN(2); break;
        case 4: DET_LAUNCH_ATTN(4); break;
        default: DET_LAUNCH_ATTN(8); break;
    }
#undef DET_LAUNCH_ATTN
#undef DET_LAUNCH_CHUNK
#undef DET_LAUNCH_TILE
    int rc = check_launch();
    if (rc != DET_OK) return rc;
    if (qscales) {
        if (!aligned16(qscales)) return DET_EALIGN;
        hipLaunchKernelGGL(attn_combine_kernel<true>, dim3(Hq, B), dim3(128), 0, s, seqlens, ws_m, ws_l, ws_o, out, Hq,
                           Lmax, ncmax, len_offset, static_cast<float*>(qscales), (B + 3) & ~3, 0);
    } else if (ncmax > 1) {  // with one chunk at most, every row is already complete
        hipLaunchKernelGGL(attn_combine_kernel<false>, dim3(Hq, B), dim3(128), 0, s, seqlens, ws_m, ws_l, ws_o, out, Hq,
                           Lmax, ncmax, len_offset, nullptr, 0, 1);
    }
    return check_launch();
}

extern "C" int det_attn_decode(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens,
                               void* out, void* ws, size_t ws_bytes, int B, int Hq, int Hkv, int D, int Lmax,
                               float scale, void* stream)
{
    return attn_decode_impl(q, kcache, vcache, seqlens, nullptr, 0, out, ws, ws_bytes, B, Hq, Hkv, D, Lmax, scale,
                            static_cast<hipStream_t>(stream));
}

extern "C" int det_attn_decode_static(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens,
                                      void* out, int B, int Hq, int Hkv, int D, int Lmax, float scale, void* stream)
{
    const size_t need = det_attn_decode_workspace_bytes(B, Hq, D, Lmax);
    if (need == 0) return (B < 1 || Hq < 1 || Lmax < 1) ? DET_EINVAL : DET_ESHAPE;
    if (need > (size_t)DET_ATTN_STATIC_WS_BYTES) return DET_EWORKSPACE;
    void* ws = nullptr;
    const int rc = static_scratch_ptr(&ws);
    if (rc != DET_OK) return rc;
    return attn_decode_impl(q, kcache, vcache, seqlens, nullptr, 0, out, ws, DET_ATTN_STATIC_WS_BYTES, B, Hq, Hkv, D,
                            Lmax, scale, static_cast<hipStream_t>(stream));
}

extern "C" int det_attn_decode_rows(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens,
                                    const int32_t* slots, void* out, void* ws, size_t ws_bytes, int R, int Hq, int Hkv,
                                    int D, int Lmax, float scale, void* stream)
{
    if (!slots) return DET_EINVAL;
    return attn_decode_impl(q, kcache, vcache, seqlens, slots, 0, out, ws, ws_bytes, R, Hq, Hkv, D, Lmax, scale,
                            static_cast<hipStream_t>(stream));
}

extern "C" int det_attn_decode_quant_q8(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens,
                                        const int32_t* slots, void* codes, void* scales, void* ws, size_t ws_bytes,
                                        int R, int Hq, int Hkv, int D, int Lmax, float scale, void* stream)
{
    if (!scales) return DET_EINVAL;
    return attn_decode_impl(q, kcache, vcache, seqlens, slots, 0, codes, ws, ws_bytes, R, Hq, Hkv, D, Lmax, scale,
                            static_cast<hipStream_t>(stream), scales);
}

extern "C" int det_softmax_f32(const float* s, const int32_t* lens, float* p, float* m_out, float* l_out,
                               int R, int Lmax, void* stream)
{
    if (!s || !lens || !p || !m_out || !l_out || R < 1 || Lmax < 1) return DET_EINVAL;
    if ((Lmax + kChunk - 1) / kChunk > kMaxChunksHook) return DET_ESHAPE;
    hipLaunchKernelGGL(softmax_kernel, dim3(R), dim3(256), 0, static_cast<hipStream_t>(stream), s, lens, p,
                       m_out, l_out, Lmax);
    return check_launch();
}

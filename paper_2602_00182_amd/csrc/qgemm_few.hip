// The block-quantized GEMM (qgemm.hip: definition, packing) for launches of at most four rows: the same operations on an
// element in the same order, so the same bytes.
#include <type_traits>

#include "qgemm.h"
#include "stream.h"

namespace det {

namespace {

constexpr int kProducers = 8;
constexpr int kBatch = 4;        // blocks of K a producer takes at a time: their activations are the sixteen columns of one operand
constexpr int kFewLds = 158 * 1024, kFewLdsHalf = 79 * 1024;
// The rows that are normalized here: two vectors of eight a thread, and up to three of them.  Every workgroup does it again, which is
// hidden by the wait for the first weights while it is short.  Quantized layer at a context of 512 with the norms' own launches, and
// without, us: small model 40.4 and 37.4 at one row, 40.9 and 38.5 at two, 41.3 and 40.0 at three, 42.2 and 42.5 at four; hidden
// 4096 (of its two norms one is in qgemm.hip's kernel, which gains at four too) 59.3 and 52.3, 58.3 and 52.7, 62.7 and 59.7, 63.5 and 63.3.
constexpr int kFewNormK = 4096, kFewNormRows = DET_QGEMM_NORM_ROWS;

// LDS: the packed weights as they lie in memory, activation codes [block][row][64], scales [block][4] and, with the norm, the rows
// as they come and the norm's weight.
__host__ __device__ constexpr int few_lds_bytes(int M, int cb, int K, bool norm)
{
    return (K >> 6) * (qstage_w_bytes(cb) + 16) + M * K + (norm ? (M + 1) * 2 * K : 0);
}

}  // namespace

// A workgroup owns 16*CB columns and all rows.  Such a launch is over in about the time its weights take to arrive, so nothing may
// stand between them: all of them have a place in LDS (122 KB at K = 14336 and 16 columns), no load waits for a slot and no
// wave for another but where it needs its results.  Eight waves (producers) take the batches of blocks of K in turn: a wave asks
// for all its batches at once, and as they arrive leaves t = d*s and the block's product P in the weights' place, (t, P) for each
// row and column, at most 512 of a column block's 544 bytes, and counts the batch.  Behind them a thread for each (row, column) runs
// acc = fma(t, P, acc) over all blocks in ascending order, which is all that has an order, eight batches (one of each producer)
// at a time.  Only those waves wait for others, so every wait ends.
// Against the general kernel, one row, us: K x N 2048 x 2048 5.8 -> 3.5, 4096 x 4096 7.7 -> 5.0, 4096 x 6144 9.9 -> 6.2, 2048 x 11264
// 8.4 -> 6.3, 5632 x 2048 9.1 -> 5.3, 14336 x 4096 15.5 -> 10.9; 40 random launches of one to four rows 1.4 to 2.5 times as fast, the
// same bytes.  (A launch of nothing takes 1.85, the loads alone of 14336 x 4096 9.4.)  What bounded earlier forms was the number
// of LDS instructions: an operand, scales and results for every single block of one to four rows instead of for four blocks took 13.7.
// 128-column packings stay with the general kernel: 2048 x 32000 11.2 there and 12.7 here.
// NORM: the rows are raw activations and the producers of every workgroup normalize and quantize them, with the operations of
// rmsnorm_kernel in its order (a team of four waves is its 256 threads), while the weights are on their way.
template <int CB, int EPI, bool NORM, int LDSB>
__global__ __launch_bounds__(64 * 16) void qgemm_few_kernel(const int8_t* __restrict__ qa, int K, const float* __restrict__ da,
                                                            const uint8_t* __restrict__ wp, void* C, int ldc, const uint16_t* R,
                                                            int ldr, int out_f32, int M, gemm_rope_args ra,
                                                            const uint16_t* __restrict__ x, const uint16_t* __restrict__ w_norm, float eps)
{
    constexpr int WST = qstage_w_bytes(CB), TC = 16 * CB;
    constexpr int U = kBatch;
    static_assert(U * kFewRows == 16, "a batch's rows are the columns of one operand");
    __shared__ uint4 lds[LDSB / 16];
    __shared__ float part[NORM ? 4 * kFewRows : 1];
    __shared__ int produced[kProducers], normed[2];  // what is done: batches of each producer, the two steps of the norm
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nst = K >> 6, nb = (nst + U - 1) / U;
    char* const base = reinterpret_cast<char*>(lds);
    const int act = nst * WST, sc = act + M * K, raw = sc + nst * 16;
    if (tid < kProducers) produced[tid] = 0;
    if (tid < 2) normed[tid] = 0;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const uint32_t addr = (uint32_t)(uintptr_t)(lds_char_t*)lds, lane16 = (uint32_t)lane * 16u;

    if (wave >= kProducers) {
        // ------------------------------------------------------------ chains
        const int ct = tid - 64 * kProducers;  // (row, column): ct / TC, ct % TC
        const bool mine = ct < M * TC;
        const int row = mine ? ct / TC : 0, n = (int)blockIdx.x * TC + (ct & (TC - 1) & ~3);
        // what the epilogue reads besides the sums; a thread and its three neighbours end with four columns of one row
        uint2 rv = make_uint2(0u, 0u);
        rope_factors rf;
        int p = 0, slot = 0;
        if constexpr (EPI == kEpiResidual) {
            if (mine) rv = *reinterpret_cast<const uint2*>(R + (size_t)row * ldr + n);
        }
        if constexpr (EPI == kEpiRopeAppend) {
            p = ra.pos[row];
            p = p < 0 ? 0 : (p >= ra.Lmax ? ra.Lmax - 1 : p);
            slot = ra.slots ? ra.slots[row] : row;
            rf = gemm_rope_factors(ra, p, n);
        }
        float acc = 0.0f;
        const char* from = base + (mine ? ct * 8 : 0);
        for (int s = 0; s < nst; s += U * kProducers) {
            await(produced, kProducers, s / (U * kProducers) + 1);
            if (s + U * kProducers <= nst) {
                float2 a[U * kProducers];
#pragma unroll
                for (int u = 0; u < U * kProducers; ++u) a[u] = *reinterpret_cast<const float2*>(from + (s + u) * WST);
#pragma unroll
                for (int u = 0; u < U * kProducers; ++u) acc = __builtin_fmaf(a[u].x, a[u].y, acc);
            } else {
#pragma unroll 4
                for (int u = s; u < nst; ++u) {
                    const float2 a = *reinterpret_cast<const float2*>(from + u * WST);
                    acc = __builtin_fmaf(a.x, a.y, acc);
                }
            }
        }
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __shfl(acc, (lane & ~3) + e, 64);
        if (!mine || (lane & 3) != 0) return;
        if constexpr (EPI == kEpiResidual)
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(C) + (size_t)row * ldc + n) = gemm_residual(v, rv);
        else if constexpr (EPI == kEpiRopeAppend)
            gemm_rope_append(v, ra, row, p, slot, n, rf);
        else
            gemm_epilogue_store<EPI>(v, C, ldc, R, ldr, row, n, out_f32);
        return;
    }

    // ---------------------------------------------------------------- producers
    const int g = lane >> 4, lr = lane & 15;
    const char* const x_bytes = reinterpret_cast<const char*>(NORM ? static_cast<const void*>(x) : qa);
    constexpr int kTeams = kProducers / 4;
    const int team = wave >> 2, tw = wave & 3, nvec = K >> 3;
    if constexpr (NORM) {  // this wave's vectors of its rows and of the norm's weight (which both teams load, the same bytes)
        auto load = [&](const char* src, int dst) __attribute__((always_inline)) {
            for (int i = 0; i < 2; ++i) {
                const int v = 256 * i + 64 * tw;
                if (v + lane < nvec) dma_block(src + 16 * v, lane16, addr + (uint32_t)(dst + 16 * v));
            }
        };
        for (int r = team; r < M; r += kTeams) load(x_bytes + (size_t)r * K * 2, raw + r * K * 2);
        load(reinterpret_cast<const char*>(w_norm), raw + M * K * 2);
    }
    int issued = 0;
    for (int b = wave; b < nb; b += kProducers) {
        const int s = U * b, n = min(U, nst - s), bytes = n * WST;
        if constexpr (!NORM) {  // lane: sixteen codes of row lane / 4 % M of block lane / 4 / M; scales of block `lane`
            const int br = lane >> 2, u = br / M, r = br - u * M;
            if (u < n) dma_lane(x_bytes + (size_t)r * K + 64 * (s + u) + 16 * (lane & 3), addr + (uint32_t)(act + s * M * 64));
            if (lane < n) dma_block(da + 4 * s, lane16, addr + (uint32_t)(sc + 16 * s));
            issued += 2;
        }
        const char* src = reinterpret_cast<const char*>(wp) + ((size_t)blockIdx.x * nst + s) * WST;
        for (int off = 0; off < bytes; off += 1024, ++issued)
            if ((int)lane16 < bytes - off) dma_block(src + off, lane16, addr + (uint32_t)(s * WST + off));
    }
    if constexpr (NORM) {
        wait_loads(issued);
        auto meet = [&](int i) __attribute__((always_inline)) {  // every wave of the teams has come this far
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (lane == 0) atomicAdd(&normed[i], 1);
            await(&normed[i], 1, kProducers);
        };
        uint4 xv[kFewRows / kTeams][2];
#pragma unroll
        for (int u = 0; u < kFewRows / kTeams; ++u) {
            const int r = team + kTeams * u;
            if (r >= M) continue;
            float ss = 0.0f;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int v = 256 * i + 64 * tw + lane;
                if (v < nvec) {
                    xv[u][i] = *reinterpret_cast<const uint4*>(base + raw + r * K * 2 + 16 * v);
                    ss = rms_fold(xv[u][i], ss);
                }
            }
            ss = wave_tree_sum(ss);
            if (lane == 0) part[4 * r + tw] = ss;
        }
        meet(0);
#pragma unroll
        for (int u = 0; u < kFewRows / kTeams; ++u) {
            const int r = team + kTeams * u;
            if (r >= M) continue;
            const float a = part[4 * r] + part[4 * r + 2], b = part[4 * r + 1] + part[4 * r + 3];
            const float rs = rms_scale(a + b, K, eps);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int v = 256 * i + 64 * tw + lane;
                if (v < nvec) {
                    const uint4 y = rms_apply(xv[u][i], *reinterpret_cast<const uint4*>(base + raw + M * K * 2 + 16 * v), rs);
                    float df;
                    const uint2 c = quant_vector_q8(y, df);
                    *reinterpret_cast<uint2*>(base + act + ((v >> 3) * M + r) * 64 + 8 * (v & 7)) = c;
                    if ((lane & 7) == 0) *reinterpret_cast<float*>(base + sc + 16 * (v >> 3) + 4 * r) = df;
                }
            }
        }
        meet(1);
    }

    // This lane's share of a batch of blocks s .. s+3: column lr of the product's activation operand is row lr % 4 of block s + lr / 4
    // (rows past M repeat the last, blocks past the end are zeros and stay unused).  So the product with the weights of block s + u
    // holds in its columns 4u .. 4u+3 what is wanted, one operand read serves four blocks, and the lane goes on with that alone: P of
    // four columns (4g .. 4g+3), the row's d and the columns' s of its block.
    const int lu = lr >> 2, row = min(lr & 3, M - 1);
    auto batch = [&](int s, int before) __attribute__((always_inline)) {
        const bool held = s + lu < nst;
        const int sl = held ? s + lu : nst - 1;
        const v4i xa = *reinterpret_cast<const v4i*>(base + act + (sl * M + row) * 64 + 16 * g);
        const float d = *reinterpret_cast<const float*>(base + sc + 16 * sl + 4 * row);
        uint2 sraw[CB], codes[CB][U];
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            sraw[j] = *reinterpret_cast<const uint2*>(base + sl * WST + 512 * CB + j * 32 + g * 8);
#pragma unroll
            for (int u = 0; u < U; ++u) codes[j][u] = *reinterpret_cast<const uint2*>(base + min(s + u, nst - 1) * WST + j * 512 + lane * 8);
        }
#pragma unroll
        for (int j = 0; j < CB; ++j) {
#pragma unroll
            for (int u = 0; u < U; ++u) asm volatile("" : "+v"(codes[j][u].x), "+v"(codes[j][u].y));
        }
        if (before > 0) publish(&produced[wave], before);  // behind these reads the writes of the batch before are done too
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            v4i pr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) pr[u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(code_bytes(codes[j][u]), xa, kProductStart, 0, 0, 0);
            float pf[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) pf[v] = product(lu < 2 ? (lu == 0 ? pr[0][v] : pr[1][v]) : (lu == 2 ? pr[2][v] : pr[3][v]));
            if (held && (lr & 3) < M) {
                float4* to = reinterpret_cast<float4*>(base + sl * WST + (row * TC + 16 * j + 4 * g) * 8);
                to[0] = make_float4(d * bf16lo_to_f32(sraw[j].x), pf[0], d * bf16hi_to_f32(sraw[j].x), pf[1]);
                to[1] = make_float4(d * bf16lo_to_f32(sraw[j].y), pf[2], d * bf16hi_to_f32(sraw[j].y), pf[3]);
            }
        }
    };
    constexpr int LB = (U * WST + 1023) / 1024 + (NORM ? 0 : 2);  // loads of a batch (a shorter one is its wave's last)
    int done = 0;
    for (int b = wave; b < nb; b += kProducers, ++done) {
        wait_loads(issued - min(LB * (done + 1), issued));
        batch(U * b, done);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    publish(&produced[wave], 0x7FFFFFFF);
}

namespace {

template <int CB, int EPI, bool NORM>
void launch(const qgemm_few_args& a, hipStream_t s)
{
    const dim3 grid(a.N / (16 * CB)), block(64 * (kProducers + (a.M * 16 * CB + 63) / 64));
    const int8_t* qa = static_cast<const int8_t*>(a.codes);
    const float* da = static_cast<const float*>(a.scales);
    const uint8_t* wp = static_cast<const uint8_t*>(a.wp);
    const uint16_t *R = static_cast<const uint16_t*>(a.R), *x = static_cast<const uint16_t*>(a.x), *wn = static_cast<const uint16_t*>(a.w_norm);
    if (few_lds_bytes(a.M, CB, a.K, NORM) <= kFewLdsHalf)
        hipLaunchKernelGGL((qgemm_few_kernel<CB, EPI, NORM, kFewLdsHalf>), grid, block, 0, s, qa, a.K, da, wp, a.C, a.ldc, R, a.ldr,
                           a.out_f32, a.M, a.ra, x, wn, a.eps);
    else
        hipLaunchKernelGGL((qgemm_few_kernel<CB, EPI, NORM, kFewLds>), grid, block, 0, s, qa, a.K, da, wp, a.C, a.ldc, R, a.ldr,
                           a.out_f32, a.M, a.ra, x, wn, a.eps);
}

template <int CB>
void launch_epi(int epi, const qgemm_few_args& a, hipStream_t s)
{
    const bool norm = a.x != nullptr;
    switch (epi) {
        case kEpiStore: launch<CB, kEpiStore, false>(a, s); break;
        case kEpiResidual: launch<CB, kEpiResidual, false>(a, s); break;
        case kEpiSwiglu: norm ? launch<CB, kEpiSwiglu, true>(a, s) : launch<CB, kEpiSwiglu, false>(a, s); break;
        default: norm ? launch<CB, kEpiRopeAppend, true>(a, s) : launch<CB, kEpiRopeAppend, false>(a, s); break;
    }
}

}  // namespace

bool qgemm_few_fits(int M, int cb, int K, bool norm)
{
    return M <= (norm ? kFewNormRows : kFewRows) && cb <= 4 && K <= (norm ? kFewNormK : 32768) && few_lds_bytes(M, cb, K, norm) <= kFewLds;
}

void qgemm_few(int epi, int cb, const qgemm_few_args& a, hipStream_t s)
{
    switch (cb) {
        case 1: launch_epi<1>(epi, a, s); break;
        case 2: launch_epi<2>(epi, a, s); break;
        default: launch_epi<4>(epi, a, s); break;
    }
}

}  // namespace det

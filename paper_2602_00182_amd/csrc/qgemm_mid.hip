// The block-quantized GEMM (qgemm.hip: definition, packing) on packings of 16 and 32 columns, for tiles of at most 48 and 32 rows:
// the same operations on an element in the same order, so the same bytes.
#include "qgemm.h"

namespace det {

namespace {

constexpr int kProducers = 8;

__host__ __device__ constexpr int mid_depth(int tiles) { return tiles == 1 ? 6 : (tiles == 2 ? 4 : 3); }  // blocks of K a producer has under way
__host__ __device__ constexpr int mid_groups(int tiles) { return tiles == 1 ? 4 : 2; }                    // groups of results LDS holds

}  // namespace

// A workgroup owns 16*CB columns and 16*RB rows.  The general kernel (qgemm_kernel) has one wave a column block and row group walk all
// of K, some 250 clocks a block of K while most of the compute unit waits; but only the accumulation has an order.  Here eight waves
// (producers) take the blocks in turn, straight from memory into registers, several blocks ahead: a block's codes and activations
// are used by one wave once, so LDS would only add a step.  They leave t = d*s and the product P in LDS, and behind them a wave for each
// 16 x 16 tile (chains) runs acc = fma(t, P, acc) over the blocks in ascending order, eight (one of each producer) at a time.  The
// two sides count in LDS what is done; a producer waits only where the results of the group that had its place are still to be read.
// (Chains wait for blocks, whose producers wait for chains of earlier groups only: every wait ends.)
// What bounds it: at one row block the weights' way into the compute unit (14336 x 4096, 8 rows: 33 MB in 14.1 us), then the
// activations, whose loads touch sixteen rows each.  Before (general kernel) and here, us:
//     K x N          8 rows         16 rows        32 rows        48 rows
//     2048 x 2048    6.7   5.2      8.0   5.7      8.1   5.8      8.9   6.5
//     2048 x 3072    6.7   5.2      8.1   5.8      8.9   6.5      9.0   8.7
//     5632 x 2048    9.9   7.6     12.9   8.3     13.0   8.4     14.1  10.7
//     4096 x 4096    8.7   7.3     11.2   8.3     11.8   9.2     12.8  11.8
//    14336 x 4096   17.0  14.1     24.2  15.2     26.8  21.3     31.5  30.1
//     4096 x 6144   10.4   8.5     11.8   8.8     12.2  11.0     (32-column packing)
template <int CB, int RB, int EPI>
__global__ __launch_bounds__(64 * (kProducers + CB * RB)) void qgemm_mid_kernel(const int8_t* __restrict__ qa, int K,
                                                                                const float* __restrict__ da, int ldd,
                                                                                const uint8_t* __restrict__ wp, void* C, int ldc,
                                                                                const uint16_t* R, int ldr, int out_f32, int M,
                                                                                gemm_rope_args ra)
{
    constexpr int WST = qstage_w_bytes(CB), TILES = CB * RB, D = mid_depth(TILES), G = mid_groups(TILES);
    __shared__ float4 results[G * kProducers * TILES * 2 * 64];  // [group][producer][tile][t, P][lane]
    __shared__ int produced[kProducers], chained[TILES];         // blocks of each producer, groups of each chain
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, lr = lane & 15;
    const int nst = K >> 6, m0 = blockIdx.y * (16 * RB);
    if (tid < kProducers) produced[tid] = 0;
    if (tid < TILES) chained[tid] = 0;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

    if (wave >= kProducers) {
        // ------------------------------------------------------------ chains
        const int tile = wave - kProducers, j = tile % CB, r = tile / CB;
        const int rowl = m0 + 16 * r + lr, n = (int)blockIdx.x * (16 * CB) + 16 * j + 4 * g;
        const bool mine = rowl < M;
        const int row = mine ? rowl : M - 1;
        uint2 rv = make_uint2(0u, 0u);  // what the epilogue reads besides the sums
        rope_factors rf;
        int p = 0, slot = 0;
        if constexpr (EPI == kEpiResidual) rv = *reinterpret_cast<const uint2*>(R + (size_t)row * ldr + n);
        if constexpr (EPI == kEpiRopeAppend) {
            p = ra.pos[row];
            p = p < 0 ? 0 : (p >= ra.Lmax ? ra.Lmax - 1 : p);
            slot = ra.slots ? ra.slots[row] : row;
            rf = gemm_rope_factors(ra, p, n);
        }
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        auto add = [&](const float4& t, const float4& pf) {
            v[0] = __builtin_fmaf(t.x, pf.x, v[0]);
            v[1] = __builtin_fmaf(t.y, pf.y, v[1]);
            v[2] = __builtin_fmaf(t.z, pf.z, v[2]);
            v[3] = __builtin_fmaf(t.w, pf.w, v[3]);
        };
        for (int i = 0; kProducers * i < nst; ++i) {
            await(produced, kProducers, i + 1);
            const float4* from = results + ((i % G) * kProducers * TILES + tile) * 128 + lane;
            if (kProducers * (i + 1) <= nst) {
                float4 t[kProducers], pf[kProducers];
#pragma unroll
                for (int w = 0; w < kProducers; ++w) {
                    t[w] = from[w * TILES * 128];
                    pf[w] = from[w * TILES * 128 + 64];
                }
#pragma unroll
                for (int w = 0; w < kProducers; ++w) add(t[w], pf[w]);
            } else {
                for (int w = 0; kProducers * i + w < nst; ++w) add(from[w * TILES * 128], from[w * TILES * 128 + 64]);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the group's results are read
            publish(&chained[tile], i + 1);
        }
        if (!mine) return;
        if constexpr (EPI == kEpiResidual)
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(C) + (size_t)row * ldc + n) = gemm_residual(v, rv);
        else if constexpr (EPI == kEpiRopeAppend)
            gemm_rope_append(v, ra, row, p, slot, n, rf);
        else
            gemm_epilogue_store<EPI>(v, C, ldc, R, ldr, row, n, out_f32);
        return;
    }

    // ---------------------------------------------------------------- producers
    struct Block {
        uint2 codes[CB], s[CB];
        v4i x[RB];
        float d[RB];
    };
    Block b[D];
    const char* const w_at = reinterpret_cast<const char*>(wp) + (size_t)blockIdx.x * nst * WST;
    const char* const x_at = reinterpret_cast<const char*>(qa) + (size_t)m0 * K;
    const char* const d_at = reinterpret_cast<const char*>(da + m0);
    uint32_t x_off[RB], d_off[RB];  // (K <= 2^22: the offsets of 48 rows fit)
#pragma unroll
    for (int r = 0; r < RB; ++r) {  // rows past M repeat the last
        const int row = min(16 * r + lr, M - 1 - m0);
        x_off[r] = (uint32_t)row * (uint32_t)K + 16u * (uint32_t)g;
        d_off[r] = 4u * (uint32_t)row;
    }
    const int mine = nst > wave ? (nst - wave + kProducers - 1) / kProducers : 0;  // blocks wave, wave + 8, ..
    auto load = [&](Block& to, int i) __attribute__((always_inline)) {
        const int st = wave + kProducers * min(i, mine - 1);  // (past the end: again the last, so that the loads in flight have one count)
        const char* w = w_at + (size_t)st * WST;  // (bases of the wave, offsets of the lane)
        const char* xs = x_at + 64 * (size_t)st;
        const char* ds = d_at + 4 * (size_t)st * ldd;
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            to.codes[j] = *reinterpret_cast<const uint2*>(w + (uint32_t)(j * 512 + lane * 8));
            to.s[j] = *reinterpret_cast<const uint2*>(w + (uint32_t)(512 * CB + j * 32 + g * 8));
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            to.x[r] = *reinterpret_cast<const v4i*>(xs + x_off[r]);
            to.d[r] = *reinterpret_cast<const float*>(ds + d_off[r]);
        }
    };
    int free_until = G;  // groups below this one have their place
    auto compute = [&](const Block& k, int i) __attribute__((always_inline)) {
        if (i >= free_until) {
            await(chained, TILES, i - G + 1);
            const int have = lds_look(&chained[lane < TILES ? lane : 0]);
            int least = __builtin_amdgcn_readfirstlane(have);
#pragma unroll
            for (int t = 1; t < TILES; ++t) least = min(least, __builtin_amdgcn_readlane(have, t));
            free_until = least + G;
        }
        float4* to = results + ((i % G) * kProducers + wave) * TILES * 128 + lane;
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            const v4i wu = code_bytes(k.codes[j]);
            const float s[4] = {bf16lo_to_f32(k.s[j].x), bf16hi_to_f32(k.s[j].x), bf16lo_to_f32(k.s[j].y), bf16hi_to_f32(k.s[j].y)};
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const v4i pr = __builtin_amdgcn_mfma_i32_16x16x64_i8(wu, k.x[r], kProductStart, 0, 0, 0);
                to[(r * CB + j) * 128] = make_float4(k.d[r] * s[0], k.d[r] * s[1], k.d[r] * s[2], k.d[r] * s[3]);
                to[(r * CB + j) * 128 + 64] = make_float4(product(pr[0]), product(pr[1]), product(pr[2]), product(pr[3]));
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the results lie in LDS
        publish(&produced[wave], i + 1 == mine ? 0x7FFFFFFF : i + 1);
    };
    if (mine == 0) {
        publish(&produced[wave], 0x7FFFFFFF);
        return;
    }
#pragma unroll
    for (int u = 0; u < D; ++u) load(b[u], u);
    for (int i = 0; i < mine; i += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (i + u < mine) compute(b[u], i + u);
            load(b[u], i + u + D);
        }
    }
}

namespace {

template <int CB, int RB>
void launch(int epi, const qgemm_few_args& a, int rows, hipStream_t s)
{
    const dim3 grid(a.N / (16 * CB), (a.M + rows - 1) / rows), block(64 * (kProducers + CB * RB));
    const int ldd = (a.M + 3) & ~3;
#define DET_MID(EPI)                                                                                                         \
    hipLaunchKernelGGL((qgemm_mid_kernel<CB, RB, EPI>), grid, block, 0, s, static_cast<const int8_t*>(a.codes), a.K,         \
                       static_cast<const float*>(a.scales), ldd, static_cast<const uint8_t*>(a.wp), a.C, a.ldc,              \
                       static_cast<const uint16_t*>(a.R), a.ldr, a.out_f32, a.M, a.ra)
    switch (epi) {
        case kEpiStore: DET_MID(kEpiStore); break;
        case kEpiResidual: DET_MID(kEpiResidual); break;
        case kEpiSwiglu: DET_MID(kEpiSwiglu); break;
        default: DET_MID(kEpiRopeAppend); break;
    }
#undef DET_MID
}

}  // namespace

// rows: of the tiles the launch is cut into (qgemm_tile_rows).  The lines lie where this form stops being the faster one: 16-column
// packings, 64 rows in one tile, us in the general kernel and here: 4096 x 4096 13.6 and 14.5, 14336 x 4096 35.6 and 37.6 (and 39.5 as two
// tiles of 32), 2048 x 3072 9.1 and 10.5; 64-column packings have four chains for a producer's every block: 2048 x 11264, 8 rows, 8.2
// and 8.6.
static_assert(DET_QGEMM_MID16_ROWS <= 48 && DET_QGEMM_MID32_ROWS <= 32, "the row blocks that qgemm_mid has kernels for");
bool qgemm_mid_fits(int M, int cb, int rows) { return (M <= rows ? M : rows) <= (cb == 1 ? DET_QGEMM_MID16_ROWS : (cb == 2 ? DET_QGEMM_MID32_ROWS : 0)); }

void qgemm_mid(int epi, int cb, const qgemm_few_args& a, int rows, hipStream_t s)
{
    const int rb = ((a.M <= rows ? a.M : rows) + 15) / 16;
    rows = 16 * rb;
    if (cb == 1) {
        switch (rb) {
            case 1: launch<1, 1>(epi, a, rows, s); break;
            case 2: launch<1, 2>(epi, a, rows, s); break;
            default: launch<1, 3>(epi, a, rows, s); break;
        }
    } else if (rb == 1) {
        launch<2, 1>(epi, a, rows, s);
    } else {
        launch<2, 2>(epi, a, rows, s);
    }
}

}  // namespace det

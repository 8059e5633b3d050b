// Deterministic block-quantized GEMM for gfx950 (the paper's primary kernel family is the quantized
// one, section 6.4; its format is not given, this one is defined here):
//
//   weights      4-bit codes q in -8..7 and a bf16 scale s per 64 consecutive k of a column
//   activations  8-bit codes p in -127..127 and an fp32 scale d per 64 consecutive k of a row
//   C[i][n] = bf16(acc),  acc = 0;  for b ascending:  acc = fma( d[i][b]*s[b][n], float(P), acc ),
//   P = sum over the block of p*q in int32 (exact: v_mfma_i32_16x16x64_i8, one instruction per block)
//
// Every floating-point operation of the definition is an individually rounded IEEE fp32 operation
// in a written order and the contraction is integer, so a CPU reproduces the bytes exactly.
// Batch invariance follows as for the bf16 kernel: an output element's chain never depends on M.
//
// Kernel shape: as the bf16 GEMM (gemm.hip) -- a workgroup owns 16*CB columns and up to 256 rows,
// K in 64-deep stages streamed through an LDS ring by waves that only load -- with two differences.
// Weights arrive packed (544*CB bytes a stage: for each 16-column block, 8 bytes a lane of codes in
// matrix-core operand order, then 16 scales), so a chunk's weights are one contiguous run copied as
// it lies.  And the eight computing waves split the tile by column block first (wave w: column block
// w % CB, row blocks w / CB, w / CB + 8/CB, ...): at small M the work per stage is the unpacking of
// the codes, which a single wave could not do at the rate the weights stream in.  Where few rows and narrow
// packings leave a workgroup one or two column blocks and at most three of rows, the stages are dealt out as well, in a kernel of its
// own (qgemm_mid.hip); launches of at most four rows have another where their weights fit LDS (qgemm_few.hip).  Launches of more rows
// take tiles of 32 or 64 rows x 64 or 128 columns instead (qgemm_tile_kernel).
#include <type_traits>

#include "internal.h"
#include "qgemm.h"
#include "stream.h"

namespace det {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kQRing = 144;   // KB of LDS ring
constexpr int kQWaves = 8;    // waves that can compute
constexpr int kQLoaders = 4;  // waves that only load

// Columns-per-workgroup factor: the largest of 8, 4, 2, 1 that divides N/16 and leaves at least 160
// workgroups (see gemm_cols_per_block); 1 if there is none.
int qgemm_cols_per_block(int N)
{
    const int nb = N / 16;
    for (int cb = 8; cb > 1; cb >>= 1)
        if (nb % cb == 0 && nb / cb >= 160) return cb;
    return 1;
}

// ------------------------------------------------------------------------------------------------
// Weight quantizer + packer: one thread per (block b, column n).
// Packed layout: workgroup slab (16*cb columns) major, then stage; inside a stage, for column block
// j: 64 lanes x 8 bytes at j*512 (lane = 16*g + column%16 holds the codes of k = 16g .. 16g+15 of the
// stage: dword t = 0,1, byte i = 0..3: low nibble = code of k = 16g + 8t + i, high nibble = code of
// k = 16g + 8t + 4 + i, each stored as q + 8); then at 512*cb the scales, 16 bf16 per column block.
// gate_up_f > 0: packed column 2j is logical column j (gate) and 2j+1 is gate_up_f + j (up).
// rope_d > 0: within every head of rope_d columns, packed columns 2i and 2i+1 are the head's logical columns i
// and i + rope_d/2 (a rotation pair).
__global__ __launch_bounds__(256) void quant_pack_w4_kernel(const uint16_t* __restrict__ W, uint8_t* __restrict__ packed,
                                                            int N, int K, int cb, int gate_up_f, int rope_d)
{
    const int nblk = K >> 6;
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)nblk * N) return;
    const int n = (int)(idx % N), b = (int)(idx / N);
    int nsrc = gate_up_f > 0 ? ((n & 1) ? gate_up_f + (n >> 1) : (n >> 1)) : n;
    if (rope_d > 0) {
        const int r = n % rope_d;
        nsrc = n - r + (r >> 1) + ((r & 1) ? rope_d >> 1 : 0);
    }
    float w[64];
    float amax = 0.0f;
#pragma unroll
    for (int k = 0; k < 64; ++k) {
        w[k] = bf16_to_f32(W[(size_t)(64 * b + k) * N + nsrc]);
        amax = fmaxf(amax, fabsf(w[k]));
    }
    const uint16_t sb = f32_to_bf16_rne(amax / 7.0f);
    const float sf = bf16_to_f32(sb);
    const int slab = n / (16 * cb), j = (n >> 4) % cb, c = n & 15;
    uint8_t* stage = packed + ((size_t)slab * nblk + b) * qstage_w_bytes(cb);
    uint32_t u[64];
#pragma unroll
    for (int k = 0; k < 64; ++k) {
        int v = 0;
        if (sf != 0.0f) {
            const float r = rintf(w[k] / sf);
            v = r < -8.0f ? -8 : (r > 7.0f ? 7 : (int)r);
        }
        u[k] = (uint32_t)(v + 8);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        uint32_t dw[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            uint32_t x = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) x |= (u[16 * g + 8 * t + i] | (u[16 * g + 8 * t + 4 + i] << 4)) << (8 * i);
            dw[t] = x;
        }
        *reinterpret_cast<uint2*>(stage + j * 512 + (16 * g + c) * 8) = make_uint2(dw[0], dw[1]);
    }
    *reinterpret_cast<uint16_t*>(stage + 512 * cb + j * 32 + c * 2) = sb;
}

// Test hook: the packed matrix back to logical codes q [K,N] (int8) and scales s [K/64,N] (bf16).
__global__ __launch_bounds__(256) void quant_unpack_w4_kernel(const uint8_t* __restrict__ packed, int8_t* __restrict__ q,
                                                              uint16_t* __restrict__ s, int N, int K, int cb)
{
    const int nblk = K >> 6;
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)nblk * N) return;
    const int n = (int)(idx % N), b = (int)(idx / N);
    const int slab = n / (16 * cb), j = (n >> 4) % cb, c = n & 15;
    const uint8_t* stage = packed + ((size_t)slab * nblk + b) * qstage_w_bytes(cb);
    for (int g = 0; g < 4; ++g) {
        const uint2 d = *reinterpret_cast<const uint2*>(stage + j * 512 + (16 * g + c) * 8);
        const uint32_t dw[2] = {d.x, d.y};
        for (int t = 0; t < 2; ++t)
            for (int i = 0; i < 4; ++i) {
                const uint32_t byte = (dw[t] >> (8 * i)) & 0xFFu;
                q[(size_t)(64 * b + 16 * g + 8 * t + i) * N + n] = (int8_t)((int)(byte & 15u) - 8);
                q[(size_t)(64 * b + 16 * g + 8 * t + 4 + i) * N + n] = (int8_t)((int)(byte >> 4) - 8);
            }
    }
    s[(size_t)b * N + n] = *reinterpret_cast<const uint16_t*>(stage + 512 * cb + j * 32 + c * 2);
}

// Activation quantizer: one wave per (row, 64-k block); grid (blocks/4, M).  p [M,K] int8 row-major;
// d stored block-major, d[b*ldd + i], so that the scales of a tile's rows for one stage are contiguous.
__global__ __launch_bounds__(256) void quant_act_q8_kernel(const uint16_t* __restrict__ A, int lda, int8_t* __restrict__ p,
                                                           float* __restrict__ d, int ldd, int K)
{
    const int i = blockIdx.y, lane = threadIdx.x & 63;
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= (K >> 6)) return;
    const float a = bf16_to_f32(A[(size_t)i * lda + 64 * b + lane]);
    float amax = fabsf(a);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
    const float df = amax / 127.0f;
    int v = 0;
    if (df != 0.0f) {
        const float r = rintf(a / df);
        v = r < -127.0f ? -127 : (r > 127.0f ? 127 : (int)r);
    }
    p[(size_t)i * K + 64 * b + lane] = (int8_t)v;
    if (lane == 0) d[(size_t)b * ldd + i] = df;
}

// ------------------------------------------------------------------------------------------------
// Schedule of one 256-row tile, worked out on the host (see gemm.hip).
struct qgemm_plan {
    int mrem, RB;
    int SPC;         // stages per chunk
    int slot_bytes;  // bytes of a ring slot
    int nslots, nchunks, last_cnt;
    int tile_bytes;  // bytes of an activation tile: 1024 (16 rows), or 512 / 256 for a single row block of <= 8 / <= 4 rows
    uint32_t inv_4rb;  // floor(2^20/(4*RB))+1
    int nrg;         // row groups in use: min(8/CB, RB)
    int ncomp;       // waves that do not load: one per (column block, row group)
    int nload;
    uint32_t inv_nload;  // floor(2^20/nload)+1
};

static int q_wrun_bytes(int s_cnt, int cb) { return (s_cnt * qstage_w_bytes(cb) + 1023) & ~1023; }

static int up1k(int n) { return (n + 1023) & ~1023; }

// resident: LDS bytes at the end of the ring that hold all activations (the normalizing form); chunks are weights only then
static qgemm_plan make_qgemm_plan(int mrem, int cb, int K, int resident = 0)
{
    qgemm_plan t;
    t.mrem = mrem;
    t.RB = (mrem + 15) >> 4;
    t.tile_bytes = t.RB == 1 ? (mrem <= 4 ? 256 : (mrem <= 8 ? 512 : 1024)) : 1024;
    t.inv_4rb = (1u << 20) / (uint32_t)(4 * t.RB) + 1u;
    // bytes of a chunk of spc stages: weight run, activation tiles, activation scales, each rounded up to 1 KB
    auto chunk_bytes = [&](int spc) {
        return q_wrun_bytes(spc, cb) + (resident ? 0 : up1k(spc * t.RB * t.tile_bytes) + up1k(spc * t.RB * 64));
    };
    const int ring_bytes = kQRing * 1024 - resident;
    const int nstages = K >> 6;
    const int rg = 8 / cb;
    t.nrg = rg < t.RB ? rg : t.RB;
    const int third = ring_bytes / 3;  // the most stages whose chunk fits a third of the ring
    t.SPC = 1;
    while (chunk_bytes(t.SPC + 1) <= third) ++t.SPC;
    t.slot_bytes = chunk_bytes(t.SPC);
    t.nslots = ring_bytes / t.slot_bytes < 4 ? ring_bytes / t.slot_bytes : 4;
    t.nchunks = (nstages + t.SPC - 1) / t.SPC;
    t.last_cnt = nstages - (t.nchunks - 1) * t.SPC;
    t.ncomp = cb * t.nrg;
    t.nload = kQWaves + kQLoaders - t.ncomp;
    t.inv_nload = (1u << 20) / (uint32_t)t.nload + 1u;
    return t;
}

// EPI: the epilogues of the bf16 kernel (plain store, residual add, SwiGLU on gate/up-interleaved columns),
// applied to the accumulator rounded to bf16, so each gives the bytes of the unfused sequence.
// NORM (one tile of at most kFewRows rows, 128-column packings): the rows are raw activations x, which the computing waves normalize
// and quantize while the first weights are on their way (as in qgemm_few.hip, which such packings are too wide for); they stay in
// LDS, [stage][row][64] and [stage][4], and the ring in front of them carries weights only.
template <int CB, int EPI, bool NORM = false>
__global__ __launch_bounds__(64 * (kQWaves + kQLoaders)) void qgemm_kernel(
    const int8_t* __restrict__ qa, int K, const float* __restrict__ da, int ldd, const uint8_t* __restrict__ wp, void* C,
    int ldc, const uint16_t* R, int ldr, int out_f32, qgemm_plan plan_full, qgemm_plan plan_tail, float* qscales_out,
    gemm_rope_args ra, const uint4* __restrict__ x, const uint4* __restrict__ w_norm, float eps)
{
    static_assert(!NORM || CB == 8, "every computing wave has the tile's row block");
    __shared__ uint4 ring[kQRing * 64];
    __shared__ float norm_part[NORM ? 4 * kFewRows : 1];
    __shared__ int normed;
    __shared__ float rowmax[EPI == kEpiSwigluQuant ? 8 * 256 : 1];  // row maxima of the eight waves, that epilogue only
    static_assert(EPI != kEpiSwigluQuant || CB == 8, "a 128-column tile holds one 64-output block per row");
    constexpr int RG = 8 / CB;        // row groups: wave w computes column block w % CB for row group w / CB
    constexpr int MAXR = 16 / RG;     // most row blocks a wave can own
    constexpr int WST = qstage_w_bytes(CB);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, lr = lane & 15;
    const int m0 = blockIdx.y * plan_full.mrem;  // full tiles hold plan_full.mrem rows (256 unless the rows are cut, see launch_qgemm)
    const qgemm_plan& tp = blockIdx.y + 1 == gridDim.y ? plan_tail : plan_full;
    const int mrem = tp.mrem, RB = tp.RB, SPC = tp.SPC, nslots = tp.nslots, nchunks = tp.nchunks;
    const int P = nslots - 1;
    const int nstages = K >> 6;
    const uint32_t ring_addr = (uint32_t)(uintptr_t)(lds_char_t*)ring;
    auto chunk_stages = [&](int c) { return c < nchunks - 1 ? SPC : (c == nchunks - 1 ? tp.last_cnt : 0); };
    // LDS layout of a chunk of s_cnt stages: the weight run (s_cnt*WST bytes as they lie in memory,
    // rounded up to 1 KB), then the activation tiles (stage, row block: rows x 64 codes, the four
    // 16-byte pieces of row i swizzled: piece t at slot t ^ ((i/4)%4)), then the activation scales.
    auto wrun = [&](int s_cnt) { return (uint32_t)((s_cnt * WST + 1023) & ~1023); };
    // The activation tiles of a chunk follow its weight run and the activation scales follow the tiles:
    // tile (stage, row block) has TB bytes (16 rows of 64 codes; a single row block of at most 8 or 4
    // rows keeps only 8 or 4), the scales of a stage are 4 bytes for each of the 16*RB rows.
    const int TB = tp.tile_bytes;
    auto abytes_of = [&](int s_cnt) { return (uint32_t)((s_cnt * RB * TB + 1023) & ~1023); };
    auto sbytes_of = [&](int s_cnt) { return (uint32_t)((s_cnt * RB * 64 + 1023) & ~1023); };
    const int lrc = min(lr, (TB >> 6) - 1);  // row of the tile this lane reads (rows past a short tile repeat its last)

    if (wave >= tp.ncomp) {
        // ---------------------------------------------------------------- loading wave
        const int nload = tp.nload, lrank = wave - tp.ncomp;
        const char* wbytes = reinterpret_cast<const char*>(wp) + (size_t)blockIdx.x * nstages * WST;
        const char* abytes = reinterpret_cast<const char*>(qa) + (size_t)m0 * K;
        const char* dbytes = reinterpret_cast<const char*>(da + m0);
        const uint32_t lane16 = (uint32_t)lane * 16u;
        const int lrow = lane >> 2;  // row of this lane inside an activation tile
        const uint32_t a_lane_off = (uint32_t)lrow * (uint32_t)K + 16u * (uint32_t)((lane & 3) ^ ((lane >> 4) & 3));
        auto strided = [&](int n) { return n > lrank ? (int)(((uint32_t)(n - lrank + nload - 1) * tp.inv_nload) >> 20) : 0; };
        auto loads_for = [&](int s_cnt) {
            return strided((int)(wrun(s_cnt) >> 10)) +
                   (NORM ? 0 : strided((int)(abytes_of(s_cnt) >> 10)) + strided((int)(sbytes_of(s_cnt) >> 10)));
        };
        // short tiles: a load covers 1024/TB stages; lane -> (stage lane/(TB/16), row (lane/4) % (TB/64), piece lane%4)
        const int srow = (lane >> 2) & ((TB >> 6) - 1);
        const int sst = lane / (TB >> 4);
        const uint32_t a_short_off = (uint32_t)srow * (uint32_t)K + 16u * (uint32_t)((lane & 3) ^ ((srow >> 2) & 3)) +
                                     64u * (uint32_t)sst;
        const int loads_full = loads_for(SPC), loads_last = loads_for(tp.last_cnt);
        auto wave_loads = [&](int c) { return c < nchunks - 1 ? loads_full : (c == nchunks - 1 ? loads_last : 0); };

        auto load_chunk = [&](int c, int slot_idx) {
            const int s_cnt = chunk_stages(c);
            if (s_cnt == 0) return;
            const int s0 = c * SPC;
            const uint32_t slot_addr = ring_addr + (uint32_t)slot_idx * (uint32_t)tp.slot_bytes;
            // weight run: 1 KB units of a contiguous byte range; the last unit may be short
            const uint32_t wlen = (uint32_t)(s_cnt * WST);
            const int nwu = (int)(wrun(s_cnt) >> 10);
            const char* wsrc = wbytes + (size_t)s0 * WST;
            // the whole units as one run of loads (three instructions each: the loaders' own instruction
            // stream is on the critical path of small tiles), the short last unit by the wave whose turn it is
            const int nfull = (int)(wlen >> 10);
            dma_run(wsrc, lane16 + (uint32_t)lrank * 1024u, (uint32_t)nload * 1024u, slot_addr + (uint32_t)lrank * 1024u,
                    (uint32_t)nload * 1024u, strided(nfull));
            if (nwu > nfull && nfull - nload * (int)(((uint32_t)nfull * tp.inv_nload) >> 20) == lrank) {
                const uint32_t off = (uint32_t)nfull << 10;
                if (off + lane16 < wlen) dma_block(wsrc + off, lane16, slot_addr + off);
            }
            if constexpr (NORM) return;
            // activation tiles; rows past M load nothing
            const uint32_t tiles = slot_addr + wrun(s_cnt);
            if (TB == 1024) {  // unit (stage, row block)
                int sl = 0, rb = lrank;
                while (rb >= RB) {
                    rb -= RB;
                    ++sl;
                }
                const int nt = s_cnt * RB;
                for (int u = lrank; u < nt; u += nload) {
                    if (16 * rb + lrow < mrem)
                        dma_block(abytes + (size_t)(16 * rb) * K + ((size_t)(s0 + sl) << 6), a_lane_off,
                                  tiles + ((uint32_t)u << 10));
                    rb += nload;
                    while (rb >= RB) {
                        rb -= RB;
                        ++sl;
                    }
                }
            } else {  // one row block of short tiles: unit = 1024/TB stages
                const int spu = 1024 / TB;
                const int nau = (int)(abytes_of(s_cnt) >> 10);
                for (int u = lrank; u < nau; u += nload)
                    if (srow < mrem && u * spu + sst < s_cnt)
                        dma_block(abytes + ((size_t)(s0 + u * spu) << 6), a_short_off, tiles + ((uint32_t)u << 10));
            }
            // activation scales: 16-byte piece p of the chunk's scale area = rows 4w .. 4w+3 of stage p / (4 RB),
            // w = p % (4 RB)
            const uint32_t scales = tiles + abytes_of(s_cnt);
            const int nsu = (int)(sbytes_of(s_cnt) >> 10);
            for (int u = lrank; u < nsu; u += nload) {
                const uint32_t pce = (uint32_t)(64 * u + lane);
                const uint32_t st = (pce * tp.inv_4rb) >> 20;
                const uint32_t w = pce - st * (uint32_t)(4 * RB);
                if ((int)st < s_cnt && (int)(4 * w) < mrem)
                    dma_block(dbytes + (size_t)s0 * ldd * 4, st * (uint32_t)ldd * 4u + 16u * w, scales + ((uint32_t)u << 10));
            }
        };

        if constexpr (NORM) asm volatile("s_barrier" ::: "memory");  // the rows' loads are issued: the memory pipe returns loads in order
        for (int c = 0; c < P; ++c) load_chunk(c, c);
        const int younger_steady = (P - 1) * loads_full;
        int slot_c = 0, slot_new = P;
        for (int c = 0; c < nchunks; ++c) {
            int younger = younger_steady;
            if (c + P > nchunks - 1) {
                younger = 0;
                for (int dd = 1; dd < P; ++dd) younger += wave_loads(c + dd);
            }
            wait_loads_then_barrier(younger);
            load_chunk(c + P, slot_new);
            slot_new = slot_c;
            slot_c = slot_c + 1 == nslots ? 0 : slot_c + 1;
        }
        if constexpr (EPI == kEpiSwigluQuant) __builtin_amdgcn_s_barrier();  // the epilogue's exchange of row maxima
        return;
    }

    // -------------------------------------------------------------------- computing wave
    const int j = wave % CB, rg = wave / CB;  // column block and row group of the wave
    const int cnt = (RB - rg + RG - 1) / RG;  // its row blocks: rg, rg + RG, ... (cnt >= 1 here)

    char* const xres = reinterpret_cast<char*>(ring) + kQRing * 1024 - nstages * (64 * mrem + 16);  // NORM: codes, then scales
    char* const dres = xres + nstages * 64 * mrem;
    const int lrow = min(lr, mrem - 1);
    if constexpr (NORM) {
        // A team of four waves is the 256 threads of rmsnorm_kernel, thread t with the vectors t and t + 256 of a row; team i
        // takes the rows i, i + 2.
        const int team = wave >> 2, vt = tid & 255, nvec = K >> 3;
        uint4 wv[2], xv[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (vt + 256 * i < nvec) wv[i] = w_norm[vt + 256 * i];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (team + 2 * u < mrem && vt + 256 * i < nvec) xv[u][i] = x[(size_t)(team + 2 * u) * nvec + vt + 256 * i];
        if (tid == 0) normed = 0;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (team + 2 * u >= mrem) continue;
            float ss = 0.0f;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (vt + 256 * i < nvec) ss = rms_fold(xv[u][i], ss);
            ss = wave_tree_sum(ss);
            if (lane == 0) norm_part[4 * (team + 2 * u) + (wave & 3)] = ss;
        }
        // the eight computing waves meet (the loading ones are not waited for)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (lane == 0) atomicAdd(&normed, 1);
        await(&normed, 1, kQWaves);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int row = team + 2 * u;
            if (row >= mrem) continue;
            const float a = norm_part[4 * row] + norm_part[4 * row + 2], b = norm_part[4 * row + 1] + norm_part[4 * row + 3];
            const float rs = rms_scale(a + b, K, eps);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int v = vt + 256 * i;
                if (v < nvec) {
                    float df;
                    const uint2 c = quant_vector_q8(rms_apply(xv[u][i], wv[i], rs), df);
                    *reinterpret_cast<uint2*>(xres + ((v >> 3) * mrem + row) * 64 + 8 * (v & 7)) = c;
                    if ((lane & 7) == 0) *reinterpret_cast<float*>(dres + 16 * (v >> 3) + 4 * row) = df;
                }
            }
        }
        // (published by the barrier that opens the first chunk)
    }

    auto run = [&](auto nr_tag) {
        constexpr int NR = decltype(nr_tag)::value;  // cnt rounded up to a power of two; the surplus
                                                     // repeats the last row block and is not stored
        float acc[NR][4];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[r][v] = 0.0f;
        int rbs[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) rbs[r] = rg + RG * (r < cnt ? r : cnt - 1);

        int slot_c = 0;
        for (int c = 0; c < nchunks; ++c) {
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            const int s_cnt = chunk_stages(c);
            const char* slot = reinterpret_cast<const char*>(ring) + (size_t)slot_c * tp.slot_bytes;
            const char* tiles = slot + wrun(s_cnt);
            const char* scales = tiles + abytes_of(s_cnt);
            // UU stages at a time: all their LDS reads and matrix-core instructions first, so that the
            // latencies overlap, then the scaling chain of each output in ascending stage order
            auto stages = [&](int sl, auto uu_tag) {
                constexpr int UU = decltype(uu_tag)::value;
                constexpr int G = NR < 4 ? NR : 4;  // row blocks at a time
                v4i wq[UU];
#pragma unroll
                for (int u = 0; u < UU; ++u)
                    wq[u] = code_bytes(*reinterpret_cast<const uint2*>(slot + (sl + u) * WST + j * 512 + lane * 8));
                // The products d*s of the UU * G tiles, tile u*G + r, as one outer product (as in qgemm_tile_kernel below): this lane's
                // scales are those of tile g.  us against four conversions a stage, a multiply for each output and a load of scales for each
                // tile: 4096 x 28672 16 rows 15.3 -> 14.7, 24 rows 20.2 -> 18.9, 48 rows 29.5 -> 25.8, 64 rows 31.1 -> 27.2; 2048 x 11264
                // 8 rows 7.9 -> 7.4, 48 rows 11.1 -> 10.8; 4096 x 6144 64 rows 16.0 -> 15.4.
                const int ub = sl + min(g / G, UU - 1), rb = g % G;
                const float sa = bf16_to_f32(*reinterpret_cast<const uint16_t*>(slot + ub * WST + 512 * CB + j * 32 + lr * 2));
#pragma unroll
                for (int r0 = 0; r0 < NR; r0 += G) {
                    v4i pr[UU][G];
                    const char* dp = scales + (size_t)ub * RB * 64 + (16 * (rg + RG * min(r0 + rb, cnt - 1)) + lr) * 4;
                    if constexpr (NORM) dp = dres + 16 * (c * SPC + ub) + 4 * lrow;
                    const f32x16 t = __builtin_amdgcn_mfma_f32_16x16x1f32(sa, *reinterpret_cast<const float*>(dp), f32x16{}, 0, 0, 0);
#pragma unroll
                    for (int u = 0; u < UU; ++u)
#pragma unroll
                        for (int r = 0; r < G; ++r) {
                            const char* xp = tiles + (size_t)((sl + u) * RB + rbs[r0 + r]) * TB + 64 * lrc + 16 * (g ^ ((lrc >> 2) & 3));
                            if constexpr (NORM) xp = xres + ((c * SPC + sl + u) * mrem + lrow) * 64 + 16 * g;
                            const v4i xa = *reinterpret_cast<const v4i*>(xp);
                            pr[u][r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wq[u], xa, kProductStart, 0, 0, 0);
                        }
#pragma unroll
                    for (int u = 0; u < UU; ++u)
#pragma unroll
                        for (int r = 0; r < G; ++r)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                acc[r0 + r][v] = __builtin_fmaf(t[4 * (u * G + r) + v], product(pr[u][r][v]), acc[r0 + r][v]);
                }
            };
            constexpr int U = NR == 1 ? 4 : (NR == 2 ? 2 : 1);
            int sl = 0;
            for (; sl + U <= s_cnt; sl += U) stages(sl, std::integral_constant<int, U>{});
            for (; sl < s_cnt; ++sl) stages(sl, std::integral_constant<int, 1>{});
            slot_c = slot_c + 1 == nslots ? 0 : slot_c + 1;
        }

        // Lane holds C[row = 16*rb + lr][n0 + 16j + 4g + v], v = 0..3.
        const int n = blockIdx.x * (16 * CB) + 16 * j + 4 * g;
        if constexpr (EPI == kEpiSwigluQuant) {
            // Columns are gate/up pairs: the lane holds outputs 8j + 2g and 8j + 2g + 1 of the tile's 64, the
            // tile row is one quantization block.  Its maximum: the lane's two values, the four lanes
            // of a row (g), then the eight waves (j) through LDS.  Here CB = 8: every wave owns all
            // row blocks (rbs[r] = r) and all of them take part in the barrier.
            float y[NR][2];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const float g0 = bf16_to_f32(f32_to_bf16_rne(acc[r][0])), u0 = bf16_to_f32(f32_to_bf16_rne(acc[r][1]));
                const float g1 = bf16_to_f32(f32_to_bf16_rne(acc[r][2])), u1 = bf16_to_f32(f32_to_bf16_rne(acc[r][3]));
                y[r][0] = bf16_to_f32(f32_to_bf16_rne(silu_mul(g0, u0)));
                y[r][1] = bf16_to_f32(f32_to_bf16_rne(silu_mul(g1, u1)));
                float mx = fmaxf(fabsf(y[r][0]), fabsf(y[r][1]));
                mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                if (g == 0) rowmax[wave * 256 + 16 * rbs[r] + lr] = mx;
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int rowl = 16 * rbs[r] + lr;
                float amax = rowmax[rowl];
#pragma unroll
                for (int w = 1; w < 8; ++w) amax = fmaxf(amax, rowmax[w * 256 + rowl]);
                const float df = amax / 127.0f;
                uint32_t c2 = 0;
                if (df != 0.0f) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float qv = rintf(y[r][e] / df);
                        const int iv = qv < -127.0f ? -127 : (qv > 127.0f ? 127 : (int)qv);
                        c2 |= (uint32_t)(iv & 0xFF) << (8 * e);
                    }
                }
                if (r < cnt && rowl < mrem) {
                    const size_t row = (size_t)(m0 + rowl);
                    *reinterpret_cast<uint16_t*>(static_cast<int8_t*>(C) + row * ldc + (n >> 1)) = (uint16_t)c2;
                    if (j == 0 && g == 0) qscales_out[(size_t)blockIdx.x * ldr + row] = df;
                }
            }
            return;
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int rowl = 16 * rbs[r] + lr;
            if (r < cnt && rowl < mrem) {
                const size_t row = (size_t)(m0 + rowl);
                const float v[4] = {acc[r][0], acc[r][1], acc[r][2], acc[r][3]};
                if constexpr (EPI == kEpiRopeAppend) {
                    int p = ra.pos[row];
                    p = p < 0 ? 0 : (p >= ra.Lmax ? ra.Lmax - 1 : p);
                    gemm_epilogue_rope_append(v, ra, row, p, ra.slots ? ra.slots[row] : (int)row, n);
                } else {
                    gemm_epilogue_store<EPI>(v, C, ldc, R, ldr, row, n, out_f32);
                }
            }
        }
    };
    // the weight codes of a stage are expanded once per wave whatever the number of row blocks
    if (NORM || cnt == 1) {
        run(std::integral_constant<int, 1>{});
        if constexpr (NORM) return;
    } else if (cnt == 2) {
        run(std::integral_constant<int, 2>{});
    } else if (MAXR >= 4 && cnt <= 4) {
        run(std::integral_constant<int, (MAXR >= 4 ? 4 : MAXR)>{});
    } else if (MAXR >= 8 && cnt <= 8) {
        run(std::integral_constant<int, (MAXR >= 8 ? 8 : MAXR)>{});
    } else {
        run(std::integral_constant<int, MAXR>{});
    }
}

// ------------------------------------------------------------------------------------------------
// The same product for launches of more rows than the kernel above is made for: tiles of 16*RB rows and 64*JB columns, four waves
// side by side of 16*RB rows x 16*JB columns each.  64 x 128 (RB 4, JB 2) where there are enough of them, 64 x 64 and 32 x 64
// below (qgemm_pick).
//
// What bounds the first is the scaling arithmetic: the subtraction that makes the product a float and the fma, a vector instruction
// each for every output and block, a wave having eight 16 x 16 outputs of it a block against eight matrix instructions, and a SIMD's
// vector and matrix instructions add up: 16 clocks each of these, at best 2.3 each of those whatever the waves (measured
// in a loop of nothing else).  The products d*s come from the matrix cores, four tiles' outer products (16 x 16 x 1 of fp32) an
// instruction of 32 clocks, where multiplies would take 42 and eight conversions of scales more; the bits are those of a multiply,
// also where they are subnormal, infinite or NaN.  So a wave and block are some 400 clocks, of which a launch reaches two thirds.  A
// wave owns a tile that is tall: it unpacks the codes of two column blocks for four row blocks.  The operands of two blocks of K (a
// chunk) travel together through a ring of LDS slots, each wave loading its share; activation rows come as whole 128-byte lines.
// Three slots and three workgroups a compute unit (four slots and two workgroups measured 5 to 15 % slower).  Outer products against
// multiplies, us: 1962 rows K x N 2048 x 11264 102.4 -> 99.4, 2048 x 3072 34.1 -> 33.5, 2048 x 2048 and 5632 x 2048 level, 1000 rows of
// 4096 x 6144 60.0 -> 56.9, 256 rows of 4096 x 28672 76.3 -> 73.2.  Against the kernel above: 1962 rows 2048 x 2048 92 -> 23, 5632 x 2048 227
// -> 52, 14336 x 4096 1084 -> 245, 2048 x 11264 160 -> 99, 4096 x 28672 593 -> 465 (0.99 POP/s).
//
// A launch of fewer workgroups than the chip holds takes the time of one walk over K, a chain of 0.2 (32 x 64) to 0.45 us
// (64 x 128) a block: loads' latency where the ring is short (32 x 64 tiles 0.25 us with three slots), one wave's instructions
// otherwise (reading a chunk's operands while the chunk before it is computed gained nothing).  So the smaller the launch, the
// smaller its tile: 4096 x 4096 33.5 -> 19 us at 192 rows, 14336 x 4096 106 -> 57, 5632 x 2048 at 500 rows 43 -> 26.  The 64-column tiles
// read a chunk's operands at once, in front of its arithmetic (with the outer products 100 rows of 4096 x 4096 17.2 -> 15.7 us, of
// 2112 x 4096 10.3 -> 9.6, 300 of 14336 x 4096 71.1 -> 67.4); in 64 x 128 tiles, whose waves are enough to hide the reads, that was up to
// 8 % slower.
// Six and four slots, so that three workgroups of every size fit a compute unit.
constexpr int kTileWaves = 4;
__host__ __device__ constexpr int qtile_slots(int rb, int jb) { return rb * jb == 8 ? 3 : (rb * jb == 4 ? 4 : 6); }

template <int N>
__device__ __forceinline__ void q_wait_then_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <int CB, int EPI, int RB, int JB>
__global__ __launch_bounds__(64 * kTileWaves, 3) void qgemm_tile_kernel(
    const int8_t* __restrict__ qa, int K, const float* __restrict__ da, int ldd, const uint8_t* __restrict__ wp, void* C,
    int ldc, const uint16_t* R, int ldr, int out_f32, int M, float* qscales_out, gemm_rope_args ra)
{
    constexpr int TR = 16 * RB, CBT = kTileWaves * JB, TC = 16 * CBT;  // rows, column blocks and columns of a tile
    constexpr int ABYTES = TR * 128;          // activation codes of a chunk
    constexpr int WBYTES = 2 * CBT * 544;     // weight codes and scales: [slab][block][544 * CB]
    constexpr int SLOT = ABYTES + WBYTES + 2 * TR * 4;  // and activation scales: [block][row]
    constexpr int AU = TR / 8 / kTileWaves;   // loads of activations of a chunk, one wave
    static_assert(CBT % CB == 0 && TR % 32 == 0, "whole slabs, a load of every wave");
    static_assert(EPI != kEpiSwigluQuant || CBT == 8, "a 128-column tile holds one 64-output block per row");
    constexpr int NS = qtile_slots(RB, JB);
    __shared__ uint4 ring[NS * SLOT / 16];
    __shared__ float rowmax[EPI == kEpiSwigluQuant ? kTileWaves * TR : 1];
    constexpr int WST = qstage_w_bytes(CB);  // bytes of a block of a slab
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, lr = lane & 15;
    const int m0 = blockIdx.y * TR, n0 = blockIdx.x * TC;
    const int nblk = K >> 6, nchunks = (nblk + 1) >> 1;
    const uint32_t ring_addr = (uint32_t)(uintptr_t)(lds_char_t*)ring;
    const char* abytes = reinterpret_cast<const char*>(qa);
    const char* wbytes = reinterpret_cast<const char*>(wp) + (size_t)(n0 / 16) * nblk * qstage_w_bytes(1);
    const char* dbytes = reinterpret_cast<const char*>(da);

    // This lane's sources.  Activations, unit u = AU*wave + i: row 8u + lane/8 (rows past M repeat the last), its 16-byte piece
    // (lane%8) ^ (row/2)%8, which spreads the sixteen rows of an operand read over the banks.  Weights, unit u = wave (and wave + 4
    // in 128-column tiles), the last 16*JB pieces by wave 0: piece 64u + lane of the chunk's 272*JB, of slab piece / (68*CB).  Scales
    // (wave 1): block lane / (TR/4), rows 4*(lane % (TR/4)) .. +3.  `odd`: a last chunk of one block repeats that block's bytes.
    uint32_t a_off[2][AU];
    const char* a_base[AU];
#pragma unroll
    for (int i = 0; i < AU; ++i) {
        const int row = 8 * (AU * wave + i) + (lane >> 3), piece = (lane & 7) ^ ((row >> 1) & 7);
        const int first = m0 + 8 * (AU * wave + i);
        a_base[i] = abytes + (size_t)(first < M ? first : M - 1) * K;
        const int src = m0 + row < M ? row : M - 1 - m0;                    // >= 0: a tile holds a row
        const int rel = first < M ? src - 8 * (AU * wave + i) : 0;           // rows from a_base
        a_off[0][i] = (uint32_t)rel * (uint32_t)K + 16u * (uint32_t)piece;
        a_off[1][i] = (uint32_t)rel * (uint32_t)K + 16u * (uint32_t)(piece & 3);
    }
    auto w_source = [&](int unit, bool odd) -> size_t {
        int p = 64 * unit + lane;
        const int slab = p / (68 * CB);
        p -= slab * (68 * CB);
        if (odd && p >= 34 * CB) p -= 34 * CB;
        return (size_t)slab * nblk * WST + 16 * (size_t)p;
    };
    const size_t w_off0 = w_source(wave, false), w_off1 = w_source(wave + 4 * (JB - 1), false), w_off2 = w_source(4 * JB, false);
    const int d_piece = min((m0 >> 2) + (lane & (TR / 4 - 1)), (ldd >> 2) - 1);

    auto issue = [&](int c) {
        const bool odd = 2 * c + 1 == nblk;
        const uint32_t slot = ring_addr + (uint32_t)(c % NS) * (uint32_t)SLOT;
#pragma unroll
        for (int i = 0; i < AU; ++i)
            dma_block(a_base[i] + (size_t)c * 128, a_off[odd ? 1 : 0][i], slot + (uint32_t)(AU * wave + i) * 1024u);
        const uint32_t w = slot + ABYTES;
        const char* wsrc = wbytes + (size_t)c * (2 * WST);
        dma_lane(wsrc + (odd ? w_source(wave, true) : w_off0), w + (uint32_t)wave * 1024u);
        if (JB == 2) dma_lane(wsrc + (odd ? w_source(wave + 4, true) : w_off1), w + (uint32_t)(wave + 4) * 1024u);
        if (wave == 0) {
            if (lane < 16 * JB) dma_lane(wsrc + (odd ? w_source(4 * JB, true) : w_off2), w + 4096u * JB);
        } else if (wave == 1) {
            const int b = 2 * c + lane / (TR / 4);
            if (lane < TR / 2) dma_lane(dbytes + ((size_t)(b < nblk ? b : nblk - 1) * ldd + 4 * (size_t)d_piece) * 4, w + WBYTES);
        }
    };
    constexpr int PER = AU + JB;  // loads of a chunk, one wave; the first two have one more

    f32x4 acc[RB][JB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int j = 0; j < JB; ++j) acc[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int per = wave < 2 ? PER + 1 : PER;
    for (int c = 0; c < NS - 1 && c < nchunks; ++c) issue(c);
    const int zr = (lr >> 1) & 7;
    auto open = [&](int c) __attribute__((always_inline)) {
        // chunk c has landed (here, then everywhere) and everyone is done with chunk c-1
        if (c + NS - 2 < nchunks) {
            if (wave < 2)
                q_wait_then_barrier<(NS - 2) * (PER + 1)>();
            else
                q_wait_then_barrier<(NS - 2) * PER>();
        } else {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wait_loads_then_barrier((nchunks - 1 - c) * per);
        }
        if (c + NS - 1 < nchunks) issue(c + NS - 1);
        return reinterpret_cast<const char*>(ring) + (c % NS) * SLOT;
    };
    // t = d*s of four 16 x 16 tiles by one outer product: of the row blocks of a block of K, or of the two of both blocks of a chunk.
    // Lane (b, i): column i's weight scale and row i's activation scale of tile b; register 4b + v: as register v of tile b's product.
    struct Block {
        uint2 codes[JB];
        float s[JB], d;
        v4i x[RB];
    };
    auto read_scales = [&](const char* slot, int s, Block& b) __attribute__((always_inline)) {
        b.d = *reinterpret_cast<const float*>(slot + ABYTES + WBYTES + s * (TR * 4) + lane * 4);
#pragma unroll
        for (int j = 0; j < JB; ++j) {
            const int cbk = JB * wave + j, st = RB == 4 ? s : lane >> 5;  // cbk: column block of the tile
            const char* wst = slot + ABYTES + (cbk / CB) * (2 * WST) + st * WST;
            b.s[j] = bf16_to_f32(*reinterpret_cast<const uint16_t*>(wst + 512 * CB + (cbk % CB) * 32 + lr * 2));
        }
    };
    auto read_codes = [&](const char* slot, int s, Block& b) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < JB; ++j) {
            const int cbk = JB * wave + j;
            const char* wst = slot + ABYTES + (cbk / CB) * (2 * WST) + s * WST;
            b.codes[j] = *reinterpret_cast<const uint2*>(wst + (cbk % CB) * 512 + lane * 8);
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) b.x[r] = *reinterpret_cast<const v4i*>(slot + (16 * r + lr) * 128 + (((4 * s + g) ^ zr) << 4));
    };
    f32x16 t[JB];
    auto scales = [&](const Block& b) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < JB; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x1f32(b.s[j], b.d, f32x16{}, 0, 0, 0);
    };
    auto products = [&](const Block& b, auto first) __attribute__((always_inline)) {
        constexpr int T0 = 4 * decltype(first)::value;
        v4i wu[JB], pr[RB][JB];
#pragma unroll
        for (int j = 0; j < JB; ++j) wu[j] = code_bytes(b.codes[j]);
#pragma unroll
        for (int r = 0; r < RB; ++r) {
#pragma unroll
            for (int j = 0; j < JB; ++j) pr[r][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wu[j], b.x[r], kProductStart, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int j = 0; j < JB; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[r][j][v] = __builtin_fmaf(t[j][T0 + 4 * r + v], product(pr[r][j][v]), acc[r][j][v]);
    };
    static_assert(RB == 4 || RB == 2, "four tiles an outer product");
    using zeroth = std::integral_constant<int, 0>;
    using second = std::integral_constant<int, RB == 4 ? 0 : 2>;
    for (int c = 0; c < (nblk >> 1); ++c) {
        const char* slot = open(c);
        Block b0, b1;
        if constexpr (JB == 1) {
            read_scales(slot, 0, b0);
            read_codes(slot, 0, b0);
            if constexpr (RB == 4) read_scales(slot, 1, b1);
            read_codes(slot, 1, b1);
            __builtin_amdgcn_sched_barrier(0);
            scales(b0);
            products(b0, zeroth{});
            if constexpr (RB == 4) scales(b1);
            products(b1, second{});
        } else {
            read_scales(slot, 0, b0);
            scales(b0);
            read_codes(slot, 0, b0);
            products(b0, zeroth{});
            read_scales(slot, 1, b1);
            scales(b1);
            read_codes(slot, 1, b1);
            products(b1, zeroth{});
        }
    }
    if (nblk & 1) {
        const char* slot = open(nchunks - 1);
        Block b0;
        read_scales(slot, 0, b0);
        read_codes(slot, 0, b0);
        scales(b0);
        products(b0, zeroth{});
    }

    // Lane holds C[row = m0 + 16r + lr][n0 + 16*JB*wave + 16j + 4g + v].
    const int n = n0 + 16 * JB * wave + 4 * g;
    if constexpr (EPI == kEpiSwigluQuant) {
        // Columns are gate/up pairs: the tile row's 64 outputs are one quantization block; the lane holds four of
        // row lr of each row block.  Its maximum: the lane's, the four lanes of a row (g), the four waves (LDS).
        float y[RB][4];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            float mx = 0.0f;
#pragma unroll
            for (int j = 0; j < JB; ++j)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float gt = bf16_to_f32(f32_to_bf16_rne(acc[r][j][2 * e])), u = bf16_to_f32(f32_to_bf16_rne(acc[r][j][2 * e + 1]));
                    y[r][2 * j + e] = bf16_to_f32(f32_to_bf16_rne(silu_mul(gt, u)));
                    mx = j + e == 0 ? fabsf(y[r][0]) : fmaxf(mx, fabsf(y[r][2 * j + e]));
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            if (g == 0) rowmax[wave * TR + 16 * r + lr] = mx;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int rowl = 16 * r + lr;
            float amax = rowmax[rowl];
#pragma unroll
            for (int w = 1; w < kTileWaves; ++w) amax = fmaxf(amax, rowmax[w * TR + rowl]);
            const float df = amax / 127.0f;
            if (m0 + rowl >= M) continue;
            const size_t row = (size_t)(m0 + rowl);
#pragma unroll
            for (int j = 0; j < JB; ++j) {
                uint32_t c2 = 0;
                if (df != 0.0f) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float qv = rintf(y[r][2 * j + e] / df);
                        const int iv = qv < -127.0f ? -127 : (qv > 127.0f ? 127 : (int)qv);
                        c2 |= (uint32_t)(iv & 0xFF) << (8 * e);
                    }
                }
                *reinterpret_cast<uint16_t*>(static_cast<int8_t*>(C) + row * ldc + ((n + 16 * j) >> 1)) = (uint16_t)c2;
            }
            if (wave == 0 && g == 0) qscales_out[(size_t)blockIdx.x * ldr + row] = df;
        }
    } else {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            if (m0 + 16 * r + lr >= M) continue;
            const size_t row = (size_t)(m0 + 16 * r + lr);
            int p = 0, slot = 0;
            if constexpr (EPI == kEpiRopeAppend) {
                p = ra.pos[row];
                p = p < 0 ? 0 : (p >= ra.Lmax ? ra.Lmax - 1 : p);
                slot = ra.slots ? ra.slots[row] : (int)row;
            }
#pragma unroll
            for (int j = 0; j < JB; ++j) {
                const float v[4] = {acc[r][j][0], acc[r][j][1], acc[r][j][2], acc[r][j][3]};
                if constexpr (EPI == kEpiRopeAppend)
                    gemm_epilogue_rope_append(v, ra, row, p, slot, n + 16 * j);
                else
                    gemm_epilogue_store<EPI>(v, C, ldc, R, ldr, row, n + 16 * j, out_f32);
            }
        }
    }
}

// Rows of the kernel above's tiles.  Matrices too narrow to give every compute unit a column tile: the rows are cut into as many
// tiles as fill the chip (a tile's rows are whole 16-row blocks; which tile a row falls in does not touch its arithmetic).
static int qgemm_tile_rows(int M, int N, int cb)
{
    const int row_blocks = (M + 15) / 16, fit = 256 / (N / (16 * cb));
    if (fit < 2 || row_blocks < 2) return 256;
    const int row_tiles = row_blocks < fit ? row_blocks : fit;
    const int rows = 16 * ((row_blocks + row_tiles - 1) / row_tiles);
    return rows < 256 ? rows : 256;
}

// The kernel and tile of a launch, a function of M, N and the packing (which is one of N).
//   * `rows`, the height of the tiles the kernel above would cut the launch into, decides whether it does: a stage
//     of it takes about 0.0025 us a row from 64 rows on, and a chain of 32 x 64 tiles 0.2 us a block, less against wider
//     packings.  They meet at 90, 65 and 49 rows of 16-, 32- and 64-column packings, with the row block that the kernel above begins
//     there (us there and here): K x N 4096 x 4096 80 rows 15.1 and 15.7, 96 rows 18.5 and 15.6, 14336 x 4096 80 rows 41.6 and 47.6; 4096 x 6144
//     64 rows 14.8 (here 17.4), 65 to 79 rows 19.2 and 17.4, 2048 x 10112 17.8, then 21.9 and 11.7, 14336 x 6144 41.1, then 55.4 and 53.1;
//     2048 x 11264 48 rows 10.0, 49 to 59 rows 11.6 and 10.3, 4096 x 11264 18.6 and 17.4, 2048 x 19968 21.7 and 12.7, 5632 x 12800 24.2 and
//     23.6; the longest K, 14336 x 11264, 52.7 and 53.0.
//     128-column packings have no tile of 64 columns; they meet 64 x 128 tiles between 64 and 96 rows (28672: 31.6 and
//     35.6, 44.8 and 38.5).
//   * The smallest tile of which the chip holds all (768): 2048 x 11264 128 rows, 704 of 32 x 64: 13.2 us against 14.7 in 64 x 64 and
//     18.1 in 64 x 128; 256 rows, 704 of 64 x 64: 19.1 against 24.2 and 22.3; 4096 x 4096 768 rows, 768 of 64 x 64: 34.4 against 43.8
//     and 38.3; 300 rows of 2048 x 11264, 880 of 64 x 64: 26.9 against 23.0 in 64 x 128, which is taken.
enum qgemm_form { kQBase, kQ32x64, kQ64x64, kQ64x128 };
static long long qtiles(int M, int N, int rows, int cols) { return (long long)((M + rows - 1) / rows) * (N / cols); }
static qgemm_form qgemm_pick(int M, int N, int cb)
{
    constexpr int kHeld = 768;
    const int tile_rows = qgemm_tile_rows(M, N, cb), rows = tile_rows < M ? tile_rows : M;
    if (M > 65535 * 64 || N % 64 != 0) return kQBase;
    if (cb == 8) return rows > 80 && qtiles(M, N, 64, 128) >= 256 ? kQ64x128 : kQBase;
    if (rows < (cb == 1 ? 90 : (cb == 2 ? 65 : 49))) return kQBase;
    if (qtiles(M, N, 32, 64) <= kHeld) return kQ32x64;
    return qtiles(M, N, 64, 64) <= kHeld || N % 128 != 0 ? kQ64x64 : kQ64x128;
}

// Where the SwiGLU output is quantized by 64 x 128 tiles rather than in a step of its own behind a product in the form
// above: there are enough of them, and enough rows, that the step (4 to 5 us) costs more than the larger tile.
static bool qgemm_tall_pays(int M, int N)
{
    if (N % 128 != 0 || M > 65535 * 64) return false;
    const long long wgs = qtiles(M, N, 64, 128);
    return (M >= 224 && wgs >= 112) || (M > 128 && wgs >= 256);
}

template <int CB, int EPI, int RB, int JB>
static void launch_qgemm_tile(const void* qa, const void* da, int ldd, const void* wp, void* C, int ldc, const void* R, int ldr,
                              int M, int N, int K, int out_f32, hipStream_t s, float* qscales_out, const gemm_rope_args& ra)
{
    hipLaunchKernelGGL((qgemm_tile_kernel<CB, EPI, RB, JB>), dim3(N / (64 * JB), (M + 16 * RB - 1) / (16 * RB)),
                       dim3(64 * kTileWaves), 0, s, static_cast<const int8_t*>(qa), K, static_cast<const float*>(da), ldd,
                       static_cast<const uint8_t*>(wp), C, ldc, static_cast<const uint16_t*>(R), ldr, out_f32, M, qscales_out,
                       ra);
}

static int q_ldd(int M) { return (M + 3) & ~3; }

template <int CB, int EPI>
static void launch_qgemm(const void* qa, const void* da, int ldd, const void* wp, void* C, int ldc, const void* R, int ldr,
                         int M, int N, int K, int out_f32, hipStream_t s, float* qscales_out = nullptr,
                         const gemm_rope_args& ra = gemm_rope_args{})
{
    if (EPI != kEpiSwigluQuant && qgemm_few_fits(M, CB, K, false)) {
        qgemm_few(EPI, CB, qgemm_few_args{qa, da, wp, C, ldc, R, ldr, M, N, K, out_f32, ra, nullptr, nullptr, 0.0f}, s);
        return;
    }
    const qgemm_form form = qgemm_pick(M, N, CB);
    if (form == kQ64x128) {
        launch_qgemm_tile<CB, EPI, 4, 2>(qa, da, ldd, wp, C, ldc, R, ldr, M, N, K, out_f32, s, qscales_out, ra);
        return;
    }
    if constexpr (CB <= 4) {  // a slab of 128 columns is not cut (qgemm_pick)
        if (form == kQ64x64) {
            launch_qgemm_tile<CB, EPI, 4, 1>(qa, da, ldd, wp, C, ldc, R, ldr, M, N, K, out_f32, s, qscales_out, ra);
            return;
        }
        if (form == kQ32x64) {
            launch_qgemm_tile<CB, EPI, 2, 1>(qa, da, ldd, wp, C, ldc, R, ldr, M, N, K, out_f32, s, qscales_out, ra);
            return;
        }
    }
    const int tile_rows = qgemm_tile_rows(M, N, CB);
    if (qgemm_mid_fits(M, CB, tile_rows)) {
        qgemm_mid(EPI, CB, qgemm_few_args{qa, da, wp, C, ldc, R, ldr, M, N, K, out_f32, ra, nullptr, nullptr, 0.0f}, tile_rows, s);
        return;
    }
    dim3 grid(N / (16 * CB), (M + tile_rows - 1) / tile_rows);
    const qgemm_plan full = make_qgemm_plan(tile_rows, CB, K);
    const qgemm_plan tail = make_qgemm_plan(M - tile_rows * ((M - 1) / tile_rows), CB, K);
    hipLaunchKernelGGL((qgemm_kernel<CB, EPI>), grid, dim3(64 * (kQWaves + kQLoaders)), 0, s,
                       static_cast<const int8_t*>(qa), K, static_cast<const float*>(da), ldd, static_cast<const uint8_t*>(wp),
                       C, ldc, static_cast<const uint16_t*>(R), ldr, out_f32, full, tail, qscales_out, ra, nullptr, nullptr, 0.0f);
}

// N: columns of the packed matrix (2F for the SwiGLU epilogue).
template <int EPI>
static int qgemm_dispatch(const void* codes, const void* scales, const void* packed_w, void* C, int ldc, const void* R,
                          int ldr, int M, int N, int K, int f32, hipStream_t s, const gemm_rope_args& ra = gemm_rope_args{})
{
    switch (qgemm_cols_per_block(N)) {
        case 1: launch_qgemm<1, EPI>(codes, scales, q_ldd(M), packed_w, C, ldc, R, ldr, M, N, K, f32, s, nullptr, ra); break;
        case 2: launch_qgemm<2, EPI>(codes, scales, q_ldd(M), packed_w, C, ldc, R, ldr, M, N, K, f32, s, nullptr, ra); break;
        case 4: launch_qgemm<4, EPI>(codes, scales, q_ldd(M), packed_w, C, ldc, R, ldr, M, N, K, f32, s, nullptr, ra); break;
        default: launch_qgemm<8, EPI>(codes, scales, q_ldd(M), packed_w, C, ldc, R, ldr, M, N, K, f32, s, nullptr, ra); break;
    }
    return check_launch();
}

static bool qgemm_shape_ok(int N, int K) { return N > 0 && K > 0 && N % 16 == 0 && K % 64 == 0 && K <= (1 << 22); }

}  // namespace det

using namespace det;

extern "C" size_t det_qgemm_packed_w_bytes(int N, int K)
{
    if (!qgemm_shape_ok(N, K)) return 0;
    return (size_t)(N / 16) * (K / 64) * qstage_w_bytes(1);
}

extern "C" int det_qgemm_tile(int M, int N, int K, int* columns)
{
    if (M < 1 || !columns || !qgemm_shape_ok(N, K)) return 0;
    const int cb = qgemm_cols_per_block(N);
    switch (qgemm_pick(M, N, cb)) {
        case kQ64x128: *columns = 128; return 64;
        case kQ64x64: *columns = 64; return 64;
        case kQ32x64: *columns = 64; return 32;
        default: *columns = 16 * cb; return qgemm_tile_rows(M, N, cb);
    }
}

static int quant_pack_impl(const void* B_kn, void* packed, int N, int K, int gate_up_f, void* stream, int rope_d = 0)
{
    if (!B_kn || !packed) return DET_EINVAL;
    if (!qgemm_shape_ok(N, K)) return DET_ESHAPE;
    if (!aligned16(packed)) return DET_EALIGN;
    const size_t total = (size_t)N * (K / 64);
    hipLaunchKernelGGL(quant_pack_w4_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<const uint16_t*>(B_kn), static_cast<uint8_t*>(packed), N,
                       K, qgemm_cols_per_block(N), gate_up_f, rope_d);
    return check_launch();
}

extern "C" int det_quant_pack_w4_qkv(const void* B_kn, void* packed, int Hq, int Hkv, int D, int K, void* stream)
{
    if (Hq < 1 || Hkv < 1 || D != 128) return DET_ESHAPE;
    return quant_pack_impl(B_kn, packed, (Hq + 2 * Hkv) * D, K, 0, stream, D);
}

extern "C" int det_quant_pack_w4(const void* B_kn, void* packed, int N, int K, void* stream)
{
    return quant_pack_impl(B_kn, packed, N, K, 0, stream);
}

extern "C" int det_quant_pack_w4_gate_up(const void* B_kn, void* packed, int F, int K, void* stream)
{
    if (F < 1 || F % 8 != 0) return DET_ESHAPE;
    return quant_pack_impl(B_kn, packed, 2 * F, K, F, stream);
}

extern "C" int det_quant_unpack_w4(const void* packed, void* q, void* s, int N, int K, void* stream)
{
    if (!packed || !q || !s) return DET_EINVAL;
    if (!qgemm_shape_ok(N, K)) return DET_ESHAPE;
    const size_t total = (size_t)N * (K / 64);
    hipLaunchKernelGGL(quant_unpack_w4_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<const uint8_t*>(packed), static_cast<int8_t*>(q),
                       static_cast<uint16_t*>(s), N, K, qgemm_cols_per_block(N));
    return check_launch();
}

extern "C" size_t det_quant_act_codes_bytes(int M, int K) { return M > 0 && K > 0 ? (size_t)M * K : 0; }
extern "C" size_t det_quant_act_scales_bytes(int M, int K)
{
    return M > 0 && K > 0 && K % 64 == 0 ? (size_t)q_ldd(M) * (K / 64) * sizeof(float) : 0;
}

extern "C" int det_quant_act_q8(const void* A, int lda, void* codes, void* scales, int M, int K, void* stream)
{
    if (!A || !codes || !scales || M < 1) return DET_EINVAL;
    if (K < 64 || K % 64 != 0 || K > (1 << 22) || M > 65535) return DET_ESHAPE;
    if (lda < K) return DET_EINVAL;
    if (!aligned16(codes) || !aligned16(scales)) return DET_EALIGN;
    hipLaunchKernelGGL(quant_act_q8_kernel, dim3((K / 64 + 3) / 4, M), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const uint16_t*>(A), lda, static_cast<int8_t*>(codes), static_cast<float*>(scales), q_ldd(M),
                       K);
    return check_launch();
}

static int qgemm_args_ok(const void* codes, const void* scales, const void* packed_w, const void* C, int ldc, int M, int N,
                         int ncols_out, int K)
{
    if (!codes || !scales || !packed_w || !C || M < 1) return DET_EINVAL;
    if (!qgemm_shape_ok(N, K)) return DET_ESHAPE;
    if (ldc < ncols_out) return DET_EINVAL;
    if (!aligned16(codes) || !aligned16(scales) || !aligned16(packed_w) || !aligned16(C) || ldc % 4 != 0 || K % 16 != 0)
        return DET_EALIGN;
    return DET_OK;
}

extern "C" int det_qgemm_w4a8(const void* codes, const void* scales, const void* packed_w, void* C, int ldc, int M, int N,
                              int K, int out_dtype, void* stream)
{
    if (out_dtype != DET_BF16 && out_dtype != DET_F32) return DET_EINVAL;
    const int rc = qgemm_args_ok(codes, scales, packed_w, C, ldc, M, N, N, K);
    if (rc != DET_OK) return rc;
    return qgemm_dispatch<kEpiStore>(codes, scales, packed_w, C, ldc, nullptr, 0, M, N, K, out_dtype == DET_F32,
                                     static_cast<hipStream_t>(stream));
}

extern "C" int det_qgemm_w4a8_residual(const void* codes, const void* scales, const void* packed_w, const void* R, int ldr,
                                       void* C, int ldc, int M, int N, int K, void* stream)
{
    const int rc = qgemm_args_ok(codes, scales, packed_w, C, ldc, M, N, N, K);
    if (rc != DET_OK) return rc;
    if (!R || ldr < N) return DET_EINVAL;
    if (!aligned16(R) || ldr % 4 != 0) return DET_EALIGN;
    return qgemm_dispatch<kEpiResidual>(codes, scales, packed_w, C, ldc, R, ldr, M, N, K, 0,
                                        static_cast<hipStream_t>(stream));
}

extern "C" int det_qgemm_w4a8_swiglu(const void* codes, const void* scales, const void* packed_gate_up, void* Y, int ldy,
                                     int M, int F, int K, void* stream)
{
    if (F < 1 || F % 8 != 0 || F > (1 << 29)) return DET_ESHAPE;
    const int rc = qgemm_args_ok(codes, scales, packed_gate_up, Y, ldy, M, 2 * F, F, K);
    if (rc != DET_OK) return rc;
    return qgemm_dispatch<kEpiSwiglu>(codes, scales, packed_gate_up, Y, ldy, nullptr, 0, M, 2 * F, K, 0,
                                      static_cast<hipStream_t>(stream));
}

extern "C" int det_qgemm_w4a8_swiglu_quant_supported(int F, int K)
{
    return F >= 8 && F % 8 == 0 && F <= (1 << 29) && qgemm_shape_ok(2 * F, K) && qgemm_cols_per_block(2 * F) == 8;
}

extern "C" int det_qgemm_w4a8_swiglu_quant(const void* codes, const void* scales, const void* packed_gate_up, void* codes_out,
                                           void* scales_out, int M, int F, int K, void* stream)
{
    if (!scales_out) return DET_EINVAL;
    if (F < 1 || F % 64 != 0 || F > (1 << 29)) return DET_ESHAPE;
    const int rc = qgemm_args_ok(codes, scales, packed_gate_up, codes_out, F, M, 2 * F, F, K);
    if (rc != DET_OK) return rc;
    if (!det_qgemm_w4a8_swiglu_quant_supported(F, K)) return DET_ESHAPE;
    if (!aligned16(scales_out)) return DET_EALIGN;
    // the kernel's ldr argument carries the row stride of the output scales
    launch_qgemm<8, kEpiSwigluQuant>(codes, scales, q_ldd(M), packed_gate_up, codes_out, F, nullptr, q_ldd(M), M, 2 * F, K, 0,
                                     static_cast<hipStream_t>(stream), static_cast<float*>(scales_out));
    return check_launch();
}

// det_qgemm_w4a8_swiglu_quant wherever some kernel's tile row holds whole 64-output blocks (the decoder layer's own
// call; the exported one takes the shapes that do at every row count).
bool det::qgemm_swiglu_quant_fits(int M, int F, int K)
{
    return det_qgemm_w4a8_swiglu_quant_supported(F, K) || (F % 64 == 0 && F <= (1 << 29) && qgemm_tall_pays(M, 2 * F));
}
int det::qgemm_swiglu_quant(const void* codes, const void* scales, const void* packed_gate_up, void* codes_out,
                            void* scales_out, int M, int F, int K, void* stream)
{
    if (det_qgemm_w4a8_swiglu_quant_supported(F, K))
        return det_qgemm_w4a8_swiglu_quant(codes, scales, packed_gate_up, codes_out, scales_out, M, F, K, stream);
    const int rc = qgemm_args_ok(codes, scales, packed_gate_up, codes_out, F, M, 2 * F, F, K);
    if (rc != DET_OK) return rc;
    if (!scales_out) return DET_EINVAL;
    if (!aligned16(scales_out)) return DET_EALIGN;
    const int ld = q_ldd(M);
    hipStream_t s = static_cast<hipStream_t>(stream);
    float* d = static_cast<float*>(scales_out);
    const gemm_rope_args ra{};
    switch (qgemm_cols_per_block(2 * F)) {
        case 1: launch_qgemm_tile<1, kEpiSwigluQuant, 4, 2>(codes, scales, ld, packed_gate_up, codes_out, F, nullptr, ld, M, 2 * F, K, 0, s, d, ra); break;
        case 2: launch_qgemm_tile<2, kEpiSwigluQuant, 4, 2>(codes, scales, ld, packed_gate_up, codes_out, F, nullptr, ld, M, 2 * F, K, 0, s, d, ra); break;
        default: launch_qgemm_tile<4, kEpiSwigluQuant, 4, 2>(codes, scales, ld, packed_gate_up, codes_out, F, nullptr, ld, M, 2 * F, K, 0, s, d, ra); break;
    }
    return check_launch();
}

// Arguments of the fused query/key/value projection; `codes` and `scales` only have to be aligned.
static int qkv_args(const void* codes, const void* scales, const void* packed_qkv, void* qbuf, void* kcache, void* vcache,
                    const int32_t* positions, const int32_t* slots, const float* rope_cos, const float* rope_sin, int M, int Hq,
                    int Hkv, int D, int Lmax, int K, gemm_rope_args& ra)
{
    if (Hq < 1 || Hkv < 1 || D != 128 || Lmax < 1) return DET_ESHAPE;
    const int N = (Hq + 2 * Hkv) * D;
    const int rc = qgemm_args_ok(codes, scales, packed_qkv, qbuf, 4, M, N, 4, K);
    if (rc != DET_OK) return rc;
    if (!kcache || !vcache || !positions || !rope_cos || !rope_sin) return DET_EINVAL;
    if (!aligned16(kcache) || !aligned16(vcache) || !aligned16(rope_cos) || !aligned16(rope_sin)) return DET_EALIGN;
    ra.pos = positions;
    ra.slots = slots;
    ra.cos_t = rope_cos;
    ra.sin_t = rope_sin;
    ra.qbuf = static_cast<uint16_t*>(qbuf);
    ra.kcache = static_cast<uint16_t*>(kcache);
    ra.vcache = static_cast<uint16_t*>(vcache);
    ra.Hq = Hq, ra.Hkv = Hkv, ra.Lmax = Lmax;
    return DET_OK;
}

extern "C" int det_qgemm_w4a8_qkv_rope_append(const void* codes, const void* scales, const void* packed_qkv, void* qbuf,
                                              void* kcache, void* vcache, const int32_t* positions, const int32_t* slots,
                                              const float* rope_cos, const float* rope_sin, int M, int Hq, int Hkv, int D,
                                              int Lmax, int K, void* stream)
{
    gemm_rope_args ra;
    const int rc = qkv_args(codes, scales, packed_qkv, qbuf, kcache, vcache, positions, slots, rope_cos, rope_sin, M, Hq, Hkv, D, Lmax, K, ra);
    if (rc != DET_OK) return rc;
    return qgemm_dispatch<kEpiRopeAppend>(codes, scales, packed_qkv, qbuf, 4, nullptr, 0, M, (Hq + 2 * Hkv) * D, K, 0,
                                          static_cast<hipStream_t>(stream), ra);
}

// The projections behind an RMSNorm on raw rows x [M, K], where one launch does it all (the decoder layer's own calls).
bool det::qgemm_norm_fits(int M, int N, int K)
{
    return M > 0 && qgemm_shape_ok(N, K) && qgemm_few_fits(M, qgemm_cols_per_block(N), K, true);
}
int det::qgemm_norm_qkv_rope_append(const void* x, const void* w_norm, float eps, const void* packed_qkv, void* qbuf, void* kcache,
                                    void* vcache, const int32_t* positions, const int32_t* slots, const float* rope_cos,
                                    const float* rope_sin, int M, int Hq, int Hkv, int D, int Lmax, int K, void* stream)
{
    gemm_rope_args ra;
    const int rc = qkv_args(x, w_norm, packed_qkv, qbuf, kcache, vcache, positions, slots, rope_cos, rope_sin, M, Hq, Hkv, D, Lmax, K, ra);
    if (rc != DET_OK) return rc;
    const int N = (Hq + 2 * Hkv) * D;
    qgemm_few(kEpiRopeAppend, qgemm_cols_per_block(N),
              qgemm_few_args{nullptr, nullptr, packed_qkv, qbuf, 4, nullptr, 0, M, N, K, 0, ra, x, w_norm, eps},
              static_cast<hipStream_t>(stream));
    return check_launch();
}
bool det::qgemm_norm_swiglu_quant_fits(int M, int F, int K)
{
    return M > 0 && M <= kFewRows && K <= 4096 && F % 64 == 0 && det_qgemm_w4a8_swiglu_quant_supported(F, K);
}
int det::qgemm_norm_swiglu_quant(const void* x, const void* w_norm, float eps, const void* packed_gate_up, void* codes_out,
                                 void* scales_out, int M, int F, int K, void* stream)
{
    const int rc = qgemm_args_ok(x, w_norm, packed_gate_up, codes_out, F, M, 2 * F, F, K);
    if (rc != DET_OK) return rc;
    if (!scales_out) return DET_EINVAL;
    if (!aligned16(scales_out)) return DET_EALIGN;
    const qgemm_plan plan = make_qgemm_plan(M, 8, K, (K >> 6) * (64 * M + 16));
    hipLaunchKernelGGL((qgemm_kernel<8, kEpiSwigluQuant, true>), dim3(2 * F / 128), dim3(64 * (kQWaves + kQLoaders)), 0,
                       static_cast<hipStream_t>(stream), nullptr, K, nullptr, 0, static_cast<const uint8_t*>(packed_gate_up), codes_out,
                       F, nullptr, q_ldd(M), 0, plan, plan, static_cast<float*>(scales_out), gemm_rope_args{},
                       static_cast<const uint4*>(x), static_cast<const uint4*>(w_norm), eps);
    return check_launch();
}
int det::qgemm_norm_swiglu(const void* x, const void* w_norm, float eps, const void* packed_gate_up, void* Y, int ldy, int M, int F,
                           int K, void* stream)
{
    const int rc = qgemm_args_ok(x, w_norm, packed_gate_up, Y, ldy, M, 2 * F, F, K);
    if (rc != DET_OK) return rc;
    qgemm_few(kEpiSwiglu, qgemm_cols_per_block(2 * F),
              qgemm_few_args{nullptr, nullptr, packed_gate_up, Y, ldy, nullptr, 0, M, 2 * F, K, 0, gemm_rope_args{}, x, w_norm, eps},
              static_cast<hipStream_t>(stream));
    return check_launch();
}

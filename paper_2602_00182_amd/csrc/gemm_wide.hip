// The bf16 GEMM of gemm.hip for launches of many rows: tiles of 32*RBW rows x 256 columns.  Same packing, same matrix-core
// instruction, one accumulator chain per element over ascending K: the same bytes.
#include "gemm_wide.h"
#include "stream.h"

namespace det {

namespace {

constexpr int kWideCols = 256;
constexpr int kWideWaves = 8;  // two rows of waves x four columns of them; a wave owns 16*RBW rows x 64 columns
constexpr int kWideLds = 160 * 1024;

// This wave's LDS reads have returned.  A builtin, and outside every branch, so that the compiler knows of it and adds no
// wait of its own behind the barrier for reads that were issued before it.
__device__ __forceinline__ void wait_reads()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
}
// At most N of this wave's loads are in flight.
template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Where the four 16-byte pieces of a row lie in its 64 bytes of LDS: piece p of row i at p ^ wide_swizzle(i / 4 % 4).
__device__ __forceinline__ int wide_swizzle(int q) { return (0x78 >> (2 * q)) & 3; }

}  // namespace

// A workgroup's 512 threads stream K in steps of 32 through a ring of LDS slots: 2*RBW KB of activations (16 rows x 64 bytes
// a load) and 16 KB of weights (blocks in operand order) a step, each wave loading its share.  What bounds the
// 256 x 128 tile of gemm.hip is the fill of LDS, 48 KB for 64 * 256 * 128 products; 256 x 256 is 64 KB for twice the work.
// The operands of step t+1 are read from LDS into registers while step t is in the matrix cores, so a step needs no wait for
// its own reads, and its slot is free as soon as it starts.  Reads and loads are dealt out among the products: issued in a row behind
// the barrier they left the matrix cores idle.  Up to 192 rows every second step has a barrier, whose turn it is for the loads of
// the two steps behind it: a barrier a step cost 1 to 4 % (K x N 4096 x 6144, 3302 rows 171 us with both, 158 dealt out, 156 with
// half the barriers; 14336 x 4096, 1500 rows 206, 206, 198).  256-row tiles have one a step: of their five slots a barrier every second
// step leaves a load one to two steps to land in instead of three to four, and where weights come from memory or a round is
// not full that is too short.  129 launches that take them, K = 1024 to 14336, 1.3 % less time with half the barriers than with reads
// and loads in a row, 29 of them more, up to 8 %; 2.9 % less with a barrier a step, none more (4096 x 28672 512 rows 122.3, 128.3, 118.7;
// 4480 x 6400 2041 rows 113.4, 121.0, 110.5; rounds that are nearly full lose 1 to 4 % of their gain, 4096 x 4096 4096 rows 119.9, 115.7,
// 117.6, 10752 x 8192 1656 rows 266, 252, 262).
// Of 160-row tiles' 158 us the products alone take 115, and 133 with no
// loads, 148 with no reads, 151 with no barriers, 155 with no wait for the loads: what is left is the fill, 26 KB a step at 43
// bytes a ns, near what a compute unit gets of data that does not hit in L2 (50 to 55).
template <int RBW, int EPI>
__global__ __launch_bounds__(64 * kWideWaves, 2) void gemm_wide_kernel(const uint16_t* __restrict__ A, int lda,
                                                                     const uint4* __restrict__ Bp, int cb, void* C, int ldc,
                                                                     const uint16_t* R, int ldr, int M, int K, int ntm, int ntn,
                                                                     int out_f32, gemm_rope_args ra)
{
    constexpr int TM = 32 * RBW, AU = TM / 16, UNITS = AU + 16;  // 1 KB loads of a step
    constexpr int SLOT = UNITS * 1024;
    constexpr int NS = kWideLds / SLOT < 6 ? kWideLds / SLOT : 6;
    static_assert(NS >= 4, "ring");
    constexpr int LMAX = (UNITS + kWideWaves - 1) / kWideWaves, LMIN = UNITS / kWideWaves;  // loads of a step, one wave
    static_assert(NS * LMAX <= 60, "load counter");
    constexpr bool kEvery = RBW == 8;  // a barrier a step
    __shared__ uint4 ring[NS * SLOT / 16];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, lr = lane & 15;
    const int wr = wave >> 2, wc = wave & 3;

    // Workgroups go round-robin over the eight XCDs; each XCD gets a run of consecutive tiles, in groups of eight row tiles by
    // all columns, so that the tiles it has at a time share rows and columns in its L2.
    int tm, tn;
    {
        const int T = ntm * ntn, x = blockIdx.x & 7, j = blockIdx.x >> 3;
        const int base = T >> 3, extra = T & 7;
        const int L = x * base + (x < extra ? x : extra) + j;
        const int grp = L / (8 * ntn), in = L - grp * (8 * ntn);
        const int gs = ntm - 8 * grp < 8 ? ntm - 8 * grp : 8;
        tm = 8 * grp + in % gs;
        tn = in / gs;
    }
    const int m0 = tm * TM, n0 = tn * kWideCols;
    const int nst = K >> 5;  // steps, even
    const uint32_t ring_addr = (uint32_t)(uintptr_t)(lds_char_t*)ring;

    // This wave's loads of a step: units wave, wave + 8, ..; below AU activations, above weights (block j = unit - AU of the
    // tile's sixteen).  A load's source is src[i] plus a lane's off[i]; src[i] moves on by inc[i][t & 1] behind step t.
    const char* src[LMAX];
    uint32_t off[LMAX], inc[LMAX][2];
    const int mrem = M - m0;
#pragma unroll
    for (int i = 0; i < LMAX; ++i) {
        const int u = wave + 8 * i;
        if (u < AU) {
            int row = 16 * u + (lane >> 2);
            row = row < mrem ? row : mrem - 1;  // rows past M repeat the last: their outputs are never stored
            src[i] = reinterpret_cast<const char*>(A + (size_t)m0 * lda);
            off[i] = (uint32_t)row * (uint32_t)lda * 2u + 16u * (uint32_t)((lane & 3) ^ wide_swizzle((lane >> 4) & 3));
            inc[i][0] = inc[i][1] = 64;
        } else {
            const int j = u - AU < 16 ? u - AU : 15, slab = j / cb, jj = j - slab * cb;
            src[i] = reinterpret_cast<const char*>(Bp) + ((size_t)(n0 / 16) + (size_t)slab * cb) * (K >> 6) * 2048 + jj * 2048;
            off[i] = (uint32_t)lane * 16u;
            inc[i][0] = 1024, inc[i][1] = (uint32_t)cb * 2048u - 1024u;
        }
    }
    auto issue = [&](int odd, int slot, int i) __attribute__((always_inline)) {
        const int u = wave + 8 * i;
        if (i >= LMIN && u >= UNITS) return;
        dma_block(src[i], off[i], ring_addr + (uint32_t)(slot * SLOT + u * 1024));
        src[i] += inc[i][odd];
    };

    struct Frags {
        bf16x8 w[4], x[RBW];
    };
    const int x_off = (wr * RBW) * 1024 + lr * 64 + ((g ^ wide_swizzle(lr >> 2)) << 4);
    const int w_off = (AU + 4 * wc) * 1024 + lane * 16;
    f32x4 acc[RBW][4];
#pragma unroll
    for (int r = 0; r < RBW; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool more = wave < UNITS % kWideWaves;  // this wave has LMAX loads a step, not LMIN
    // Passing this in front of step t: everyone has the operands of step t in registers, so its slot is free.  With a barrier a step,
    // step t+1 has landed for everyone and the free slot takes step t+NS; else t is even, steps t+1 and t+2 have landed, and the slot and
    // the one before it take the steps t+NS and t+NS-1.
    int slot_r = 1, slot_w = kEvery ? 0 : NS - 1;  // slot of the step read next, and of the step issued next
    constexpr int kBehind = kEvery ? NS - 2 : NS - 4;  // steps behind those, under way
    auto open = [&](bool steady) __attribute__((always_inline)) {
        wait_reads();
        if (!steady)
            wait_loads<0>();
        else if (LMAX != LMIN && more)
            wait_loads<kBehind * LMAX>();
        else
            wait_loads<kBehind * LMIN>();
        asm volatile("s_barrier" ::: "memory");
    };
    // The products of a step (operands f), with the reads of the next step's operands (into nf) and, if `load`, the loads of the
    // step whose slot is free (its parity is that of odd + NS) dealt out among them: after every row block a share.
    auto step = [&](bool load, int odd, const Frags& f, Frags& nf) __attribute__((always_inline)) {
        const char* base = reinterpret_cast<const char*>(ring) + slot_r * SLOT;
#pragma unroll
        for (int r = 0; r < RBW; ++r) {
            constexpr int NR = 4 + RBW;
            const int i0 = NR * r / RBW, i1 = NR * (r + 1) / RBW;
#pragma unroll
            for (int i = i0; i < i1; ++i) {
                if (i < 4)
                    nf.w[i] = *reinterpret_cast<const bf16x8*>(base + w_off + i * 1024);
                else
                    nf.x[i - 4] = *reinterpret_cast<const bf16x8*>(base + x_off + (i - 4) * 1024);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[j], f.x[r], acc[r][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < i1 - i0; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // a matrix-core instruction
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // an LDS read
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < LMAX; ++i)
                if (i * RBW / LMAX == r) {
                    if (load) issue((odd + NS) & 1, slot_w, i);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        slot_r = slot_r + 1 == NS ? 0 : slot_r + 1;
        slot_w = slot_w + 1 == NS ? 0 : slot_w + 1;
    };

#pragma unroll
    for (int t = 0; t < (kEvery ? NS : NS - 1); ++t)
        if (t < nst) {
#pragma unroll
            for (int i = 0; i < LMAX; ++i) issue(t & 1, t, i);
        }
    Frags f0, f1;
    open(true);
    {
        const char* base = reinterpret_cast<const char*>(ring);
#pragma unroll
        for (int j = 0; j < 4; ++j) f0.w[j] = *reinterpret_cast<const bf16x8*>(base + w_off + j * 1024);
#pragma unroll
        for (int r = 0; r < RBW; ++r) f0.x[r] = *reinterpret_cast<const bf16x8*>(base + x_off + r * 1024);
    }
    open(true);
    if constexpr (kEvery) {
        for (int t = 0; t < nst; t += 2) {
            step(t + NS < nst, 0, f0, f1);
            open(t + NS < nst);
            step(t + 1 + NS < nst, 1, f1, f0);  // (past the last step: reads whatever the slot holds, not used)
            if (t + 2 < nst) open(t + 2 + NS - 1 < nst);
        }
    } else {
        for (int t = 0; t < nst; t += 2) {
            step(t - 1 + NS < nst, 1, f0, f1);
            step(t + NS < nst, 0, f1, f0);  // (past the last step: reads whatever the slot holds, not used)
            if (t + 2 < nst) open(t + 2 + NS - 2 < nst);
        }
    }

    // Lane holds C[row = m0 + 16*(wr*RBW + r) + lr][n0 + 64*wc + 16j + 4g + v].
    const int n1 = n0 + 64 * wc + 4 * g;
#pragma unroll
    for (int r = 0; r < RBW; ++r) {
        const int rowl = 16 * (wr * RBW + r) + lr;
        if (rowl >= mrem) continue;
        const size_t row = (size_t)(m0 + rowl);
        int p = 0, slot = 0;
        if constexpr (EPI == kEpiRopeAppend) {
            p = ra.pos[row];
            p = p < 0 ? 0 : (p >= ra.Lmax ? ra.Lmax - 1 : p);
            slot = ra.slots ? ra.slots[row] : (int)row;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float v[4] = {acc[r][j][0], acc[r][j][1], acc[r][j][2], acc[r][j][3]};
            if constexpr (EPI == kEpiRopeAppend)
                gemm_epilogue_rope_append(v, ra, row, p, slot, n1 + 16 * j);
            else
                gemm_epilogue_store<EPI>(v, C, ldc, R, ldr, row, n1 + 16 * j, out_f32);
        }
    }
}

template <int RBW, int EPI>
static void launch(const gemm_wide_args& a, hipStream_t s)
{
    const int ntm = (a.M + 32 * RBW - 1) / (32 * RBW), ntn = a.N / kWideCols;
    hipLaunchKernelGGL((gemm_wide_kernel<RBW, EPI>), dim3(ntm * ntn), dim3(64 * kWideWaves), 0, s,
                       static_cast<const uint16_t*>(a.A), a.lda, static_cast<const uint4*>(a.Bp), a.cb, a.C, a.ldc,
                       static_cast<const uint16_t*>(a.R), a.ldr, a.M, a.K, ntm, ntn, a.out_f32, a.ra);
}

template <int EPI>
static void launch_rows(int rbw, const gemm_wide_args& a, hipStream_t s)
{
    switch (rbw) {
        case 4: launch<4, EPI>(a, s); break;
        case 5: launch<5, EPI>(a, s); break;
        case 6: launch<6, EPI>(a, s); break;
        default: launch<8, EPI>(a, s); break;
    }
}

// What a launch costs is the rounds of 256 workgroups it takes, times what one of its tiles takes for a step of 32 of K, which is
// nearly the same over all shapes (fitted over K = 1024 .. 14336, N = 1024 .. 28672, 256 to 5000 rows; single launches are up to 15 %
// off).  Here 0.45 / 0.54 / 0.60 / 0.78 us for tiles of 128 / 160 / 192 / 256 rows, 0.49 / 0.61 / 0.61 / 0.78 of 128-column packings.  In
// gemm.hip 0.53 us for a 256 x 128 tile (0.51 in launches of four rounds and more), and in its narrower tilings, which it takes where those
// do not fill the chip, 1.4 ns (16- and 32-column
// packings) or 1.18 ns (64-column packings) for each row and column of a tile.  The last row of tiles there is as short as
// its rows: 0.34 of a whole 256 x 128 tile's time and the rest by rows, and it fills the compute units that the last round of
// whole tiles leaves idle.  (Counted as whole tiles, 258 rows of K = 4416, N = 11264 took this form in 62 us instead of 42, 519 rows
// of 2048 x 6144 in 34 instead of 28.)  So the choice is the tile height whose tiles fit the rounds best: 3302 rows of N = 6144,
// K = 4096 are 13 x 48 tiles there (three rounds, 193 us), 13 x 24 of 256 rows here (two), 21 x 24 of 160 rows
// (two, 153 us).  6 % must be won by this count, 21 % where a tile there is as wide as the
// packing and the weights alone are much of the time.  522 random launches that take this form take 19 % less time than in the tilings of
// gemm.hip; 19 of them more, by over 2 %: most are a few rows past whole tiles there and 4 to 10 % slower, three of N = 5632 at 616 to 638
// rows 30 %, since the 64-column tiles have become up to a fifth faster than the 1.4 ns counted for them.  Others: K x N 4096 x 6144
// 700 rows 77 -> 61 us, 14336 x 4096 1500 rows 260 -> 202, 4096 x 28672 4096 rows 955 -> 859 (1.12 PFLOP/s; torch's product of two
// 8192 x 8192 matrices reaches 1.19 on the same card).
namespace {

long long rounds(long long wgs) { return (wgs + 255) / 256; }

// Time of n columns of tiles over M rows, `rows` to a tile; tile(x): time of a tile of x rows.
template <class F>
long long span(int M, int n, int rows, F&& tile)
{
    const int full = (M - 1) / rows, last = 16 * ((M - rows * full + 15) / 16);
    const long long t_full = tile(rows), t_last = tile(last < rows ? last : rows);
    const long long wgs = (long long)n * full, idle = (256 - wgs % 256) % 256;
    const long long rest = n - idle * (t_full / t_last);  // last tiles that do not fit the last round of whole ones
    return rounds(wgs) * t_full + (rest > 0 ? rounds(rest) * t_last : 0);
}

}  // namespace

int gemm_wide_rows(int M, int N, int K, int cb)
{
    if (N % kWideCols != 0 || 16 % cb != 0 || M < 256 || K < 1024) return 0;
    // costs in units of 0.1 ns
    const long long row_tiles = (M + 255) / 256, there = row_tiles * (N / 128);
    long long cost;
    if (there < 256 && cb <= 4) {
        int rows = 256;
        if (cb < 4) {
            const int fit = 256 / (N / 64) > 1 ? 256 / (N / 64) : 1;
            const int even = 16 * (((M + 15) / 16 + fit - 1) / fit);
            rows = even < 256 ? even : 256;
        }
        cost = span(M, N / 64, rows, [&](int x) { return (long long)(x + 64) * (cb < 4 ? 1400 : 1180) / 100; });
    } else {
        const int t = rounds(there) < 4 ? 5300 : 5100;
        cost = span(M, N / 128, 256, [&](int x) { return (long long)t * (34 * 256 + 66 * x) / 25600; });
    }
    static const struct {
        // cost8: 128-column packings.  While 128 rows of those counted 4500 too, launches took them that are faster in other heights or in
        // gemm.hip: 3328 x 25088 1590 rows 316 us instead of 282, 13824 x 27904 1109 rows (now 160) 15 % more.
        int rbw, cost, cost8;
    } kTiles[4] = {{4, 4500, 4900}, {5, 5400, 6060}, {6, 6000, 6060}, {8, 7800, 7800}};
    int best = 0;
    long long best_cost = 100 * cost;
    for (const auto& t : kTiles) {
        const long long n = rounds((long long)((M + 32 * t.rbw - 1) / (32 * t.rbw)) * (N / kWideCols));
        const long long c = cb < 8 ? n * t.cost * 106 : n * t.cost8 * 121;
        if (c < best_cost) best = t.rbw, best_cost = c;
    }
    return best;
}

int gemm_wide(int epi, int rbw, const gemm_wide_args& a, hipStream_t s)
{
    switch (epi) {
        case kEpiStore: launch_rows<kEpiStore>(rbw, a, s); break;
        case kEpiResidual: launch_rows<kEpiResidual>(rbw, a, s); break;
        case kEpiSwiglu: launch_rows<kEpiSwiglu>(rbw, a, s); break;
        default: launch_rows<kEpiRopeAppend>(rbw, a, s); break;
    }
    return check_launch();
}

}  // namespace det

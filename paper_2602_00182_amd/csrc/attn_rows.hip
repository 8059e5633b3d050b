// Attention of many rows that name their cache slots (the tokens of prompts): one workgroup walks the
// chunks of its rows' slot and finishes the rows, with no partials in memory and no second pass.  The
// arithmetic of a (row, head) is that of attn.hip, operation for operation; only where the values live
// and who computes them differs.
#include <math.h>

#include "attn_lane.h"
#include "attn_rows.h"
#include "geometry.h"
#include "internal.h"
#include "stream.h"

namespace det {

namespace {

constexpr int kChunk = 256;   // tokens of a chunk of the canonical order
constexpr int kSub = 64;      // tokens of a staged subtile: 16 KB of K or V, one 64-leaf group of the tree
constexpr int kD = 128;
constexpr int kSlots = 4;     // ring of staged subtiles
constexpr int kTableChunks = 44;  // chunks whose maxima are kept in LDS between the sweeps
// Groups of rows that are not walked (see `few`): pairs, chunks whose sums wait in registers, and chunks in all.
constexpr int kFewPairs = DET_ATTN_FEW_PAIRS, kFewChunks = 8, kFewMax = 80;

// index (in floats) of token tok in pair p's row of e: the row's 16-byte pieces are rotated by p, to spread over the banks
__device__ __forceinline__ int e_index(int p, int tok) { return p * kChunk + ((((tok >> 2) + p) & 63) << 2) + (tok & 3); }

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int N>
__device__ __forceinline__ void wait_then_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

}  // namespace

// One workgroup (256 threads) = 64 / G consecutive rows x the G query heads of one KV head; wave w owns the
// pairs 16w .. 16w+15 from the scores to the output, so that nothing but K, V and the chunk maxima goes
// through LDS.
//
// The rows of a tile that name one slot (a "group") are walked together.  K and V come as subtiles of 64
// tokens x 128 dimensions through a ring of four LDS slots (LDS-DMA, three in flight, one barrier a
// subtile).  Two sweeps: the first takes every chunk's maximum m_c (and with them the row maximum m, which
// the fold needs before its first chunk), the second computes the scores again subtile by subtile, e, l_c and
// O_c, and folds w_c*l_c and w_c*O_c straight into L and O in registers.  The repeated scores are a quarter
// of a chunk's matrix-core work; writing the O_c instead costs 512 bytes out and back per (row, head, chunk).
//
// Registers: the score block of 16 tokens x 16 pairs is computed with the tokens dealt to the operand's rows
// so that a lane ends up with tokens 8g .. 8g+7 of every 32-token step of its pair (g = lane/16): the
// lane's share of the second product's operand.  The 64-leaf trees pair steps (stride 32), lanes
// (16, 8, 2, 1) and registers (4); V^T operands are transposed by the LDS read itself.
//
// Two workgroups a compute unit (243 to 256 registers), so two waves a SIMD.  No unit bounds it alone: on the prompts of 2000 + 1402
// + 1000 tokens below, vector instructions take 48 % of the cycles (about 30 a score, 16 of them exp, 6 the split), the matrix
// cores 24 % (the two of them add up on a SIMD), LDS 15 % (25 with the bank conflicts that the K rows' swizzle took out; 244 -> 237 us), and
// scores, exponentials and weighted sums follow one another inside a wave.  Measured on one layer, against eight rows a workgroup with chunk
// partials in memory and a second pass: prompts of 2000 + 1402 + 1000 tokens, 32/8 heads 1267 -> 237 us; one of 4000 tokens
// 2240 -> 491 us; 24 of 16..512 tokens, 16/4 heads 195 -> 100 us.  Copies cut down from an earlier form that took 297 us on
// prompts of 2000 + 1400 + 1000 tokens: 234 without the exponentials, 109 with the loads and barriers alone.
//
// The grid: `helpers` workgroups, then Hkv per tile, tiles from the last (longest prefixes first).  The (run of rows, KV
// head) items of mixed tiles (attn_rows.h) are dealt out over the helpers, which count them by looking at all rows.  Groups of
// few pairs there take a form of their own (`few`): a walk keeps one wave of four busy on them.  Against eight rows a workgroup,
// 497 rows of as many slots, 32/8 heads: 40 tokens 98 -> 50 us (68 walked), 256 138 -> 92 (149), 1000 498 -> 308 (472),
// 4000 1965 -> 1730 (2040); 961 rows, 16/16 heads: 256 352 -> 319 (555), 1000 1336 -> 1114 (1747).  What bounds `few` is memory from
// a few hundred tokens on (4.9 of 5.2 TB/s in the last case) and about 6 us of each item that its length does not change.
// The form does not pay for 17 to 32 pairs (five to eight rows of four heads), which walk and are the slowest here: 497 rows,
// eight a slot, 32/8 heads, 200 tokens 25 -> 37 us, 1000 108 -> 117, 2048 198 -> 243; 994 rows 46 -> 47, 214 -> 154.
// Deep rows are not touched here.
template <int G, bool QUANT>
__global__ __launch_bounds__(256, 2) void attn_walk_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ kcache,
                                                          const uint16_t* __restrict__ vcache,
                                                          const int32_t* __restrict__ seqlens,
                                                          const int32_t* __restrict__ slots, void* __restrict__ out,
                                                          float* __restrict__ qscales, float* ws_o, int ldd, int R, int Hq,
                                                          int Hkv, int Lmax, int ncmax, int ntiles, int helpers, float scale,
                                                          int len_offset)
{
    constexpr int NP = kWalkPairs;  // pairs of a workgroup: four waves of sixteen
    constexpr int RT = NP / G;   // rows of a tile
    __shared__ uint4 ring[kSlots * 1024];
    __shared__ float mc_table[kTableChunks * NP];
    __shared__ int samples;
    __shared__ uint8_t mixed[1024];  // byte w: the runs of mixed tiles among the rows 64w .. 64w+63

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, lr = lane & 15;
    const int pair = 16 * wave + lr;  // this lane's pair as an operand column
    const uint32_t ring_addr = (uint32_t)(uintptr_t)(lds_char_t*)ring;
    const char* ringc = reinterpret_cast<const char*>(ring);

    // ---- source offsets of this lane's four loads of a subtile: load b of wave w fills rows 16w+4b .. +3 of
    // the subtile (256 bytes each).  The sixteen 16-byte pieces of a row are swizzled by the row, for K so that
    // the operand reads (one piece of sixteen rows), for V so that the transposing reads (one 32-byte unit of
    // sixteen rows) spread over the banks.
    const int sp = lane & 15, rl = lane >> 4;
    auto k_piece = [&](int b) { return sp ^ k_swizzle((2 * wave + (b >> 1)) & 3, rl); };
    auto v_piece = [&](int b) { return (((sp >> 1) ^ (rl | (((b >> 1) & 1) << 2))) << 1) | (sp & 1); };
    // subtile `sub` of K or V (rows past maxlen repeat its last row: K rows there are masked, V rows cleared)
    auto stage = [&](const uint16_t* base, bool is_v, int sub, int maxlen, int slot) __attribute__((always_inline)) {
        const char* src = reinterpret_cast<const char*>(base) + (size_t)sub * (kSub * kD * 2);
        const uint32_t dst = ring_addr + (uint32_t)slot * 16384u + (uint32_t)wave * 4096u;
        const int last = maxlen - 1 - kSub * sub;  // >= 0
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            int row = 16 * wave + 4 * b + rl;
            row = row < last ? row : last;
            const int piece = is_v ? v_piece(b) : k_piece(b);
            dma_block(src, (uint32_t)(row * 256 + piece * 16), dst + (uint32_t)b * 1024u);
        }
    };

    // Products of the K subtile in ring slot `slot` with the queries: acc[st][b][v] = token 32*st + 8g + 4b + v.
    // The operand reads of a 32-token step go out together; its two chains advance in turn.
    auto products = [&](int slot, const uint4 (&qf)[4], f32x4 (&acc)[2][2]) __attribute__((always_inline)) {
        const char* base = ringc + slot * 16384 + (8 * (lr >> 2) + (lr & 3)) * 256;
        const int kz = k_swizzle(lr >> 2, lr & 3);
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            uint4 kf[2][4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    kf[b][i] = *reinterpret_cast<const uint4*>(base + st * 8192 + b * 1024 + (((4 * g + i) ^ kz) << 4));
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[st][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[st][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[b][i]),
                                                                         __builtin_bit_cast(bf16x8, qf[i]), acc[st][b], 0, 0, 0);
        }
    };

    // ---- one group's rows: my_len is the length of this lane's row, 0 where it is not one of them
    auto walk = [&](int kvh, int my_len, int group_slot, int minlen, int maxlen, const uint4 (&qf)[4], float& L,
                    f32x4 (&O)[8]) __attribute__((always_inline)) {
        const size_t kv_base = ((size_t)group_slot * Hkv + kvh) * (size_t)Lmax * kD;
        const uint16_t* kp = kcache + kv_base;
        const uint16_t* vp = vcache + kv_base;
        const int nsub = (maxlen + kSub - 1) / kSub, nchunk = (maxlen + kChunk - 1) / kChunk;
        // The stream of subtiles: K of the first sweep; then K0 V0 K1 V1 .., where the K of a chunk whose maxima do not
        // fit the table go once more in front of its first.
        const int total = 3 * nsub + max(0, nsub - 4 * kTableChunks);
        int i_n = 0, i_sub = 0, i_phase = 0;  // next to issue; phase 0 first sweep, 1 maxima again, 2 K, 3 V
        auto issue = [&]() __attribute__((always_inline)) {
            if (i_n >= total) return;
            stage(i_phase == 3 ? vp : kp, i_phase == 3, i_sub, maxlen, i_n & (kSlots - 1));
            ++i_n;
            if (i_phase == 0) {
                if (++i_sub == nsub) i_sub = 0, i_phase = 2;  // chunk 0 is in the table
            } else if (i_phase == 1) {
                ++i_sub;
                if ((i_sub & 3) == 0 || i_sub == nsub) i_sub = (i_sub - 1) & ~3, i_phase = 2;
            } else if (i_phase == 2) {
                i_phase = 3;
            } else {
                ++i_sub;
                i_phase = (i_sub & 3) == 0 && (i_sub >> 2) >= kTableChunks ? 1 : 2;
            }
        };
        int j = 0;  // next subtile of the stream
        // passing this for subtile j: it has landed for every wave, and every wave is done with subtile j-1, whose
        // slot takes subtile j+3.  A wave's loads of a subtile are always four.
        auto open = [&]() __attribute__((always_inline)) {
            if (j + 2 < total)
                wait_then_barrier<8>();
            else if (j + 1 < total)
                wait_then_barrier<4>();
            else
                wait_then_barrier<0>();
            issue();
        };
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");  // the ring is free, nothing else is in flight
#pragma unroll 1
        for (int i = 0; i < kSlots - 1; ++i) issue();

        // -inf for the tokens past the row's length, of the subtile at t0
        auto mask = [&](f32x4 (&acc)[2][2], int t0) __attribute__((always_inline)) {
            const int lim = my_len - t0 - 8 * g;
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const float a = acc[x >> 3][(x >> 2) & 1][x & 3];
                acc[x >> 3][(x >> 2) & 1][x & 3] = 32 * (x >> 3) + (x & 7) < lim ? a : -INFINITY;
            }
        };
        auto wave_live = [&](int t0) { return __ballot(my_len > t0) != 0; };
        // m_c of chunk c, subtiles j .. of the stream.  Rounding is monotonic, so for a positive scale the largest
        // product times the scale is the largest scaled product.
        const bool scale_last = scale > 0.0f;
        auto chunk_max = [&](int c) __attribute__((always_inline)) -> float {
            float mx = -INFINITY;
            const int ns = min(4, nsub - 4 * c);
#pragma unroll 1
            for (int u = 0; u < ns; ++u, ++j) {
                open();
                const int t0 = kChunk * c + kSub * u;
                if (!wave_live(t0)) continue;
                f32x4 acc[2][2];
                products(j & (kSlots - 1), qf, acc);
                if (!scale_last) {
#pragma unroll
                    for (int x = 0; x < 16; ++x) acc[x >> 3][(x >> 2) & 1][x & 3] *= scale;
                }
                if (t0 + kSub > minlen) mask(acc, t0);
#pragma unroll
                for (int x = 0; x < 16; x += 2)
                    mx = fmaxf(mx, fmaxf(acc[x >> 3][(x >> 2) & 1][x & 3], acc[x >> 3][(x >> 2) & 1][(x & 3) + 1]));
            }
            mx = max_rows(mx);
            return scale_last ? mx * scale : mx;
        };

        float m = -INFINITY;
#pragma unroll 1
        for (int c = 0; c < nchunk; ++c) {
            const float mc = chunk_max(c);
            m = fmaxf(m, mc);
            // (the table's entries of a wave are read by that wave alone)
            if (c < kTableChunks && g == 0) mc_table[c * NP + pair] = mc;
        }

        // Second sweep.
#pragma unroll 1
        for (int c = 0; c < nchunk; ++c) {
            const bool mine = my_len > kChunk * c;
            const float mc = c < kTableChunks ? mc_table[c * NP + pair] : chunk_max(c);
            // a row without tokens in this chunk (other rows of the wave have some): subtracting 0 from -inf gives e = 0
            const float mu = mine ? mc : 0.0f;
            float tree[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            f32x4 acc[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int ns = min(4, nsub - 4 * c);
#pragma unroll 1
            for (int u = 0; u < ns; ++u) {
                const int t0 = kChunk * c + kSub * u;
                const bool live = wave_live(t0);
                float e[2][8];
                open();
                if (live) {
                    f32x4 sc[2][2];
                    products(j & (kSlots - 1), qf, sc);
#pragma unroll
                    for (int x = 0; x < 16; ++x) sc[x >> 3][(x >> 2) & 1][x & 3] *= scale;
                    if (t0 + kSub > minlen) mask(sc, t0);
#pragma unroll
                    for (int x = 0; x < 16; ++x) e[x >> 3][x & 7] = exp_nonpos(sc[x >> 3][(x >> 2) & 1][x & 3] - mu);
                    // the tree over the 64 leaves of this subtile, down to stride 4
                    float a[8];  // stride 32: leaf 8g + k
#pragma unroll
                    for (int k = 0; k < 8; ++k) a[k] = e[0][k] + e[1][k];
                    const float r0 = add32(a[0], a[1]), r1 = add32(a[2], a[3]);  // stride 16
                    const float r2 = add32(a[4], a[5]), r3 = add32(a[6], a[7]);
                    const float t01 = add16(r0, r1), t23 = add16(r2, r3);  // stride 8: rows hold leaves 0 2 1 3 and 4 6 5 7
                    const float t4 = t01 + t23;                            // stride 4
#pragma unroll
                    for (int x = 0; x < 4; ++x) tree[x] = x == u ? t4 : tree[x];
                }
                ++j;
                open();
                const int slot = j & (kSlots - 1);
                ++j;
                const int held = maxlen - t0;  // rows of V that hold tokens: clear the others
                if (held < kSub) {
                    for (int i = tid; i < (kSub - held) * 16; i += 256) ring[slot * 1024 + held * 16 + i] = make_uint4(0, 0, 0, 0);
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                }
                if (!live) continue;
                // The V operands of four 16-wide blocks of d at a time, read while the four before them are in the
                // matrix core: hi of all, then mid, then lo, so that the three products of a chain are four apart.
                const uint32_t base = ring_addr + (uint32_t)slot * 16384u + (uint32_t)(8 * g + (lr >> 2)) * 256u + 8u * (uint32_t)(lr & 3);
                const uint32_t f = (uint32_t)((lr >> 2) | ((g & 1) << 2));
                typedef __attribute__((address_space(3))) short4v lds_short4;
                short4v vt[2][4][2];
                auto read_v = [&](int h) __attribute__((always_inline)) {  // h = 2*st + half of the d blocks
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const uint32_t at = base + (uint32_t)(h >> 1) * 8192u + (((uint32_t)(4 * (h & 1) + x) ^ f) << 5);
                        vt[h & 1][x][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)at);
                        vt[h & 1][x][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)(at + 1024u));
                    }
                };
                bf16x8 piece[3];
                read_v(0);
                split_pieces(e[0], piece);
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    if (h == 2) split_pieces(e[1], piece);
                    if (h < 3) read_v(h + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int y = 0; y < 3; ++y)
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            typedef short short8v __attribute__((ext_vector_type(8)));
                            const bf16x8 vf = __builtin_bit_cast(
                                bf16x8, (short8v)__builtin_shufflevector(vt[h & 1][x][0], vt[h & 1][x][1], 0, 1, 2, 3, 4, 5, 6, 7));
                            f32x4& a = acc[4 * (h & 1) + x];
                            a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, piece[y], a, 0, 0, 0);
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (wave_live(kChunk * c)) {
                const float w0 = add16(tree[0], tree[1]), w1 = add16(tree[2], tree[3]);  // stride 2
                const float z = add32(w0, w1);  // stride 1: row r holds q_r
                const float y = add32(z, z);    // q0+q2, q1+q3
                const float l_c = add16(y, y);
                const float w = det_expf(mc - m);
                const float wl = w * l_c;
                L = mine ? L + wl : L;
#pragma unroll
                for (int db = 0; db < 8; ++db)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float wo = w * acc[db][v];
                        O[db][v] = mine ? O[db][v] + wo : O[db][v];
                    }
            }
        }
    };

    // ---- the rows of a tile: lane i of every wave holds row i's length (0 or less: no tokens) and slot; sets of rows
    // are bit masks
    int tlen = 0, tslot = -1;
    auto with_slot = [&](int sl) -> uint64_t { return __ballot(tlen > 0 && tslot == sl); };
    auto slot_of = [&](int i) -> int { return __builtin_amdgcn_readlane(tslot, i); };
    auto store_pair = [&](int row, int kvh, float L, const f32x4 (&O)[8]) {
        const int h = kvh * G + pair % G;
        if constexpr (!QUANT) {
            uint16_t* orow = static_cast<uint16_t*>(out) + ((size_t)row * Hq + h) * kD + 4 * g;
#pragma unroll
            for (int db = 0; db < 8; ++db)
                *reinterpret_cast<uint2*>(orow + 16 * db) =
                    make_uint2(pack_bf16x2(O[db][0] / L, O[db][1] / L), pack_bf16x2(O[db][2] / L, O[db][3] / L));
        } else {
            int8_t* crow = static_cast<int8_t*>(out) + ((size_t)row * Hq + h) * kD + 4 * g;
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                float y[16], amax = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    y[i] = bf16_to_f32(f32_to_bf16_rne(O[4 * blk + (i >> 2)][i & 3] / L));
                    amax = i == 0 ? fabsf(y[0]) : fmaxf(amax, fabsf(y[i]));
                }
                amax = max_rows(amax);
                const float df = amax / 127.0f;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    uint32_t c4 = 0;
                    if (df != 0.0f) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float r = rintf(y[4 * u + e] / df);
                            const int v = r < -127.0f ? -127 : (r > 127.0f ? 127 : (int)r);
                            c4 |= (uint32_t)(v & 0xFF) << (8 * e);
                        }
                    }
                    *reinterpret_cast<uint32_t*>(crow + 16 * (4 * blk + u)) = c4;
                }
                if (g == 0) qscales[(size_t)(2 * h + blk) * ldd + row] = df;
            }
        }
    };
    // the shortest and the longest of the rows in `members`
    auto length_range = [&](uint64_t members, int& minlen, int& maxlen) {
        if ((members & (members - 1)) == 0) {
            minlen = maxlen = __builtin_amdgcn_readlane(tlen, __builtin_ctzll(members));
            return;
        }
        const bool in = (members >> lane) & 1ull;
        int lo = in ? tlen : 0x7FFFFFFF, hi = in ? tlen : 0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            lo = min(lo, __shfl_xor(lo, off, kWave));
            hi = max(hi, __shfl_xor(hi, off, kWave));
        }
        minlen = uni(lo);
        maxlen = uni(hi);
    };
    auto do_group = [&](int tile, int kvh, int group_slot, uint64_t members, int minlen, int maxlen) __attribute__((always_inline)) {
        const int ri = pair / G, row = tile * RT + ri;
        const int l = __shfl(tlen, ri, kWave);
        const int my_len = ((members >> ri) & 1ull) ? l : 0;
        uint4 qf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) qf[i] = make_uint4(0, 0, 0, 0);
        if (my_len > 0) {
            const uint4* qp = reinterpret_cast<const uint4*>(q + ((size_t)row * Hq + (size_t)kvh * G + pair % G) * kD + 32 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) qf[i] = qp[i];
        }
        float L = 0.0f;
        f32x4 O[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) O[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        walk(kvh, my_len, group_slot, minlen, maxlen, qf, L, O);
        if (my_len > 0) store_pair(row, kvh, L, O);
    };
    // ---- a group of at most kFewPairs pairs, a chunk at a time: wave w takes the scores of subtile w, of all pairs, then dimensions
    // 32w .. 32w+31 of all weighted sums.  K and V are read once: the chunks' sums wait for the row maximum in registers, the newest
    // first, or, of more than kFewChunks chunks, in the workspace, where every lane finds its own again.  K lies in the four
    // slots of the ring, then e in the last and V in the others.
    auto few = [&](int tile, int kvh, int group_slot, uint64_t members, int maxlen) __attribute__((always_inline)) {
        float* es = reinterpret_cast<float*>(ring + 3 * 1024);  // e, [pair][token], e_index
        float* wave_m = mc_table;
        float* wave_l = mc_table + 64;
        float* wave_q = mc_table + 128;
        float* chunk_m = mc_table + 192;  // [chunk][pair], of many chunks
        float* chunk_l = chunk_m + kFewMax * kFewPairs;
        int ri = 0;  // column lr is head lr % G of member lr / G
        {
            uint64_t rest = members;
#pragma unroll
            for (int i = 0; i < kFewPairs / G; ++i) {
                if (rest != 0 && lr / G == i) ri = __builtin_ctzll(rest);
                rest &= rest - 1;
            }
        }
        const int l = __shfl(tlen, ri, kWave);
        const bool in = lr < G * __builtin_popcountll(members);
        const int my_len = in ? l : 0;
        const size_t at = ((size_t)(tile * RT + ri) * Hq + (size_t)kvh * G + lr % G) * kD;
        const size_t kv_base = ((size_t)group_slot * Hkv + kvh) * (size_t)Lmax * kD;
        const uint16_t* kp = kcache + kv_base;
        const uint16_t* vp = vcache + kv_base;
        const int nchunk = (maxlen + kChunk - 1) / kChunk;
        const bool many = nchunk > kFewChunks;
        float* op = ws_o + (at / kD * ncmax) * kD + 32 * wave + 4 * g;  // this lane's sums of the row's first chunk
        uint4 qf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) qf[i] = make_uint4(0, 0, 0, 0);
        f32x4 oc[kFewChunks][2];
        float mc[kFewChunks], lc[kFewChunks];
#pragma unroll
        for (int i = 0; i < kFewChunks; ++i) {
            mc[i] = -INFINITY;
            lc[i] = 0.0f;
            oc[i][0] = oc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll 1
        for (int c = 0; c < nchunk; ++c) {
            const int t0 = kChunk * c, n = min(4, (maxlen - t0 + kSub - 1) / kSub);
            wait_then_barrier<0>();  // the ring is free, nothing else is in flight
#pragma unroll 1
            for (int u = 0; u < n; ++u) stage(kp, false, 4 * c + u, maxlen, u);
            if (c == 0 && in) {
                const uint4* qp = reinterpret_cast<const uint4*>(q + at + 32 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i) qf[i] = qp[i];
            }
            wait_then_barrier<0>();
            float s[2][8];
            float m_c = -INFINITY;
#pragma unroll
            for (int x = 0; x < 16; ++x) s[x >> 3][x & 7] = -INFINITY;
            if (wave < n) {
                f32x4 acc[2][2];
                products(wave, qf, acc);
                const int lim = my_len - t0 - kSub * wave - 8 * g;
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const float a = acc[x >> 3][(x >> 2) & 1][x & 3] * scale;
                    s[x >> 3][x & 7] = 32 * (x >> 3) + (x & 7) < lim ? a : -INFINITY;
                    m_c = fmaxf(m_c, s[x >> 3][x & 7]);
                }
            }
            m_c = max_rows(m_c);
            if (g == 0) wave_m[16 * wave + lr] = m_c;
            lds_barrier();
#pragma unroll 1
            for (int u = 0; u < min(n, 3); ++u) stage(vp, true, 4 * c + u, maxlen, u);
            m_c = fmaxf(fmaxf(wave_m[lr], wave_m[16 + lr]), fmaxf(wave_m[32 + lr], wave_m[48 + lr]));
            // a row without tokens in this chunk (others have some): subtracting 0 from -inf gives e = 0
            const float mu = my_len > t0 ? m_c : 0.0f;
            {
                float a[8];
#pragma unroll
                for (int st = 0; st < 2; ++st)
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        s[st][k] = exp_nonpos(s[st][k] - mu);
                        a[k] = st == 0 ? s[st][k] : a[k] + s[st][k];
                    }
                const float r0 = add32(a[0], a[1]), r1 = add32(a[2], a[3]), r2 = add32(a[4], a[5]), r3 = add32(a[6], a[7]);
                const float t4 = add16(r0, r1) + add16(r2, r3);
                const float t2 = add16(t4, t4);
                const float t1 = add32(t2, t2);
                if (g == 0) wave_l[16 * wave + lr] = t1;
#pragma unroll
                for (int st = 0; st < 2; ++st)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        *reinterpret_cast<float4*>(&es[e_index(lr, kSub * wave + 32 * st + 8 * g + 4 * x)]) =
                            make_float4(s[st][4 * x], s[st][4 * x + 1], s[st][4 * x + 2], s[st][4 * x + 3]);
            }
#pragma unroll
            for (int i = kFewChunks - 1; i > 0; --i) {
                mc[i] = mc[i - 1];
                lc[i] = lc[i - 1];
                oc[i][0] = oc[i - 1][0];
                oc[i][1] = oc[i - 1][1];
            }
            mc[0] = m_c;
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll 1
            for (int u = 0; u < n; ++u) {
                const int behind = (u < 2 ? min(n, 3) : n) - 1 - u;  // subtiles of V in flight behind this one
                if (behind == 2)
                    wait_then_barrier<8>();
                else if (behind == 1)
                    wait_then_barrier<4>();
                else
                    wait_then_barrier<0>();
                if (u == 1 && n == 4) stage(vp, true, 4 * c + 3, maxlen, 0);  // every wave is done with subtile 0
                const int slot = u == 3 ? 0 : u;
                const int held = maxlen - t0 - kSub * u;  // rows of V that hold tokens: clear the others
                if (held < kSub) {
                    for (int i = tid; i < (kSub - held) * 16; i += 256) ring[slot * 1024 + held * 16 + i] = make_uint4(0, 0, 0, 0);
                    lds_barrier();
                }
                const uint32_t base = ring_addr + (uint32_t)slot * 16384u + (uint32_t)(8 * g + (lr >> 2)) * 256u + 8u * (uint32_t)(lr & 3);
                const uint32_t f = (uint32_t)((lr >> 2) | ((g & 1) << 2));
                typedef __attribute__((address_space(3))) short4v lds_short4;
                typedef short short8v __attribute__((ext_vector_type(8)));
#pragma unroll
                for (int st = 0; st < 2; ++st) {
                    const float4 a = *reinterpret_cast<const float4*>(&es[e_index(lr, kSub * u + 32 * st + 8 * g)]);
                    const float4 b = *reinterpret_cast<const float4*>(&es[e_index(lr, kSub * u + 32 * st + 8 * g + 4)]);
                    const float e[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
                    bf16x8 piece[3], vf[2];
                    split_pieces(e, piece);
#pragma unroll
                    for (int x = 0; x < 2; ++x) {
                        const uint32_t from = base + (uint32_t)st * 8192u + (((uint32_t)(2 * wave + x) ^ f) << 5);
                        const short4v v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)from);
                        const short4v v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)(from + 1024u));
                        vf[x] = __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
                    }
#pragma unroll
                    for (int y = 0; y < 3; ++y)
#pragma unroll
                        for (int x = 0; x < 2; ++x) acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[x], piece[y], acc[x], 0, 0, 0);
                }
            }
            lc[0] = (wave_l[lr] + wave_l[32 + lr]) + (wave_l[16 + lr] + wave_l[48 + lr]);
            oc[0][0] = acc[0];
            oc[0][1] = acc[1];
            if (many) {
                if (wave == 0 && g == 0) {
                    chunk_m[c * kFewPairs + lr] = m_c;
                    chunk_l[c * kFewPairs + lr] = lc[0];
                }
                if (my_len > t0) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        float2* dst = reinterpret_cast<float2*>(op + (size_t)c * kD + 16 * u);  // ws_o is only that aligned
                        dst[0] = make_float2(acc[u][0], acc[u][1]);
                        dst[1] = make_float2(acc[u][2], acc[u][3]);
                    }
                }
            }
        }
        // the fold over the chunks, oldest first
        float m = -INFINITY, L = 0.0f;
        f32x4 O[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        auto fold = [&](float m_c, float l_c, const f32x4 (&o)[2]) {
            const float w = det_expf(m_c - m);
            const float wl = w * l_c;
            L = L + wl;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float wo = w * o[u][v];
                    O[u][v] = O[u][v] + wo;
                }
        };
        if (!many) {
#pragma unroll
            for (int i = 0; i < kFewChunks; ++i) m = fmaxf(m, mc[i]);
#pragma unroll
            for (int i = kFewChunks - 1; i >= 0; --i)
                if (i < nchunk && my_len > kChunk * (nchunk - 1 - i)) fold(mc[i], lc[i], oc[i]);
        } else {
            lds_barrier();
            for (int c = 0; c < nchunk; ++c) m = fmaxf(m, chunk_m[c * kFewPairs + lr]);
#pragma unroll 4
            for (int c = 0; kChunk * c < my_len; ++c) {
                f32x4 o[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const float2* src = reinterpret_cast<const float2*>(op + (size_t)c * kD + 16 * u);
                    const float2 a = src[0], b = src[1];
                    o[u] = f32x4{a.x, a.y, b.x, b.y};
                }
                fold(chunk_m[c * kFewPairs + lr], chunk_l[c * kFewPairs + lr], o);
            }
        }
        // lane holds O[d = 32w + 16u + 4g + v][pair lr]
        if constexpr (!QUANT) {
            if (!in) return;
#pragma unroll
            for (int u = 0; u < 2; ++u)
                *reinterpret_cast<uint2*>(static_cast<uint16_t*>(out) + at + 32 * wave + 16 * u + 4 * g) =
                    make_uint2(pack_bf16x2(O[u][0] / L, O[u][1] / L), pack_bf16x2(O[u][2] / L, O[u][3] / L));
        } else {
            float y[8], amax = 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                y[i] = bf16_to_f32(f32_to_bf16_rne(O[i >> 2][i & 3] / L));
                amax = i == 0 ? fabsf(y[0]) : fmaxf(amax, fabsf(y[i]));
            }
            amax = max_rows(amax);
            if (g == 0) wave_q[16 * wave + lr] = amax;
            lds_barrier();
            if (!in) return;
            amax = fmaxf(amax, wave_q[16 * (wave ^ 1) + lr]);  // a block of 64 is two waves' share
            const float df = amax / 127.0f;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                uint32_t c4 = 0;
                if (df != 0.0f) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float r = rintf(y[4 * u + e] / df);
                        const int v = r < -127.0f ? -127 : (r > 127.0f ? 127 : (int)r);
                        c4 |= (uint32_t)(v & 0xFF) << (8 * e);
                    }
                }
                *reinterpret_cast<uint32_t*>(static_cast<int8_t*>(out) + at + 32 * wave + 16 * u + 4 * g) = c4;
            }
            if (g == 0 && (wave & 1) == 0) qscales[(size_t)(2 * (kvh * G + lr % G) + (wave >> 1)) * ldd + tile * RT + ri] = df;
        }
    };
    // A row shorter than its group's longest gives the tokens past its length the weight 0, which keeps them out
    // of its output as long as their V is finite.  If some is not, the group's rows are walked one by one.
    auto window_finite = [&](int kvh, int group_slot, int minlen, int maxlen) {
        if (minlen == maxlen) return true;
        const uint4* vp = reinterpret_cast<const uint4*>(vcache + ((size_t)group_slot * Hkv + kvh) * (size_t)Lmax * kD);
        bool bad = false;
        for (size_t i = (size_t)minlen * 16 + tid; i < (size_t)maxlen * 16; i += 256) {
            const uint4 x = vp[i];
            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                bad = bad || (w[k] & 0x7F80u) == 0x7F80u || (w[k] & 0x7F800000u) == 0x7F800000u;
        }
        return uni(__syncthreads_or(bad)) == 0;
    };
    // f for the group of row `first`: together, or its rows one by one
    auto for_groups = [&](int kvh, int first, auto f) __attribute__((always_inline)) {
        const int group_slot = slot_of(first);
        uint64_t rest = with_slot(group_slot);
        int minlen, maxlen;
        length_range(rest, minlen, maxlen);
        const bool together = window_finite(kvh, group_slot, minlen, maxlen);
#pragma unroll 1
        while (rest != 0) {
            const uint64_t members = together ? rest : rest & (~rest + 1);
            if (!together) length_range(members, minlen, maxlen);
            f(group_slot, members, minlen, maxlen);
            rest &= ~members;
        }
    };

    // ---- what this workgroup walks: the groups of its tile and KV head, or a helper's share of the mixed tiles'
    int limit = kWalkChunks;
    uint64_t lead = 0;  // the first rows of the tile's groups that walk
    auto load_tile = [&](int tile) __attribute__((always_inline)) {
        const int r = tile * RT + lane;
        tlen = 0;
        tslot = -1;
        if (lane < RT && r < R) {
            tlen = attn_row_len(seqlens, r, len_offset, Lmax);
            tslot = slots[r];
        }
    };
    auto classify = [&]() __attribute__((always_inline)) -> bool {  // whether the tile is mixed
        const attn_row_classes k = attn_classify_rows<RT>(tlen, tslot, limit);
        if ((k.deep >> lane) & 1ull) tlen = 0;
        lead = 0;
        for (uint64_t rest = __ballot(tlen > 0); rest != 0;) {
            const int f = __builtin_ctzll(rest);
            lead |= 1ull << f;
            rest &= ~with_slot(slot_of(f));
        }
        return k.mixed != 0;
    };
    const bool helper = (int)blockIdx.x < helpers;
    int tile = 0, kvh = 0, first = 0;  // the current item
    int word = 0, items = 0, item = 0;  // a helper's word, the items of the word, and its current one among them
    auto rewind = [&]() {
        word = 0;
        items = uni((int)mixed[0]) * Hkv;
        item = (int)blockIdx.x - helpers;
    };
    if (!helper) {
        const int i = (int)blockIdx.x - helpers;
        kvh = i % Hkv;
        tile = ntiles - 1 - i / Hkv;
        load_tile(tile);
        const int ri = pair / G, row = tile * RT + ri;
        const int l = __shfl(tlen, ri, kWave);
        if (row < R && l <= 0) {  // rows without tokens: zeros
            f32x4 O[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) O[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            store_pair(row, kvh, 1.0f, O);
        }
        if (__ballot(tlen > kWalkChunks * kChunk) != 0)  // the same in every wave
            limit = attn_walk_limit(seqlens, len_offset, Lmax, R, ntiles, RT, Hkv, &samples);
        if (classify()) return;
    } else {
        if (Lmax > kWalkChunks * kChunk) limit = attn_walk_limit(seqlens, len_offset, Lmax, R, ntiles, RT, Hkv, &samples);
        attn_for_row_words<RT>(seqlens, slots, len_offset, Lmax, R, limit, [&](int w, const attn_row_classes& k) {
            if (lane == 0) mixed[w] = (uint8_t)__builtin_popcountll(k.starts & k.mixed);
        });
        __syncthreads();
        rewind();
    }
    // Moves to the next item; false: none left.  A word of 64 rows has Hkv items for each run of its mixed tiles; the items of
    // all words in ascending order are dealt round-robin over the helpers.  (Dealt by row instead of by run, regular slots put
    // all the work on a few helpers: 962 rows, eight a slot at 400 tokens, 32/16 heads 911 us instead of 134.)
    auto advance = [&]() __attribute__((always_inline)) -> bool {
        if (!helper) {
            if (lead == 0) return false;
            first = __builtin_ctzll(lead);
            lead &= lead - 1;
            return true;
        }
        for (;;) {
            item += helpers;
            while (item >= items) {
                item -= items;
                if (++word >= (R + 63) / 64) return false;
                items = uni((int)mixed[word]) * Hkv;
            }
            const int r = 64 * word + lane;
            const int l = r < R ? attn_row_len(seqlens, r, len_offset, Lmax) : 0;
            const int sl = r < R ? slots[r] : -1;
            const attn_row_classes k = attn_classify_rows<RT>(l, sl, limit);
            uint64_t starts = k.starts & k.mixed;
            for (int n = item / Hkv; n > 0; --n) starts &= starts - 1;
            const int bit = __builtin_ctzll(starts);
            kvh = item % Hkv;
            tile = (64 * word + bit) / RT;
            first = bit % RT;
            const int from = (bit & ~(RT - 1)) + (lane & (RT - 1));  // lane i takes row i of the tile
            tslot = __shfl(sl, from, kWave);
            tlen = __shfl(l, from, kWave);
            if (lane >= RT || ((k.walks >> from) & 1ull) == 0) tlen = 0;
            // a slot's later runs went with its first
            if (__builtin_ctzll(with_slot(slot_of(first))) == first) return true;
        }
    };
    auto is_few = [&](int first) -> bool {
        const uint64_t members = with_slot(slot_of(first));
        if (G * __builtin_popcountll(members) > kFewPairs) return false;
        int minlen, maxlen;
        length_range(members, minlen, maxlen);
        return maxlen <= kFewMax * kChunk;
    };
    if (helper) {  // the groups of few pairs in a loop of their own: what the two forms keep in registers does not fit together
        bool others = false;
#pragma unroll 1
        while (advance()) {
            if (is_few(first))
                for_groups(kvh, first, [&](int group_slot, uint64_t members, int, int maxlen) __attribute__((always_inline)) {
                    few(tile, kvh, group_slot, members, maxlen);
                });
            else
                others = true;
        }
        if (!others) return;
        rewind();
    }
#pragma unroll 1
    while (advance())
        if (!helper || !is_few(first))
            for_groups(kvh, first, [&](int group_slot, uint64_t members, int minlen, int maxlen) __attribute__((always_inline)) {
                do_group(tile, kvh, group_slot, members, minlen, maxlen);
            });
}

// (row tile, KV head) workgroups of a launch
long long attn_walk_workgroups(int R, int G, int Hkv)
{
    const int RT = kWalkPairs / G;
    return (long long)((R + RT - 1) / RT) * Hkv;
}

template <int G>
static void launch_walk(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens, const int32_t* slots,
                        int len_offset, void* out, float* qscales, float* ws_o, int R, int Hq, int Hkv, int Lmax, int ncmax,
                        float scale, hipStream_t s)
{
    constexpr int RT = kWalkPairs / G;
    const int ntiles = (R + RT - 1) / RT, ldd = (R + 3) & ~3;
    // Helpers: two a compute unit, a multiple of the eight XCDs so that a KV head's tiles stay on their XCDs.
    const int helpers = 512;
    const dim3 grid((unsigned)(helpers + ntiles * Hkv));
    const uint16_t *qq = static_cast<const uint16_t*>(q), *kk = static_cast<const uint16_t*>(kcache),
                   *vv = static_cast<const uint16_t*>(vcache);
    if (qscales)
        hipLaunchKernelGGL((attn_walk_kernel<G, true>), grid, dim3(256), 0, s, qq, kk, vv, seqlens, slots, out, qscales, ws_o,
                           ldd, R, Hq, Hkv, Lmax, ncmax, ntiles, helpers, scale, len_offset);
    else
        hipLaunchKernelGGL((attn_walk_kernel<G, false>), grid, dim3(256), 0, s, qq, kk, vv, seqlens, slots, out, qscales, ws_o,
                           ldd, R, Hq, Hkv, Lmax, ncmax, ntiles, helpers, scale, len_offset);
}

int attn_walk(const void* q, const void* kcache, const void* vcache, const int32_t* seqlens, const int32_t* slots,
              int len_offset, void* out, float* qscales, float* ws_o, int R, int Hq, int Hkv, int Lmax, int ncmax, float scale,
              hipStream_t s)
{
#define DET_LAUNCH_WALK(GG) \
    launch_walk<GG>(q, kcache, vcache, seqlens, slots, len_offset, out, qscales, ws_o, R, Hq, Hkv, Lmax, ncmax, scale, s)
    switch (Hq / Hkv) {
        case 1: DET_LAUNCH_WALK(1); break;
        case 2: DET_LAUNCH_WALK(2); break;
        case 4: DET_LAUNCH_WALK(4); break;
        default: DET_LAUNCH_WALK(8); break;
    }
#undef DET_LAUNCH_WALK
    return check_launch();
}

}  // namespace det

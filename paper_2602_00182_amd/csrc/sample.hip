// Seeded temperature / top-k / top-p sampling in a canonical iteration order (the paper's section
// 6.6: a fixed-seed PRNG and a canonical order make the emitted token a function of (seed, decode
// policy) alone).  One 256-thread workgroup per row.
//
//   z_j = logits_j / T (NaN counts as -inf, -0 as +0);  candidates ordered by (z descending, index
//   ascending);  the first k = min(top_k, V) kept;  e_i = det_expf(z_i - z_0);  c_i = c_{i-1} + e_i
//   in rank order, sequential fp32 adds from +0;  n = smallest i+1 with c_i >= top_p * c_{k-1};
//   u = counter-based uniform of (seed, sequence id, step);  target = u * c_{n-1};  the token is the
//   candidate of the smallest rank i < n with c_i > target (rank n-1 if rounding leaves none).
//
// The order is total (index breaks ties), so the k kept candidates and their ranks are unique and any
// selection / sorting network gives them: here an 8-bit radix select on the 64-bit key
// (order-preserving image of z, then ~index) with integer LDS histograms, and a bitonic sort of the
// k survivors.  The prefix sums are one thread's adds in rank order.  sample_kernel reads the row once
// per radix pass and serves any V; sample_kernel_reg (rows of at most 65536 logits) keeps the keys in
// registers and takes wider digits.
#include <math.h>

#include "common.h"

namespace det {

constexpr int kMaxTopK = 1024;

// Order-preserving map fp32 -> uint32 (larger float, larger key) and its inverse.
__device__ __forceinline__ uint32_t order_key(float z)
{
    const uint32_t u = __float_as_uint(z);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float order_key_inv(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// order_key with NaN = -inf and -0 = +0: the same candidate value has the same key.
__device__ __forceinline__ uint32_t value_key(float z)
{
    if (z != z) z = -INFINITY;
    if (z == 0.0f) z = 0.0f;
    return order_key(z);
}
__device__ __forceinline__ uint64_t candidate_key(float logit, float temperature, int j)
{
    return ((uint64_t)value_key(logit / temperature) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)j);
}

__device__ __forceinline__ uint64_t splitmix64_mix(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(256) void sample_kernel(const float* __restrict__ logits, int V, float temperature,
                                                     int top_k, float top_p, uint64_t seed,
                                                     const int32_t* __restrict__ seq_ids,
                                                     const int32_t* __restrict__ steps,
                                                     int32_t* __restrict__ tokens)
{
    __shared__ uint32_t hist[256];
    __shared__ uint64_t sel[kMaxTopK];
    __shared__ float ebuf[kMaxTopK];
    __shared__ int s_digit, s_need, s_bin, s_count;

    const int tid = threadIdx.x;
    const float* row = logits + (size_t)blockIdx.x * V;
    const int k = top_k < V ? top_k : V;

    // ---- radix select: the k-th largest key, 8 bits per pass from the top
    uint64_t prefix = 0;   // decided top bits of the k-th largest key
    int need = k;          // rank still to be found among the keys that share the prefix
    int shift = 56;
    bool all_of_bin = false;
    for (int pass = 0; pass < 8; ++pass, shift -= 8) {
        hist[tid] = 0;
        __syncthreads();
        for (int j = tid; j < V; j += 256) {
            const uint64_t key = candidate_key(row[j], temperature, j);
            if (pass == 0 || (key >> (shift + 8)) == prefix) atomicAdd(&hist[(uint32_t)(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        uint32_t above = 0;  // keys with the prefix and a larger digit than tid
        for (int b = tid + 1; b < 256; ++b) above += hist[b];
        const uint32_t mine = hist[tid];
        if ((int)above < need && need <= (int)(above + mine)) {
            s_digit = tid;
            s_need = need - (int)above;
            s_bin = (int)mine;
        }
        __syncthreads();
        prefix = (prefix << 8) | (uint64_t)s_digit;
        need = s_need;
        all_of_bin = s_bin == need;  // every key of this bin is wanted: no need to look at lower bits
        __syncthreads();
        if (all_of_bin) break;
    }
    const uint64_t threshold = all_of_bin ? (prefix << shift) : prefix;

    // ---- gather the k survivors (any order), pad to a power of two, sort descending
    if (tid == 0) s_count = 0;
    __syncthreads();
    for (int j = tid; j < V; j += 256) {
        const uint64_t key = candidate_key(row[j], temperature, j);
        if (key >= threshold) sel[atomicAdd(&s_count, 1)] = key;
    }
    int kp = 1;
    while (kp < k) kp <<= 1;
    __syncthreads();
    for (int i = k + tid; i < kp; i += 256) sel[i] = 0;  // below every real key
    __syncthreads();
    for (int size = 2; size <= kp; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < (kp >> 1); i += 256) {
                const int lo = 2 * i - (i & (stride - 1));
                const int hi = lo + stride;
                const bool desc = (lo & size) == 0;
                const uint64_t a = sel[lo], b = sel[hi];
                if ((a < b) == desc) {
                    sel[lo] = b;
                    sel[hi] = a;
                }
            }
            __syncthreads();
        }
    }

    // ---- probabilities in rank order
    const float z0 = order_key_inv((uint32_t)(sel[0] >> 32));
    for (int i = tid; i < k; i += 256) ebuf[i] = det_expf(order_key_inv((uint32_t)(sel[i] >> 32)) - z0);
    __syncthreads();
    if (tid == 0) {
        float acc = 0.0f;
        for (int i = 0; i < k; ++i) {
            acc = acc + ebuf[i];
            ebuf[i] = acc;  // c_i
        }
        const float cut = top_p * ebuf[k - 1];
        int n = k;
        for (int i = 0; i < k; ++i)
            if (ebuf[i] >= cut) {
                n = i + 1;
                break;
            }
        const uint64_t ctr = ((uint64_t)(uint32_t)seq_ids[blockIdx.x] << 32) | (uint64_t)(uint32_t)steps[blockIdx.x];
        const uint64_t r = splitmix64_mix(seed + (ctr + 1) * 0x9E3779B97F4A7C15ull);
        const float u = (float)(uint32_t)(r >> 40) * 0x1p-24f;
        const float target = u * ebuf[n - 1];
        int pick = n - 1;
        for (int i = 0; i < n; ++i)
            if (ebuf[i] > target) {
                pick = i;
                break;
            }
        tokens[blockIdx.x] = (int32_t)(0xFFFFFFFFu - (uint32_t)sel[pick]);
    }
}

// The same selection for rows of at most 1024*KPT logits, with the row read once: 1024 threads, each
// keeps the keys of its KPT candidates in registers, so that what follows touches no memory but LDS.  VEC: rows of 16-byte
// pieces, which are loaded as such.  The prefix sums are sequential adds in rank order (their order is part of the definition); the
// two searches over them take the first index that satisfies a condition, which does not depend on how it is found.
//
// Up to top-k 256 the candidates come from group maxima: at least k of G groups of threads hold a logit that is at least the k-th
// largest of the groups' largest logits, so that value bounds the k-th largest logit of the row from below, and with G of
// two to four times k few more than k logits reach it (of 32000 normal ones some 65 for k = 50).  Dividing by a finite temperature keeps
// the order up to ties, so only the logits that may reach the bound's quotient are divided.
// What bounds it is one chain in one workgroup a row: the row's 128 KB (9 us of 16 with loads of four bytes and a division for
// each logit), then steps that wait for LDS.  64 rows of 32000, us before (the k-th largest of the threads' maxima by two
// histograms, every logit divided, sums and searches through LDS with a barrier each) and now: top-k 1 17.9 -> 9.4, 50 20.7 -> 11.7,
// 64 21.4 -> 12.1, 100 to 128 25 -> 20, 256 34 -> 28, 1000 51 -> 50; of 8000 at 40 12.4 -> 6.3, of 50000 at 50 36 -> 27.
// A row where more than kMaxRanked keys reach the bound (ties) has paid for the bound in vain and is selected by radix.
constexpr int kSampleThreads = 1024;
constexpr int kBoundTopK = 256, kGroupTopK = 128, kMaxRanked = 512;

// The value of the lane N away inside a group of 2, 4, 8 or 16 lanes whose halves each agree on their value (xor 1, xor 2, and mirror
// images of the group of 8 and of 16).
template <int N>
__device__ __forceinline__ int other_half(int v)
{
    constexpr int ctrl = N == 1 ? 0xB1 : (N == 2 ? 0x4E : (N == 4 ? 0x141 : 0x140));
    return __builtin_amdgcn_update_dpp(0, v, ctrl, 0xF, 0xF, true);
}
template <int KPT, bool VEC>
__global__ __launch_bounds__(kSampleThreads) void sample_kernel_reg(const float* __restrict__ logits, int V,
                                                                    float temperature, int top_k, float top_p,
                                                                    uint64_t seed, const int32_t* __restrict__ seq_ids,
                                                                    const int32_t* __restrict__ steps,
                                                                    int32_t* __restrict__ tokens)
{
    constexpr int T = kSampleThreads;
    __shared__ uint32_t hist2[2][2 * kSampleThreads];  // the histogram of pass p is hist2[p & 1]; the other one is cleared meanwhile
    __shared__ uint64_t sel[kMaxTopK], cand[kMaxRanked];
    __shared__ uint4 maxima[kSampleThreads / 4 / 4];
    __shared__ uint32_t s_bound;
    __shared__ __align__(16) float ebuf[kMaxTopK];
    __shared__ int s_digit, s_need, s_bin, s_count, s_n, s_pick;
    __shared__ float s_cut, s_target;
    __shared__ uint32_t wave_tot[kSampleThreads / kWave];

    const int tid = threadIdx.x;
    const float* row = logits + (size_t)blockIdx.x * V;
    const int k = top_k < V ? top_k : V;

    const uint64_t ctr = ((uint64_t)(uint32_t)seq_ids[blockIdx.x] << 32) | (uint64_t)(uint32_t)steps[blockIdx.x];

    auto index_of = [&](int i) { return VEC ? 4 * (tid + T * (i >> 2)) + (i & 3) : tid + T * i; };
    // Keys of the logits as long as `divided` is false, then those of their quotients (the high half of candidate_key; the low half is
    // 0xFFFFFFFF - index).  An absent one is 0, below every real one.
    uint32_t zk[KPT];
    constexpr bool kLate = KPT <= 32;  // (of 64 a thread they are divided first: keys and divisions do not fit the registers)
    bool divided = !kLate || k > kBoundTopK;
    {
        float x[KPT];
        if constexpr (VEC) {
#pragma unroll
            for (int i = 0; i < KPT; i += 4) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (index_of(i) < V) v = reinterpret_cast<const float4*>(row)[tid + T * (i >> 2)];
                x[i] = v.x, x[i + 1] = v.y, x[i + 2] = v.z, x[i + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < KPT; ++i) x[i] = index_of(i) < V ? row[index_of(i)] : 0.0f;
        }
        if (divided) {
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                x[i] = x[i] / temperature;
                if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < KPT; ++i) zk[i] = index_of(i) < V ? value_key(x[i]) : 0u;
    }
    auto divide = [&]() {
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            zk[i] = zk[i] != 0 ? value_key(order_key_inv(zk[i]) / temperature) : 0u;
            if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // (all divisions side by side do not fit the registers)
        }
        divided = true;
    };
    auto key_of = [&](int i) { return ((uint64_t)zk[i] << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)index_of(i)); };

    // The digit of the rank-`need` key of a 2048-bin histogram (thread t owns bins 2t and 2t+1): above(b) = keys with a
    // larger digit than b, from the suffix sums of the threads' pair sums inside each wave and the totals of the higher waves.
    // Leaves s_digit, s_need (the rank left inside the bin) and s_bin; `between` runs before its second barrier.
    auto find_digit = [&](const uint32_t* hist, int need, auto between) {
        const uint32_t h_lo = hist[2 * tid], h_hi = hist[2 * tid + 1];
        uint32_t incl = h_lo + h_hi;
        const int l = tid & (kWave - 1);
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t other = (uint32_t)__shfl_down((int)incl, off, kWave);
            if (l + off < kWave) incl += other;
        }
        if (l == 0) wave_tot[tid >> 6] = incl;
        between();
        __syncthreads();
        uint32_t above_hi = incl - (h_lo + h_hi);  // pairs of higher threads of this wave
        for (int w = (tid >> 6) + 1; w < T / kWave; ++w) above_hi += wave_tot[w];
        const uint32_t above_lo = above_hi + h_hi;
        if ((int)above_hi < need && need <= (int)(above_hi + h_hi)) {
            s_digit = 2 * tid + 1;
            s_need = need - (int)above_hi;
            s_bin = (int)h_hi;
        } else if ((int)above_lo < need && need <= (int)(above_lo + h_lo)) {
            s_digit = 2 * tid;
            s_need = need - (int)above_lo;
            s_bin = (int)h_lo;
        }
        __syncthreads();
    };

    // ---- candidates from the groups' maxima
    bool done = false;
    if (k <= kBoundTopK) {
        const int l = tid & (kWave - 1);
        uint32_t top = 0, bound_key;
#pragma unroll
        for (int i = 0; i < KPT; ++i) top = zk[i] > top ? zk[i] : top;
        if (tid == 0) s_count = 0, s_bound = 0xFFFFFFFFu;
        if (k <= kGroupTopK) {  // the smallest maximum that fewer than k others exceed
            const int per = k <= 64 ? 8 : 4;  // threads of a group, which look at a share of the other groups' maxima each
            top = max(top, (uint32_t)other_half<1>((int)top));
            top = max(top, (uint32_t)other_half<2>((int)top));
            if (per >= 8) top = max(top, (uint32_t)other_half<4>((int)top));
            if (tid % per == 0) reinterpret_cast<uint32_t*>(maxima)[tid / per] = top;
            __syncthreads();
            const int share = T / per / 4 / per;  // of uint4
            const uint4* from = maxima + (tid % per) * share;
            int above = 0;
#pragma unroll 4
            for (int c = 0; c < share; ++c) {
                const uint4 w = from[c];
                above += (w.x > top ? 1 : 0) + (w.y > top ? 1 : 0) + (w.z > top ? 1 : 0) + (w.w > top ? 1 : 0);
            }
            above += other_half<1>(above);
            above += other_half<2>(above);
            if (per >= 8) above += other_half<4>(above);
            uint32_t least = above < k ? top : 0xFFFFFFFFu;
            least = min(least, (uint32_t)other_half<4>((int)least));
            least = min(least, (uint32_t)other_half<8>((int)least));
            if ((l & 15) == 0 && least != 0xFFFFFFFFu) atomicMin(&s_bound, least);
            __syncthreads();
            bound_key = s_bound;
        } else {  // of the threads' maxima, by two histograms of one increment a thread: 11 bits of the key, then 11 more
            uint32_t prefix = 0;
            int need = k;
            hist2[0][2 * tid] = 0;
            hist2[0][2 * tid + 1] = 0;
            hist2[1][2 * tid] = 0;
            hist2[1][2 * tid + 1] = 0;
            __syncthreads();
            for (int pass = 0; pass < 2; ++pass) {
                if (top != 0 && (pass == 0 || (top >> 21) == prefix)) atomicAdd(&hist2[pass][(pass == 0 ? top >> 21 : top >> 10) & 2047u], 1u);
                __syncthreads();
                find_digit(hist2[pass], need, [] {});
                prefix = (prefix << 11) | (uint32_t)s_digit;
                need = s_need;
            }
            bound_key = prefix << 10;
        }
        // `low`: every logit whose quotient reaches the bound's has this key or a larger one
        const float bound = order_key_inv(max(bound_key, 1u)), quotient = bound / temperature;
        uint32_t low;
        if (!kLate) {
            low = max(bound_key, 1u);
        } else if (fabsf(bound) >= 0x1p-100f && fabsf(quotient) >= 0x1p-100f && fabsf(bound) <= 0x1p120f && fabsf(quotient) <= 0x1p120f) {
            low = order_key(bound - fabsf(bound) * 0x1p-20f);  // 2^-20 below it is more than a rounding away
        } else {  // zeros, infinities, quotients that round coarsely: by the quotients themselves
            divide();
            low = bound == bound ? value_key(quotient) : 1u;  // (no number: fewer than k groups have a logit, all are candidates)
        }
        int count = 0;
#pragma unroll
        for (int i = 0; i < KPT; ++i) count += __builtin_popcountll(__ballot(zk[i] >= low));
        if (count != 0) {  // one add a wave; the order of the list does not matter
            int at = 0;
            if (l == 0) at = atomicAdd(&s_count, count);
            at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                const bool in = zk[i] >= low;
                const uint64_t m = __ballot(in);
                if (m == 0 || at >= kMaxRanked) continue;
                const int to = at + __builtin_popcountll(m & ((1ull << l) - 1ull));
                if (in && to < kMaxRanked) cand[to] = key_of(i);
                at += __builtin_popcountll(m);
            }
        }
        __syncthreads();
        const int n = s_count;
        if (kLate && n <= kMaxRanked && !divided) {
            if (tid < n) cand[tid] = candidate_key(order_key_inv((uint32_t)(cand[tid] >> 32)), temperature, (int)(0xFFFFFFFFu - (uint32_t)cand[tid]));
            __syncthreads();
        }
        if (n <= kMaxRanked) {  // each candidate counts the larger ones, which is its rank
            int np = 16;  // candidates rounded up to a power of two; T / np neighbouring threads share one
            while (np < n) np <<= 1;
            const int parts = T / np;
            const int i = tid / parts;
            const uint64_t mine = i < n ? cand[i] : 0;
            int above = 0;
            for (int j = tid % parts; j < n; j += parts) above += cand[j] > mine ? 1 : 0;
            if (parts > 1) above += other_half<1>(above);
            if (parts > 2) above += other_half<2>(above);
            if (parts > 4) above += other_half<4>(above);
            if (parts > 8) above += other_half<8>(above);
            for (int off = 16; off < parts; off <<= 1) above += __shfl_xor(above, off, kWave);
            if (i < n && tid % parts == 0 && above < k) sel[above] = mine;
            done = true;
        } else if (kLate && !divided) {
            divide();
        }
        __syncthreads();
    }

    if (!done) {
        // ---- radix select as in sample_kernel, with digits of 11, 11, 10 bits for each half of the key: the
        // top byte of a float (sign and seven exponent bits) takes a handful of values over a row of logits
        // and the increments of a pass would queue up on those few counters; three more bits spread them.
        // Thread t owns bins 2t and 2t+1 of the 2048.
        uint64_t prefix = 0;
        int need = k;
        int shift = 64;
        bool all_of_bin = false;
        hist2[0][2 * tid] = 0;
        hist2[0][2 * tid + 1] = 0;
        __syncthreads();
        for (int pass = 0; pass < 6; ++pass) {
            const int width = (pass % 3 == 2) ? 10 : 11;
            shift -= width;
            const uint32_t dmask = (1u << width) - 1u;
            uint32_t* hist = hist2[pass & 1];
#pragma unroll
            for (int i = 0; i < KPT; ++i) {
                const bool in = zk[i] != 0;
                const uint64_t key = key_of(i);
                if (in && (pass == 0 || (key >> (shift + width)) == prefix)) atomicAdd(&hist[(uint32_t)(key >> shift) & dmask], 1u);
            }
            __syncthreads();
            find_digit(hist, need, [&] {
                hist2[(pass + 1) & 1][2 * tid] = 0;  // next pass's histogram
                hist2[(pass + 1) & 1][2 * tid + 1] = 0;
            });
            // (s_digit, s_need, s_bin and wave_tot are next written a barrier or more into the next pass)
            prefix = (prefix << width) | (uint64_t)s_digit;
            need = s_need;
            all_of_bin = s_bin == need;  // every key of this bin is wanted: no need to look at lower bits
            if (all_of_bin) break;
        }
        // all 64 bits decided (shift == 0) or the rest left open
        const uint64_t threshold = all_of_bin ? (prefix << shift) : prefix;

        // ---- gather the k survivors (any order), pad to a power of two, sort descending
        if (tid == 0) s_count = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            if (zk[i] != 0) {
                const uint64_t key = key_of(i);
                if (key >= threshold) sel[atomicAdd(&s_count, 1)] = key;
            }
        }
        int kp = 1;
        while (kp < k) kp <<= 1;
        __syncthreads();
        for (int i = k + tid; i < kp; i += T) sel[i] = 0;  // below every real key
        __syncthreads();
        for (int size = 2; size <= kp; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int i = tid; i < (kp >> 1); i += T) {
                    const int lo = 2 * i - (i & (stride - 1));
                    const int hi = lo + stride;
                    const bool desc = (lo & size) == 0;
                    const uint64_t a = sel[lo], b = sel[hi];
                    if ((a < b) == desc) {
                        sel[lo] = b;
                        sel[hi] = a;
                    }
                }
                __syncthreads();
            }
        }
    }

    if (k <= kWave) {  // all of them in the lanes of one wave: no barriers
        if (tid >= kWave) return;
        const uint64_t mine = tid < k ? sel[tid] : 0;
        const float z = order_key_inv((uint32_t)(mine >> 32));
        auto lane_of = [](float v, int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l)); };
        ebuf[tid] = det_expf(z - lane_of(z, 0));
        float c = 0.0f;  // lane i adds the first i + 1 of them, in order (what lanes from k on add is not used)
        for (int i = 0; i < k; i += 8) {
            const float4 a = *reinterpret_cast<const float4*>(&ebuf[i]), b = *reinterpret_cast<const float4*>(&ebuf[i + 4]);
            const float e[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float with = c + e[u];
                c = tid >= i + u ? with : c;
            }
        }
        const float cut = top_p * lane_of(c, k - 1);
        const uint64_t reach = __ballot(tid < k && c >= cut);
        const int n = reach != 0 ? __builtin_ctzll(reach) + 1 : k;
        const uint64_t r = splitmix64_mix(seed + (ctr + 1) * 0x9E3779B97F4A7C15ull);
        const float u = (float)(uint32_t)(r >> 40) * 0x1p-24f;
        const float target = u * lane_of(c, n - 1);
        const uint64_t over = __ballot(tid < n && c > target);
        const int pick = over != 0 ? __builtin_ctzll(over) : n - 1;
        if (tid == pick) tokens[blockIdx.x] = (int32_t)(0xFFFFFFFFu - (uint32_t)mine);
        return;
    }

    // ---- probabilities in rank order
    const float z0 = order_key_inv((uint32_t)(sel[0] >> 32));
    for (int i = tid; i < k; i += T) ebuf[i] = det_expf(order_key_inv((uint32_t)(sel[i] >> 32)) - z0);
    __syncthreads();
    if (tid == 0) {
        float acc = 0.0f;
        int i = 0;
        for (; i + 8 <= k; i += 8) {  // eight reads in flight, then their adds in order
            float e[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = ebuf[i + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                acc = acc + e[u];
                e[u] = acc;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) ebuf[i + u] = e[u];  // c_i
        }
        for (; i < k; ++i) {
            acc = acc + ebuf[i];
            ebuf[i] = acc;
        }
        s_cut = top_p * ebuf[k - 1];
        s_n = k;
    }
    __syncthreads();
    {   // n = 1 + the first i with c_i >= cut (k if rounding leaves none)
        const float cut = s_cut;
        int best = k;
        for (int i = tid; i < k; i += T)
            if (ebuf[i] >= cut) {
                best = i + 1;
                break;
            }
        if (best < k) atomicMin(&s_n, best);
    }
    __syncthreads();
    const int n = s_n;
    if (tid == 0) {
        const uint64_t r = splitmix64_mix(seed + (ctr + 1) * 0x9E3779B97F4A7C15ull);
        const float u = (float)(uint32_t)(r >> 40) * 0x1p-24f;
        s_target = u * ebuf[n - 1];
        s_pick = n - 1;
    }
    __syncthreads();
    {   // the first i < n with c_i > target (n-1 if rounding leaves none)
        const float target = s_target;
        for (int i = tid; i < n; i += T)
            if (ebuf[i] > target) {
                atomicMin(&s_pick, i);
                break;
            }
    }
    __syncthreads();
    if (tid == 0) tokens[blockIdx.x] = (int32_t)(0xFFFFFFFFu - (uint32_t)sel[s_pick]);
}

}  // namespace det

using namespace det;

extern "C" int det_sample(const float* logits, int B, int V, float temperature, int top_k, float top_p,
                          uint64_t seed, const int32_t* seq_ids, const int32_t* steps, int32_t* tokens,
                          void* stream)
{
    if (!logits || !seq_ids || !steps || !tokens || B < 1 || V < 1) return DET_EINVAL;
    if (!(temperature > 0.0f) || !(top_p > 0.0f) || !(top_p <= 1.0f)) return DET_EINVAL;
    if (top_k < 1 || top_k > kMaxTopK) return DET_ESHAPE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // 16-byte pieces where every row is made of such and every thread gets one.  Of more than 32768 logits only where the
    // candidates come from few groups: the radix select spills more registers with them (V = 50000, top-k 1000 94 us with and 75 without).
    const bool vec = aligned16(logits) && V % 4 == 0 && V >= 4 * kSampleThreads && (V <= 32 * kSampleThreads || top_k <= kGroupTopK);
#define DET_SAMPLE(KPT)                                                                                                      \
    if (vec)                                                                                                                 \
        hipLaunchKernelGGL((sample_kernel_reg<KPT, true>), dim3(B), dim3(kSampleThreads), 0, s, logits, V, temperature,     \
                           top_k, top_p, seed, seq_ids, steps, tokens);                                                      \
    else                                                                                                                     \
        hipLaunchKernelGGL((sample_kernel_reg<KPT, false>), dim3(B), dim3(kSampleThreads), 0, s, logits, V, temperature,    \
                           top_k, top_p, seed, seq_ids, steps, tokens)
    // An infinite temperature changes the order (+inf / T is no number, behind the zeros that finite logits become): the form that
    // divides in front of its search takes it.  (A test of it in the other two cost 2 %: 3 rows of 16454 at top-k 112 17.2 us instead of 16.8.)
    const bool late = temperature < INFINITY;
    if (late && V <= kSampleThreads * 8) {
        DET_SAMPLE(8);
    } else if (late && V <= kSampleThreads * 32) {
        DET_SAMPLE(32);
    } else if (V <= kSampleThreads * 64) {
        DET_SAMPLE(64);
    } else
#undef DET_SAMPLE
        hipLaunchKernelGGL(sample_kernel, dim3(B), dim3(256), 0, s, logits, V, temperature, top_k, top_p, seed, seq_ids,
                           steps, tokens);
    return check_launch();
}

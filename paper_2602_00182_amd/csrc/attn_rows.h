// Which rows of a call that names slots walk their chunks inside one workgroup (attn_rows.hip), in which workgroup, and
// which are left to the per-chunk kernels (attn.hip).  Every kernel of the call works it out from the lengths and slots.
#pragma once

#include "common.h"

namespace det {

constexpr int kWalkPairs = 64;    // (row, head) pairs of a walking workgroup: 64 / G consecutive rows, a "tile"
constexpr int kWalkChunks = 8;    // rows of at most this many chunks are never left for their length
constexpr int kWalkSamples = 128;

__device__ __forceinline__ int attn_row_len(const int32_t* seqlens, int r, int len_offset, int Lmax)
{
    const int l = seqlens[r] + len_offset;
    return l > Lmax ? Lmax : l;
}

// Longest row, in chunks, that still walks.  A walk is serial, about 11 us a chunk, so a few long rows among short
// ones would outlast everything else of the call: they are left.  With W = the walks' chunks of the whole call
// (estimated from the last rows of up to 128 tiles), the per-chunk kernels take about W * Hkv / 6.4 us for all of
// it, so rows of more than W * Hkv / 70 chunks are left.  At least 128 threads, all of them, call it together.
__device__ __forceinline__ int attn_walk_limit(const int32_t* seqlens, int len_offset, int Lmax, int R, int ntiles, int rows,
                                               int Hkv, int* scratch)
{
    if (threadIdx.x == 0) *scratch = 0;
    __syncthreads();
    if (threadIdx.x < kWalkSamples) {
        const int n = ntiles < kWalkSamples ? ntiles : kWalkSamples;
        if ((int)threadIdx.x < n) {
            const int tile = (int)((long long)threadIdx.x * ntiles / n);
            const int r = (tile + 1) * rows - 1;
            const int l = attn_row_len(seqlens, r < R ? r : R - 1, len_offset, Lmax);
            atomicAdd(scratch, l > 0 ? (l + 255) >> 8 : 0);
        }
    }
    __syncthreads();
    const long long walks = (long long)*scratch * ntiles / (ntiles < kWalkSamples ? ntiles : kWalkSamples);
    const long long limit = walks * Hkv / 70;
    return limit < kWalkChunks ? kWalkChunks : (limit > (1 << 20) ? 1 << 20 : (int)limit);
}

// Rows of 64 consecutive ones (the first a multiple of 64), or of one tile, by how they are computed; lane i holds row
// i's length (0 or less: no tokens) and slot.  ROWS: rows of a tile, 8, 16, 32 or 64, neighbouring lanes.
//   deep  : longer than `limit` chunks: left to the per-chunk kernels.
//   walks : the others that have tokens.  Those of a tile, in order, fall into runs of one slot; `starts` are the runs' first
//           rows.  (The first row of a slot in its tile always starts a run.)
//   mixed : rows that walk, of tiles of more than one run.  A walk shares nothing between slots, so they are not walked one
//           after the other by the tile's own workgroup (sixteen slots of 1000 tokens would take it 500 us; eight rows
//           a slot at 200 tokens, 994 rows, 32/8 heads 48 us that way, 45 dealt out; 18 prompts of up to 119 tokens 42 and 37).
struct attn_row_classes {
    uint64_t deep, walks, starts, mixed;
};
template <int ROWS>
__device__ __forceinline__ attn_row_classes attn_classify_rows(int len, int slot, int limit)
{
    const int lane = threadIdx.x & 63;
    const uint64_t mine = (ROWS == 64 ? ~0ull : ((1ull << (ROWS & 63)) - 1ull)) << (lane & ~(ROWS - 1));  // the lanes of this lane's tile
    attn_row_classes k;
    k.deep = __ballot(len > limit * 256);
    const bool walks = len > 0 && len <= limit * 256;
    k.walks = __ballot(walks);
    const uint64_t above = k.walks & mine & ((1ull << lane) - 1ull);  // walking rows of the tile before this one
    const int before = __shfl(slot, above != 0 ? 63 - __builtin_clzll(above) : lane, 64);
    k.starts = __ballot(walks && (above == 0 || slot != before));
    k.mixed = __ballot(walks && __builtin_popcountll(k.starts & mine) > 1);
    return k;
}

// f(w, classes) for the 64-row words w of all rows, dealt to the waves of the workgroup; eight words' loads at a time.
template <int ROWS, class F>
__device__ __forceinline__ void attn_for_row_words(const int32_t* __restrict__ seqlens, const int32_t* __restrict__ slots,
                                                   int len_offset, int Lmax, int R, int limit, F&& f)
{
    constexpr int U = 8;
    const int words = (R + 63) >> 6, lane = threadIdx.x & 63, waves = (int)(blockDim.x >> 6);
    for (int w0 = (int)(threadIdx.x >> 6); w0 < words; w0 += U * waves) {
        int l[U], sl[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = 64 * (w0 + u * waves) + lane;
            l[u] = r < R ? attn_row_len(seqlens, r, len_offset, Lmax) : 0;
            sl[u] = r < R ? slots[r] : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (w0 + u * waves < words) f(w0 + u * waves, attn_classify_rows<ROWS>(l[u], sl[u], limit));
    }
}

}  // namespace det

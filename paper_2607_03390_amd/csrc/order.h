// Blend order of the tiles to rasterise, run by the first block of the tile
// sort's last launch or, on grids that take the general sort, by a kernel of
// its own.
#pragma once

#include "match.h"
#include "tgs_internal.h"

namespace tgs {

// Blend order of the tiles to rasterise: longest lists first, bucketed by
// floor(log2(length)).  Tile lists are bimodal (a few thousand long tiles
// next to many short ones); launched in raster order, long tiles dispatched
// last would set the blend's tail.  Tiles are independent, so the order
// within a bucket changes only scheduling, never a result; the split set is
// a union of whole buckets.
// Bucket of a list length: floor(log2(len)) + 1, 0 for an empty list.
__device__ inline uint32_t length_bucket(uint32_t len) { return len ? 32u - (uint32_t)__clz(len) : 0u; }

// Length bucket from which a frame splits its tiles, at most `most`: of n_keys
// keys of n_visible Gaussians on n_tiles tiles to render, `busy` of them with
// lists of 2^(kBusyBucket - 1) entries and more.  Splitting pays where a few
// tiles are still walked when the rest of the chip has run dry (about 2048 tile
// blocks are resident at once); everywhere else the quadrants only stage their
// lists four times.
//  - Narrow Gaussians (fewer than kWideKeys tiles each): a tile takes about as
//    long as its list.  Split are lists of at least the keys that 1024 evenly
//    loaded blocks would each hold, rounded up to a power of two.
//  - Wide ones: pixels stop long before their lists end, so that the lengths
//    say little; what counts is whether the tiles fill the chip.  With up to
//    kFewTiles busy tiles, lists are split from 2^kFewLog entries on at the
//    latest, with more as few as may be.
// Either way a lower bound: 32 where all tiles' quadrants are resident at once
// (512 tiles), and more on larger grids, where quadrants of short lists are
// only more blocks to launch.
//
// Measured at thresholds of 2^5 .. 2^12 (blend launch, microseconds; 2^12 splits
// hardly any tile).  Narrow: 107k keys on 920 tiles with every output 54 up to
// 2^9, 88 at 2^10, 149 at 2^12; 745k on 3600 tiles 59 up to 2^8, 69 at 2^10, 88
// at 2^12; 632k on 230 of 390 tiles 31 up to 2^8, 57 at 2^10, 85 from 2^11;
// 201k on 8160 tiles 24 at 2^8, 32 from 2^10; 572k - 1.1M on the selected tiles
// of a room 72 up to 2^9, 58 from 2^10; at worst 457k on 3600 tiles 42 at 2^9,
// 38 from 2^10.  Wide, few tiles: 1.07M keys on 600 of 1000 tiles 35 at 2^7, 38
// at 2^8, 55 at 2^10, 59 at 2^12.  Many: 531k on 1300 of 2280 tiles 42 to 49 up
// to 2^10, 38 from 2^11; 1.77M on as many 54 to 64 up to 2^11, 44 at 2^12; 1.89M
// on 3000 of 8160 72 up to 2^10, 62 at 2^11, 46 at 2^12; at worst 20k needles
// on all of 1000 tiles 33 at 2^10, 39 at 2^12.  (By the first rule for all
// frames those five took 62, 45, 58, 62 and 33.)  By the grid: 34k keys on 256
// tiles 12 up to 2^7, 16 at 2^8, 22 from 2^9; 53k on 1600 tiles 15.0 at 2^6,
// 13.1 from 2^7; 72k on 3600 tiles 17.6 at 2^6, 16.1 at 2^7, 18.3 at 2^8; 96k
// on 6300 tiles 17.3 at 2^7, 16.3 at 2^8.
constexpr uint32_t kWideKeys = 5, kFewTiles = 768;
constexpr int kBusyBucket = 5, kFewLog = 8;
__device__ inline int split_bucket_for(uint32_t n_keys, uint32_t n_visible, int n_tiles, uint32_t busy,
                                       int most) {
    const uint32_t mean = n_keys >> 10;
    const int least = 5 + (n_tiles > 512) + (n_tiles > 1024) + (n_tiles > 4096);
    const int lg = mean > 1u << least ? 32 - __clz(mean - 1u) : least;
    if (lg + 1 >= most) return most;
    return n_keys / kWideKeys < n_visible ? lg + 1 : busy > kFewTiles ? most : lg < kFewLog ? lg + 1 : kFewLog + 1;
}

constexpr int kOrderBuckets = 33;
// LDS words of order_tiles_share<NT>: two copies of the bucket counters per
// wave, twice.
constexpr int order_lds_words(int nt) { return 4 * (nt / 64) * kOrderBuckets; }

// Ranks N items per lane against running bucket counters wc[33] (in
// order: item k before item k + 1, lanes in order): lanes with equal
// buckets are matched over the six bucket bits and the lowest lane of each
// group advances the counter by the group's size with one LDS atomic, whose
// old value the group shares.  The N atomics are all issued before the
// first result is used.
template <int N>
__device__ inline void wave_bucket_rank(uint32_t *wc, const uint32_t (&b)[N], const bool (&active)[N],
                                        uint32_t (&rank)[N]) {
    const int lane = threadIdx.x & 63;
    const uint64_t lt = (1ull << lane) - 1ull;
    uint64_t pm[N];
#pragma unroll
    for (int k = 0; k < N; ++k) pm[k] = __ballot(active[k]);
    match_digits<N>(b, 6, pm);
    int leader[N];
    uint32_t base[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        leader[k] = pm[k] ? __ffsll((long long)pm[k]) - 1 : lane;
        base[k] = 0u;
        if (active[k] && lane == leader[k]) base[k] = atomicAdd(&wc[b[k]], (uint32_t)__popcll(pm[k]));
    }
#pragma unroll
    for (int k = 0; k < N; ++k) rank[k] = __shfl(base[k], leader[k]) + (uint32_t)__popcll(pm[k] & lt);
}

// First place of bucket 32 - tid in the order (buckets longest first) from
// its tiles c (of n in all); with `publish` also the split count and, for the
// host, the longest bucket.  Run by one whole wave (tid < 64; c = 0 from tid
// 33 on).
__device__ inline uint32_t order_bucket_start(const OrderK &o, uint32_t c, int n, bool publish) {
    const int tid = threadIdx.x, b = 32 - tid;
    uint32_t inc = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t x = __shfl_up(inc, d);
        if (tid >= d) inc += x;
    }
    if (!publish) return inc - c;   // block-uniform
    // the tiles the blend splits, a prefix of the order: those of the
    // buckets from the lowest one >= split_bucket that leaves at most
    // max_split tiles in it and above (whole buckets)
    const uint32_t busy = __shfl(inc, 32 - kBusyBucket);
    const int sb = o.cnt && o.split_bucket >= 1
                       ? split_bucket_for(o.cnt->n_sorted, o.cnt->n_visible, n, busy, o.split_bucket)
                       : o.split_bucket;
    const uint64_t fit = __ballot(sb >= 1 && b >= sb && inc <= (uint32_t)o.max_split);
    const uint32_t ns = __shfl(inc, fit ? 63 - __clzll((long long)fit) : 0);
    if (o.n_split && tid == 0) *o.n_split = fit ? ns : 0u;
    const uint64_t nz = __ballot(c != 0u);
    // the host reads this value some frames later: no fence needed (a frame
    // without keys, for one that is about to be rendered again, says nothing
    // of the next one's lists)
    const int longest = nz ? 32 - (__ffsll((long long)nz) - 1) : 0;
    if (o.max_bucket && tid == 0 && longest)
        __hip_atomic_store(o.max_bucket, (uint32_t)longest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return inc - c;
}

// Share `share` of n_shares blocks of NT threads that order the n tiles
// tile_at(0 .. n - 1) by bucket_of(tile) into o.tile_out (s_cnt:
// order_lds_words(NT) words of LDS).  Every block counts all tiles (a few
// loads and LDS adds per thread, on two copies of the counters per wave) and
// places those of its share only: after the tiles of longer buckets and
// after those of the same bucket in the shares before it.  No block waits for
// another.
template <int NT, typename Tile, typename Bucket>
__device__ void order_tiles_share(const OrderK &o, int n, int share, int n_shares, uint32_t *s_cnt,
                                  Tile tile_at, Bucket bucket_of) {
    constexpr int kPer = 8;   // tiles per thread and round: all loads of a round in flight
    constexpr int kWaves = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // counters: [wave, copy][bucket] of the shares before, then of the others
    uint32_t *before = s_cnt, *after = s_cnt + 2 * kWaves * kOrderBuckets;
    for (int k = tid; k < order_lds_words(NT); k += NT) s_cnt[k] = 0u;
    __syncthreads();
    const int per = (n + n_shares - 1) / n_shares, i0 = share * per;
    const int i1 = i0 + per < n ? i0 + per : n;
    const int row = (2 * wave + (lane & 1)) * kOrderBuckets;
    for (int c0 = 0; c0 < n; c0 += kPer * NT) {
        uint32_t bk[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = c0 + k * NT + tid;
            bk[k] = i < n ? bucket_of(tile_at(i)) : 0u;
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = c0 + k * NT + tid;
            if (i < n) atomicAdd(&(i < i0 ? before : after)[row + bk[k]], 1u);
        }
    }
    __syncthreads();
    if (tid < 64) {
        uint32_t cb = 0, ca = 0;
        if (tid <= 32) {
#pragma unroll
            for (int w = 0; w < 2 * kWaves; ++w) {
                cb += before[w * kOrderBuckets + 32 - tid];
                ca += after[w * kOrderBuckets + 32 - tid];
            }
        }
        const uint32_t start = order_bucket_start(o, cb + ca, n, share == 0);
        if (tid <= 32) before[32 - tid] = start + cb;
    }
    __syncthreads();
    // the block's own tiles, from the running starts (shared by its waves:
    // the order within a bucket follows their timing)
    for (int c0 = i0; c0 < i1; c0 += kPer * NT) {
        int t[kPer];
        uint32_t bk[kPer], rank[kPer];
        bool act[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = c0 + k * NT + tid;
            act[k] = i < i1;
            t[k] = act[k] ? tile_at(i) : 0;
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) bk[k] = act[k] ? bucket_of(t[k]) : 0u;
        wave_bucket_rank<kPer>(before, bk, act, rank);
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (act[k]) o.tile_out[rank[k]] = t[k];
    }
}

}  // namespace tgs

// What the radix sorts share: sizes, block scans and the layout of the count
// tables (k_sort.hip: sorts of (key, value) pairs; k_tilesort.hip: the tile
// sort of packed keys).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tgs {

constexpr int kSortThreads = 256;
constexpr int kRadix = 256;
// The partitions holding keys are cut into kChunks chunks of consecutive
// partitions: the column scan turns their digit counts into prefixes within
// the chunk and per-chunk sums, the downsweep adds the sums of earlier chunks.
constexpr int kChunks = 16;

__device__ inline uint32_t chunk_len(uint32_t npa) {
    const uint32_t L = (npa + kChunks - 1) / kChunks;
    return L ? L : 1u;
}

__device__ inline uint32_t sat32(uint64_t v) { return v > 0xffffffffull ? 0xffffffffu : (uint32_t)v; }

// Blocks are dealt to the eight XCDs in turn; each XCD takes a run of
// consecutive partitions.  A partition writes runs of 20-40 keys per digit
// that neither begin nor end on a cache line, and the next partition's run
// continues each of them: written through the same L2 the two halves of
// a line leave as one full line, through two they leave as partial lines
// (2.27G keys at 8 + 7 bits: 19.0 -> 10.5 ms per pass; 5.0M keys, which
// the last-level cache holds: 21.2 -> 21.1 us).
// Partition of block b of a grid of whole rounds of eight blocks; false: none.
__device__ inline bool xcd_partition(uint32_t b, uint32_t npa, uint32_t &part) {
    const uint32_t per_xcd = npa ? (npa + 7) / 8 : 1u;
    part = (b & 7u) * per_xcd + (b >> 3);
    return (b >> 3) < per_xcd;
}

template <typename T>
__device__ inline T block_exclusive_scan256(T v, T *s_wave, T *total = nullptr) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    T inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const T o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    T off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const T x = s_wave[w];
        if (w < wave) off += x;
        tot += x;
    }
    __syncthreads();
    if (total) *total = tot;
    return off + inc - v;
}

}  // namespace tgs

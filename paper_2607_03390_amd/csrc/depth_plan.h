// Sizes of the sample sort by depth (k_depthsort.hip).  Host arithmetic only.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace tgs {

constexpr int kDepthSamples = 16384;   // ranked samples, at most
constexpr int kBucketMost = 16384;     // entries of a bucket's region, at most
constexpr int kBucketSmall = 4096;     // buckets sorted by 512-thread blocks, three to a CU
constexpr int kFillBits = 24;          // a bucket's fill: Gaussians in the low bits, keys above

struct DepthPlan {
    bool ok;            // the sort is taken at all
    int stride, ns;     // samples: one per stride Gaussians
    int nb, log_nb;     // buckets
    uint32_t cap;       // entries of a bucket's region
    size_t entries;     // bytes of all regions
    size_t words;       // 8-byte words of the other scratch
};

// A bucket per CU while they hold up to 6144 Gaussians each (of whom half to
// three quarters are usually visible), more buckets above: the fewer they
// are, the longer the runs of a block's entries in one region and the fewer
// samples have to be ranked.  Regions of four times a bucket's share of the
// Gaussians, as far as the LDS that sorts them goes: at least 2.67 times, at
// the most Gaussians of 256, 512 and 1024 buckets.
//
// A bucket ends at a given number of samples after its start (16; 8 of 2048
// buckets), so it overflows where a region's worth of Gaussians holds fewer.
// With every Gaussian visible and depths that know nothing of the order of
// the scene, their number is Poisson with mean cap / stride, and the chance that
// any bucket of a frame overflows is below 1e-3 at every n (the most at 1024 x
// 6144: mean 42.7, 1e-6 a bucket; 2e-4 at 2^23 - 1: mean 32, 1e-7 a bucket).
inline DepthPlan depth_plan(int n, int n_tiles) {
    DepthPlan p{};
    if (n < 1 || n >= 1 << 23 || (uint64_t)n * (uint64_t)n_tiles >= 1ull << (64 - kFillBits)) return p;
    p.ok = true;
    const int want = n <= 256 * 6144 ? 256 : n <= 512 * 6144 ? 512 : n <= 1024 * 6144 ? 1024 : 2048;
    const int per = 16 * want <= kDepthSamples ? 16 : kDepthSamples / want;   // samples per bucket
    p.stride = (n + per * want - 1) / (per * want);
    p.ns = (n + p.stride - 1) / p.stride;
    p.nb = (p.ns + per - 1) / per;
    while ((1 << p.log_nb) < p.nb) p.log_nb += 1;
    const int share = (n + p.nb - 1) / p.nb;
    p.cap = share <= kBucketSmall / 3 ? kBucketSmall : share <= kBucketMost / 4 ? 4 * share : kBucketMost;
    p.entries = 16 * (size_t)p.nb * p.cap;
    // splitters, fills, sorted rectangles, samples (4 bytes each)
    p.words = 2 * (size_t)p.nb + (size_t)n + ((size_t)p.ns + 1) / 2;
    return p;
}

}  // namespace tgs

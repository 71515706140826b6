// Depth order of the Gaussians that have keys (Sec. III-A), by a sample sort
// in three launches, for scenes of fewer than 2^23 Gaussians and 2^40
// (Gaussian, tile) pairs (k_sort.hip's radix passes otherwise, and when a
// bucket overflows):
//
//  1. The preprocess leaves one sample per stratum of consecutive Gaussians:
//     the depth bits of a Gaussian at a hashed place (kNoDepth: it has no
//     keys).  The splitter kernel ranks every valid sample against all the
//     others and takes one in sixteen (of 2048 buckets: one in eight) as a
//     splitter (depth bits, index): with the index, equal depths (a wall seen
//     head-on) are split as evenly as any others.
//  2. The scatter kernel finds each Gaussian's bucket by bisection of the
//     splitters in LDS, counts its block's Gaussians and keys per bucket
//     there, reserves places in the buckets' regions with one add per (block,
//     bucket), and writes (depth bits, index, rectangle).
//  3. A block per bucket (scenes above 1.5M Gaussians: a second launch for
//     buckets of more than 8192) sorts it in LDS (ranges of equal width, then
//     compares inside a range, ties by index), sums the counts of the buckets
//     before it, and writes the sorted indices and rectangles, the start of
//     each Gaussian's keys and the key blocks' owners.  Block 0 publishes the
//     frame's counters.
//
// The order of arrival in a bucket depends on timing, its sorted order does
// not.  A bucket beyond its region (depth_plan.h: below one frame in a
// thousand where depths know nothing of the order of the scene) makes the
// frame publish no keys and HostCounters::redo, and the host renders it again
// by another way.
//
// Against twelve launches of radix passes (count, column scan, scatter, four
// times), each latency-bound: 1.13M of 1.5M Gaussians 98 -> 66 us, 300k 62 -> 27
// us, 3.3M of 6M 175 -> 168 us; and with the rectangles in that order the key
// emission reads them in line: 24.0 -> 15.9, 8.3 -> 5.7 and 75 -> 25.6 us.
#include "radix.h"
#include "tgs_internal.h"

namespace tgs {

namespace {

constexpr int kRankThreads = 512;
constexpr int kRankBlocks = 256;      // of the splitter kernel, at most: one per CU
constexpr int kScatterThreads = 512;
constexpr int kBucketShort = 8192;    // buckets sorted with half the LDS of the longest

// Members of a sub-bucket up to which a bucket is ranked by compares: a compare
// per member for each entry.  Where one has more, those of more than kCrowd
// are cut again.  The cuts have their own cost, and a bucket between a near and a
// far part of a scene reaches a hundred at its ends: a room of 1.5M, whose
// slowest bucket is one, 33.0 us on average by compares and 42.7 cut again from
// 49 on.
constexpr uint32_t kCrowdMost = 128;
constexpr uint32_t kCrowd = 48;

// A bucket's fill and keys in one word: Gaussians in the low kFillBits, keys
// above (scenes of under 2^23 Gaussians and 2^40 (Gaussian, tile) pairs).
__device__ inline uint32_t fill_of(uint64_t v) { return (uint32_t)v & ((1u << kFillBits) - 1u); }

// Ranks the valid samples (depth bits, by stratum, that is by index) against
// each other and writes one per bucket, evenly spaced, as a splitter: thread (g, l) holds PER
// of the block's 4 PER samples (g = tid & 3) and compares them with every
// 128th of all (l = tid >> 2), one LDS read and PER compares at a time.  Samples
// of equal depth rank by stratum: those before the block's count as lower
// up to equality, those after it below it only.
template <int PER>
__global__ __launch_bounds__(kRankThreads) void depth_splitters_kernel(const uint32_t *samples, int ns,
                                                                       int stride, int n, int nb,
                                                                       uint64_t *splitters, uint64_t *fill) {
    constexpr int kRankPer = 4 * PER;
    __shared__ uint32_t s_d[kRankPer * kRankBlocks];
    constexpr int kWaves = kRankThreads / 64, kSlices = kRankThreads / 4;
    __shared__ uint32_t s_red[kWaves][kRankPer];
    __shared__ uint32_t s_valid[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int b = blockIdx.x * kRankThreads + tid; b < nb; b += gridDim.x * kRankThreads) fill[b] = 0ull;
    uint32_t valid = 0;
    for (int i0 = 0; i0 < ns; i0 += 8 * kRankThreads) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * kRankThreads + tid;
            v[u] = i < ns ? samples[i] : kNoDepth;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * kRankThreads + tid;
            if (i < ns) s_d[i] = v[u];
            valid += v[u] != kNoDepth ? 1u : 0u;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) valid += __shfl_xor(valid, o);
    if (lane == 0) s_valid[wave] = valid;
    __syncthreads();
    uint32_t m = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) m += s_valid[w];
    if (m == 0u) {   // block-uniform: one bucket
        for (int b = blockIdx.x * kRankThreads + tid; b < nb - 1; b += gridDim.x * kRankThreads)
            splitters[b] = ~0ull;
        return;
    }
    const int e0 = blockIdx.x * kRankPer, e1 = min(e0 + kRankPer, ns), g = tid & 3, l = tid >> 2;
    uint32_t d[PER], rank[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        d[k] = e0 + PER * g + k < ns ? s_d[e0 + PER * g + k] : kNoDepth;
        rank[k] = 0u;
    }
    int i = l;
#pragma unroll 4
    for (; i < e0; i += kSlices) {
        const uint32_t x = s_d[i];
#pragma unroll
        for (int k = 0; k < PER; ++k) rank[k] += x <= d[k] ? 1u : 0u;
    }
    for (; i < e1; i += kSlices) {
        const uint32_t x = s_d[i];
#pragma unroll
        for (int k = 0; k < PER; ++k)
            rank[k] += x < d[k] || (x == d[k] && i < e0 + PER * g + k) ? 1u : 0u;
    }
#pragma unroll 4
    for (; i < ns; i += kSlices) {
        const uint32_t x = s_d[i];
#pragma unroll
        for (int k = 0; k < PER; ++k) rank[k] += x < d[k] ? 1u : 0u;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        uint32_t r = rank[k];
#pragma unroll
        for (int o = 4; o <= 32; o <<= 1) r += __shfl_xor(r, o);
        if (lane < 4) s_red[wave][PER * g + k] = r;
    }
    __syncthreads();
    if (tid >= kRankPer || e0 + tid >= ns) return;
    const uint32_t mine = s_d[e0 + tid];
    if (mine == kNoDepth) return;
    uint32_t r = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) r += s_red[w][tid];
    // splitter j (1 .. nb - 1) is the sample of rank floor(j m / nb)
    uint64_t j = ((uint64_t)r * nb + m - 1) / m;
    if (j == 0) j = 1;
    for (; j < (uint64_t)nb && j * m / nb == r; ++j)
        splitters[j - 1] = (uint64_t)mine << 32 | depth_sample_at((uint32_t)(e0 + tid), (uint32_t)stride, n);
}

template <int IPT>
__global__ __launch_bounds__(kScatterThreads) void depth_scatter_kernel(
    int n, const uint32_t *__restrict__ dkey, const ushort4 *__restrict__ rect, const uint32_t *sat, int TX,
    const uint64_t *__restrict__ splitters, int nb, int log_nb, uint32_t cap, unsigned long long *fill,
    uint4 *entries) {
    extern __shared__ uint64_t s_mem[];
    uint64_t *s_split = s_mem;                                           // 2^log_nb
    unsigned long long *s_fill = reinterpret_cast<unsigned long long *>(s_mem + ((size_t)1 << log_nb));
    const int tid = threadIdx.x, nb2 = 1 << log_nb;
    const uint32_t base = blockIdx.x * (uint32_t)(kScatterThreads * IPT);
    uint32_t key[IPT];
    ushort4 rc[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t i = base + (uint32_t)(j * kScatterThreads + tid);
        key[j] = i < (uint32_t)n ? dkey[i] : kNoDepth;
        rc[j] = i < (uint32_t)n ? rect[i] : make_ushort4(1, 1, 0, 0);
    }
    for (int b = tid; b < nb2; b += kScatterThreads) {
        s_split[b] = b < nb - 1 ? splitters[b] : ~0ull;
        s_fill[b] = 0ull;
    }
    __syncthreads();
    // number of splitters <= (depth, index): the items' bisections side by
    // side (the padding exceeds every item)
    uint32_t at[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) at[j] = 0u;
    for (int s = nb2 >> 1; s >= 1; s >>= 1) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const uint64_t v = (uint64_t)key[j] << 32 | (base + (uint32_t)(j * kScatterThreads + tid));
            at[j] += s_split[at[j] + s - 1] <= v ? (uint32_t)s : 0u;
        }
    }
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t c = key[j] == kNoDepth ? 0u
                         : sat ? masked_count(rc[j], sat, TX)
                               : (uint32_t)(rc[j].z - rc[j].x + 1) * (uint32_t)(rc[j].w - rc[j].y + 1);
        // bucket << 16 | place among the block's; all ones: no keys
        if (c) {
            const uint64_t old = atomicAdd(&s_fill[at[j]], 1ull | (unsigned long long)c << kFillBits);
            at[j] = at[j] << 16 | fill_of(old);
        } else {
            at[j] = 0xffffffffu;
        }
    }
    __syncthreads();
    for (int b = tid; b < nb; b += kScatterThreads) {
        const unsigned long long c = s_fill[b];
        if (c) s_fill[b] = atomicAdd(&fill[b], c);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        if (at[j] != 0xffffffffu) {
            const uint32_t b = at[j] >> 16, o = fill_of(s_fill[b]) + (at[j] & 0xffffu);
            if (o < cap)
                entries[(size_t)b * cap + o] =
                    make_uint4(key[j], base + (uint32_t)(j * kScatterThreads + tid),
                               (uint32_t)rc[j].x | (uint32_t)rc[j].y << 16,
                               (uint32_t)rc[j].z | (uint32_t)rc[j].w << 16);
        }
    }
}

// Exclusive scan across the block (of kWaves waves) of one value per thread;
// *total the sum.
template <int kWaves, typename T>
__device__ inline T bucket_scan(T v, T *s_wave, T *total) {
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
    for (int w = 0; w < kWaves; ++w) {
        const T x = s_wave[w];
        if (w < wave) off += x;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

struct BucketIo {
    const uint64_t *fill;
    const uint4 *entries;
    int nb;
    uint32_t cap;               // entries of a region
    const uint32_t *sat;        // selective frames
    int TX;
    uint32_t *didx, *offs, *kfirst;
    ushort4 *srect;
    Counters *cnt;
    HostCounters *host;
    uint32_t tag, key_cap;
    const uint32_t *pre_partial;
    int n_pre;
};

// A crowded sub-bucket: its entries stand at kv[at, at + n), pre of those in
// crowded sub-buckets come before them, and their places in the bucket's order
// begin at fin.  Bounds of their differences (d) and indices (i).
struct Crowd {
    uint32_t at, n, pre, fin;
    uint32_t dlo, dhi, ilo, ihi;
};

// LDS of a block of NT threads sorting a bucket of up to CAP entries.
template <int CAP, int NT>
struct BucketLds {
    static constexpr int kSub = 4 * NT;   // sub-buckets
    static constexpr int kGroups = CAP / (kCrowd + 1);
    Crowd crowd[kGroups];
    uint32_t shift[kGroups];              // fin - pre of the cut before
    uint64_t kv[CAP];                     // keys by sub-bucket, then the sorted entries' key counts
    uint32_t cur[kSub];                   // sub-bucket sizes, starts, ends
    uint32_t scan[2 * (NT / 64)];
};

// Key count of an entry's rectangle.
__device__ inline uint32_t entry_keys(const BucketIo &io, uint4 v) {
    const ushort4 r = make_ushort4((unsigned short)(v.z & 0xffffu), (unsigned short)(v.z >> 16),
                                   (unsigned short)(v.w & 0xffffu), (unsigned short)(v.w >> 16));
    return io.sat ? masked_count(r, io.sat, io.TX)
                  : (uint32_t)(r.z - r.x + 1) * (uint32_t)(r.w - r.y + 1);
}

// Min and max over the block of the threads' lo and hi.
template <int kWaves>
__device__ inline void bucket_range(uint32_t *s, uint32_t &lo, uint32_t &hi) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o));
        hi = max(hi, __shfl_xor(hi, o));
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        s[wave] = lo;
        s[kWaves + wave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        lo = min(lo, s[w]);
        hi = max(hi, s[kWaves + w]);
    }
    __syncthreads();
}

// How a bucket was cut into sub-buckets: by depth (its least: lo), or where
// all depths are one by index (its least), shifted by sh.
struct Cut {
    uint32_t lo;
    int sh;
    bool one_depth;
};

// Places of a bucket's E entries where sub-buckets are crowded, to tmp[0, E).
// On entry kv holds (difference, index) by sub-bucket and s.cur each one's end
// (c: how they were cut).  Entries of the others are ranked by compares; those of the crowded ones are cut again,
// every group of them into its share of the kSub sub-buckets over its own
// least to largest difference (or index, where the difference is one), until
// none is crowded.
//
// A group has 49 entries or more and so a dozen sub-buckets, and its bounds
// differ (indices do); its least entry falls into the first of them and its
// largest into the upper half: every cut takes each group apart, and its range
// by a factor of ten or so, so the loop ends (31 bits of difference, 23 of
// index; a plane seen head-on: one cut).
//
// Entries and places are read from memory (the cache) in every step, not held:
// registers for them would be taken from buckets that are not crowded.
template <int CAP, int NT>
__device__ __attribute__((always_inline)) inline void rank_crowded(BucketLds<CAP, NT> &s, const uint4 *ent,
                                                                   uint32_t E, const Cut &c, uint32_t *tmp) {
    constexpr int kWaves = NT / 64, kSub = BucketLds<CAP, NT>::kSub, kPer = kSub / NT;
    // an entry without a place: the group it was in (bits 16 - 30) and its sub-bucket
    constexpr uint32_t kActive = 1u << 31;
    static_assert(kSub <= 1 << 16 && CAP < 1 << 16, "packed words");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto entry = [&](uint32_t i) {
        const uint2 x = *reinterpret_cast<const uint2 *>(ent + i);
        return make_uint2((c.one_depth ? x.y : x.x) - c.lo, x.y);
    };
    uint32_t lim = E;       // of kv
    uint32_t cnt[kPer];     // sizes of the thread's own sub-buckets
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = tid * kPer + k;
        cnt[k] = s.cur[i] - (i ? s.cur[i - 1] : 0u);
    }
    for (int round = 0;; ++round) {
        uint32_t mine = 0, tot;   // entries in crowded sub-buckets, and those << 16
#pragma unroll
        for (int k = 0; k < kPer; ++k) mine += cnt[k] > kCrowd ? cnt[k] | 1u << 16 : 0u;
        uint32_t p = bucket_scan<kWaves, uint32_t>(mine, s.scan, &tot);
        const uint32_t ng = tot >> 16, act = tot & 0xffffu;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (cnt[k] > kCrowd) {
                uint32_t &end = s.cur[tid * kPer + k];
                s.crowd[p >> 16] = Crowd{end - cnt[k], cnt[k], p & 0xffffu, end - cnt[k], ~0u, 0u, ~0u, 0u};
                end = kActive | p >> 16;
                p += cnt[k] | 1u << 16;
            }
        }
        __syncthreads();
#pragma unroll 2
        for (uint32_t i = (uint32_t)tid; i < E; i += NT) {
            const uint2 x = entry(i);
            const uint32_t was = round ? tmp[i] : kActive | x.x >> c.sh;
            if (!(was & kActive)) continue;
            const uint32_t cell = was & 0xffffu, end = s.cur[cell];
            // from a place in kv to one in the bucket's order
            const uint32_t shift = round ? s.shift[was >> 16 & 0x7fffu] : 0u;
            if (end & kActive) {
                const uint32_t g = end & 0xffffu;
                if (round) s.crowd[g].fin = s.crowd[g].at + shift;   // the same from each of its entries
                tmp[i] = kActive | g << 16;
            } else {
                uint32_t q = cell ? s.cur[cell - 1u] : 0u;
                if (q & kActive) q = s.crowd[q & 0xffffu].at + s.crowd[q & 0xffffu].n;
                const uint64_t key = (uint64_t)x.x << 32 | x.y;
                uint32_t r = q;
                for (; q < end; ++q) r += s.kv[q] < key ? 1u : 0u;
                tmp[i] = r + shift;
            }
        }
        if (tot == 0u) return;   // block-uniform
        __syncthreads();
        // each group's bounds: a wave takes its share of kv
        const uint32_t share = (lim + kWaves - 1) / kWaves, k0 = (uint32_t)wave * share, k1 = k0 + share;
        for (uint32_t g0 = 0; g0 < ng; g0 += 64) {
            const uint32_t gl = min(g0 + (uint32_t)lane, ng - 1u);
            if (g0 + (uint32_t)lane < ng && (gl & (kWaves - 1)) == (uint32_t)wave)
                s.shift[gl] = s.crowd[gl].fin - s.crowd[gl].pre;
            const bool meets = g0 + (uint32_t)lane < ng && s.crowd[gl].at < k1 && s.crowd[gl].at + s.crowd[gl].n > k0;
            for (uint64_t left = __ballot(meets); left != 0ull; left &= left - 1ull) {
                Crowd &x = s.crowd[g0 + (uint32_t)(__ffsll((long long)left) - 1)];
                uint32_t dl = ~0u, dh = 0u, il = ~0u, ih = 0u;
                const uint32_t e = min(x.at + x.n, k1);
                for (uint32_t i = max(x.at, k0) + (uint32_t)lane; i < e; i += 64) {
                    const uint64_t key = s.kv[i];
                    dl = min(dl, (uint32_t)(key >> 32));
                    dh = max(dh, (uint32_t)(key >> 32));
                    il = min(il, (uint32_t)key);
                    ih = max(ih, (uint32_t)key);
                }
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) {
                    dl = min(dl, __shfl_xor(dl, o));
                    dh = max(dh, __shfl_xor(dh, o));
                    il = min(il, __shfl_xor(il, o));
                    ih = max(ih, __shfl_xor(ih, o));
                }
                if (lane == 0) {
                    atomicMin(&x.dlo, dl);
                    atomicMax(&x.dhi, dh);
                    atomicMin(&x.ilo, il);
                    atomicMax(&x.ihi, ih);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) s.cur[k * NT + tid] = 0u;
        __syncthreads();
        // sub-buckets by the entries before a group (and so its neighbour's
        // end where its own begin); conversions and products of the same
        // factor keep the order
        const float per = (float)kSub / (float)act;
#pragma unroll 2
        for (uint32_t i = (uint32_t)tid; i < E; i += NT) {
            const uint2 v = entry(i);
            const uint32_t was = tmp[i];
            if (!(was & kActive)) continue;
            const Crowd x = s.crowd[was >> 16 & 0x7fffu];
            const uint32_t b0 = (uint32_t)((float)x.pre * per), b1 = (uint32_t)((float)(x.pre + x.n) * per);
            const bool one = x.dlo == x.dhi;
            const uint32_t a = one ? v.y - x.ilo : v.x - x.dlo, range = one ? x.ihi - x.ilo : x.dhi - x.dlo;
            const float f = (float)(b1 - b0) / ((float)range + 1.0f);
            const uint32_t cell = b0 + min((uint32_t)((float)a * f), b1 - b0 - 1u);
            tmp[i] = was | cell;
            atomicAdd(&s.cur[cell], 1u);
        }
        __syncthreads();
        uint32_t sum = 0, all;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            cnt[k] = s.cur[tid * kPer + k];
            sum += cnt[k];
        }
        uint32_t o = bucket_scan<kWaves, uint32_t>(sum, s.scan, &all);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            s.cur[tid * kPer + k] = o;
            o += cnt[k];
        }
        __syncthreads();
#pragma unroll 2
        for (uint32_t i = (uint32_t)tid; i < E; i += NT) {
            const uint2 v = entry(i);
            const uint32_t was = tmp[i];
            if (was & kActive) s.kv[atomicAdd(&s.cur[was & 0xffffu], 1u)] = (uint64_t)v.x << 32 | v.y;
        }
        __syncthreads();
        lim = act;
    }
}

// The rest of bucket_sort where sub-buckets are crowded.
template <int CAP, int NT>
__device__ __attribute__((always_inline)) inline void bucket_crowded(const BucketIo &io, BucketLds<CAP, NT> &s,
                                                                     const uint4 *ent, uint32_t E,
                                                                     uint32_t pos0, unsigned long long key0,
                                                                     const Cut &c) {
    const int tid = threadIdx.x;
    uint32_t *tmp = io.didx + pos0;   // the bucket's part of the output, not yet written
    rank_crowded<CAP, NT>(s, ent, E, c, tmp);
    __syncthreads();
#pragma unroll 2
    for (uint32_t i = (uint32_t)tid; i < E; i += NT) {
        const uint4 x = ent[i];
        s.kv[tmp[i]] = (uint64_t)x.w << 32 | x.z;
    }
    __syncthreads();
    uint64_t *srect = reinterpret_cast<uint64_t *>(io.srect);
    for (uint32_t p = (uint32_t)tid; p < E; p += NT) srect[pos0 + p] = s.kv[p];
    __syncthreads();
    uint32_t *s_cnt = reinterpret_cast<uint32_t *>(s.kv), *s_idx = s_cnt + CAP;
#pragma unroll 2
    for (uint32_t i = (uint32_t)tid; i < E; i += NT) {
        const uint4 x = ent[i];
        const uint32_t p = tmp[i];
        s_cnt[p] = entry_keys(io, x);
        s_idx[p] = x.y;
    }
    __syncthreads();
    // exclusive prefix of the counts in sorted order, consecutive ones per thread
    const uint32_t per = (E + NT - 1) / NT, p0 = min((uint32_t)tid * per, E), p1 = min(p0 + per, E);
    uint32_t sum = 0, tot;
    for (uint32_t p = p0; p < p1; ++p) sum += s_cnt[p];
    uint32_t o = bucket_scan<NT / 64, uint32_t>(sum, s.scan, &tot);
    for (uint32_t p = p0; p < p1; ++p) {
        const uint32_t n = s_cnt[p];
        s_cnt[p] = o;
        o += n;
    }
    __syncthreads();
    for (uint32_t p = (uint32_t)tid; p < E; p += NT) {
        const uint32_t a = s_cnt[p], e = p + 1u < E ? s_cnt[p + 1u] : tot;
        io.didx[pos0 + p] = s_idx[p];
        io.offs[pos0 + p] = sat32(key0 + a);
        mark_key_blocks(io.kfirst, (uint32_t)key_blocks(io.key_cap), pos0 + p, key0 + a, e - a);
    }
}

// The bucket's E (<= NT IPT) entries, whose first comes at place pos0 of the
// order with its keys at key0.  The depths of a bucket lie between two
// neighbouring splitters and are spread about evenly there, so their
// differences to the least one, cut into 4 NT equal ranges, give sub-buckets
// of about one entry: placed by LDS counters, ranked inside by comparing
// (difference, index) with each other member.  (Three passes of an LDS radix
// sort took 45-100 us for 1.13M Gaussians, by the number of buckets.)  Where
// all depths are one, the indices take their place.  Where more than kCrowdMost
// entries share a range (planes seen head-on, two of them in one bucket), the
// compares would grow with their number squared: it ends there, returns false
// and leaves the rest to bucket_crowded, which is in the kernel once and not
// for each IPT.
template <int IPT, int CAP, int NT>
__device__ __attribute__((always_inline)) inline bool bucket_sort(const BucketIo &io, BucketLds<CAP, NT> &s,
                                                                  const uint4 *ent, uint32_t E, uint32_t pos0,
                                                                  unsigned long long key0, Cut &cut) {
    constexpr int kWaves = NT / 64, kSub = BucketLds<CAP, NT>::kSub;
    const int tid = threadIdx.x;
    uint4 v[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) v[j] = ent[min((uint32_t)(j * NT + tid), E - 1u)];
#pragma unroll
    for (int k = 0; k < kSub / NT; ++k) s.cur[k * NT + tid] = 0u;
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        lo = min(lo, v[j].x);
        hi = max(hi, v[j].x);
    }
    bucket_range<kWaves>(s.scan, lo, hi);
    const bool one_depth = lo == hi;   // block-uniform
    if (one_depth) {
        lo = 0xffffffffu;
        hi = 0u;
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            v[j].x = v[j].y;
            lo = min(lo, v[j].x);
            hi = max(hi, v[j].x);
        }
        bucket_range<kWaves>(s.scan, lo, hi);
    }
    const int bits = 32 - __clz((int)((hi - lo) | 1u));
    constexpr int kSubBits = 31 - __builtin_clz((unsigned)kSub);
    const int sh = bits > kSubBits ? bits - kSubBits : 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        v[j].x -= lo;
        if ((uint32_t)(j * NT + tid) < E) atomicAdd(&s.cur[v[j].x >> sh], 1u);
    }
    __syncthreads();
    uint32_t c4[kSub / NT], sum = 0, most = 0, tot;
#pragma unroll
    for (int k = 0; k < kSub / NT; ++k) {
        c4[k] = s.cur[tid * (kSub / NT) + k];
        sum += c4[k];
        most = max(most, c4[k]);
    }
    uint32_t o = bucket_scan<kWaves, uint32_t>(sum, s.scan, &tot);
#pragma unroll
    for (int k = 0; k < kSub / NT; ++k) {
        s.cur[tid * (kSub / NT) + k] = o;
        o += c4[k];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j)
        if ((uint32_t)(j * NT + tid) < E)
            s.kv[atomicAdd(&s.cur[v[j].x >> sh], 1u)] = (uint64_t)v[j].x << 32 | v[j].y;
    const bool crowded = __syncthreads_or(most > kCrowdMost) != 0;
    if (crowded) {   // block-uniform
        cut = Cut{lo, sh, one_depth};
        return false;
    }
    // (a counter now stands at its sub-bucket's end)
    uint32_t to[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        to[j] = 0u;
        if ((uint32_t)(j * NT + tid) < E) {
            const uint32_t b = v[j].x >> sh, end = s.cur[b];
            const uint64_t mine = (uint64_t)v[j].x << 32 | v[j].y;
            uint32_t q = b ? s.cur[b - 1u] : 0u;
            to[j] = q;
            for (; q < end; ++q) to[j] += s.kv[q] < mine ? 1u : 0u;
        }
    }
    __syncthreads();
    // everything goes to its place in LDS first and from there to memory in
    // whole lines (stored from here, every lane would write a line of its own)
    uint32_t *s_cnt = reinterpret_cast<uint32_t *>(s.kv), *s_idx = s_cnt + CAP;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        if ((uint32_t)(j * NT + tid) < E) {
            s_cnt[to[j]] = entry_keys(io, v[j]);
            s_idx[to[j]] = v[j].y;
        }
    }
    __syncthreads();
    // exclusive prefix of the counts in sorted order, consecutive ones per thread
    uint32_t x[IPT];
    sum = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t p = (uint32_t)(tid * IPT + j);
        x[j] = p < E ? s_cnt[p] : 0u;
        sum += x[j];
    }
    o = bucket_scan<kWaves, uint32_t>(sum, s.scan, &tot);
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t p = (uint32_t)(tid * IPT + j);
        if (p < E) s_cnt[p] = o;
        o += x[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t p = (uint32_t)(j * NT + tid);
        if (p < E) {
            const uint32_t a = s_cnt[p], e = p + 1u < E ? s_cnt[p + 1u] : tot;
            io.didx[pos0 + p] = s_idx[p];
            io.offs[pos0 + p] = sat32(key0 + a);
            mark_key_blocks(io.kfirst, (uint32_t)key_blocks(io.key_cap), pos0 + p, key0 + a, e - a);
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j)
        if ((uint32_t)(j * NT + tid) < E) s.kv[to[j]] = (uint64_t)v[j].w << 32 | v[j].z;
    __syncthreads();
    uint64_t *srect = reinterpret_cast<uint64_t *>(io.srect);
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t p = (uint32_t)(j * NT + tid);
        if (p < E) srect[pos0 + p] = s.kv[p];
    }
    return true;
}

// With the fewest items per thread (a power of two up to MAX, or 12: sixteen
// take more registers than a wave has here) that hold E.
template <int MAX, int CAP, int NT>
__device__ __attribute__((always_inline)) inline bool bucket_sort_for(const BucketIo &io, BucketLds<CAP, NT> &s,
                                                                      const uint4 *ent, uint32_t E, uint32_t pos0,
                                                                      unsigned long long key0, Cut &cut) {
    if constexpr (MAX > 1) {
        if (E <= (uint32_t)(MAX / 2 * NT))   // block-uniform
            return bucket_sort_for<MAX / 2, CAP, NT>(io, s, ent, E, pos0, key0, cut);
    }
    if constexpr (MAX == 16) {
        if (E <= (uint32_t)(12 * NT)) return bucket_sort<12, CAP, NT>(io, s, ent, E, pos0, key0, cut);
    }
    return bucket_sort<MAX, CAP, NT>(io, s, ent, E, pos0, key0, cut);
}

// Block b sorts bucket b if it holds more than MIN and at most CAP entries
// (the first launch of a frame, MIN = 0, also publishes its counters).
template <int CAP, int MIN, int NT>
__global__ __launch_bounds__(NT) void depth_buckets_kernel(BucketIo io) {
    constexpr int kWaves = NT / 64;
    __shared__ BucketLds<CAP, NT> s;
    __shared__ unsigned long long s_scan64[kWaves];
    const int tid = threadIdx.x, b = blockIdx.x;
    const uint32_t E = fill_of(io.fill[b]);
    if (MIN > 0 && E <= (uint32_t)MIN) return;   // block-uniform
    // fills of the buckets before this one, and of all
    unsigned long long pre = 0, all = 0;
    int over = 0;
    for (int k0 = 0; k0 < io.nb; k0 += 4 * NT) {
        uint64_t f[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + u * NT + tid;
            f[u] = k < io.nb ? io.fill[k] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            over |= fill_of(f[u]) > io.cap ? 1 : 0;
            all += f[u];
            if (k0 + u * NT + tid < b) pre += f[u];
        }
    }
    over = __syncthreads_or(over);
    (void)bucket_scan<kWaves, unsigned long long>(pre, s_scan64, &pre);
    if (MIN == 0 && b == 0) {   // block-uniform
        (void)bucket_scan<kWaves, unsigned long long>(all, s_scan64, &all);
        uint32_t surv = 0, newly = 0;
        const uint2 *pp = reinterpret_cast<const uint2 *>(io.pre_partial);
        for (int k0 = 0; k0 < io.n_pre; k0 += 8 * NT) {
            uint2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = k0 + u * NT + tid;
                v[u] = k < io.n_pre ? pp[k] : make_uint2(0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                surv += v[u].x;
                newly += v[u].y;
            }
        }
        (void)bucket_scan<kWaves, uint32_t>(surv, s.scan, &surv);
        (void)bucket_scan<kWaves, uint32_t>(newly, s.scan, &newly);
        if (tid == 0) {
            const uint32_t k32 = over ? 0u : sat32(all >> kFillBits);
            const uint32_t sorted = k32 <= io.key_cap ? k32 : 0u;
            io.cnt->n_visible = fill_of(all);
            io.cnt->n_keys = k32;
            io.cnt->n_sorted = sorted;
            io.cnt->n_survivors = surv;
            io.cnt->n_newly = newly;
            // n_selected was written by the tile selection
            publish_host(io.host, k32, surv, newly, io.cnt->n_selected, fill_of(all), sorted, over ? 1u : 0u,
                         io.tag);
        }
    }
    if (over || E == 0u || E > (uint32_t)CAP) return;   // block-uniform
    const uint4 *ent = io.entries + (size_t)b * io.cap;
    Cut cut;
    if (!bucket_sort_for<CAP / NT, CAP, NT>(io, s, ent, E, fill_of(pre), pre >> kFillBits, cut))
        bucket_crowded<CAP, NT>(io, s, ent, E, fill_of(pre), pre >> kFillBits, cut);
}

template <int IPT>
void scatter(const DepthPlan &dp, int n, const uint32_t *dkey, const ushort4 *rect, const uint32_t *sat,
             int TX, const DepthScratch &d, hipStream_t st) {
    const int per = kScatterThreads * IPT;
    const size_t lds = ((size_t)1 << dp.log_nb) * 16;
    depth_scatter_kernel<IPT><<<(n + per - 1) / per, kScatterThreads, lds, st>>>(
        n, dkey, rect, sat, TX, d.splitters, dp.nb, dp.log_nb, dp.cap,
        reinterpret_cast<unsigned long long *>(d.fill), d.entries);
}

}  // namespace

DepthScratch depth_scratch(const DepthPlan &dp, int n, void *entries, void *rest) {
    DepthScratch d{};
    d.entries = static_cast<uint4 *>(entries);
    d.splitters = static_cast<uint64_t *>(rest);
    d.fill = d.splitters + dp.nb;
    d.srect = reinterpret_cast<ushort4 *>(d.fill + dp.nb);
    d.samples = reinterpret_cast<uint32_t *>(d.srect + n);
    return d;
}

void launch_depth_samplesort(const DepthPlan &dp, const DepthScratch &d, int n, const uint32_t *dkey,
                             const ushort4 *rect, const uint32_t *sat, int TX, uint32_t *didx,
                             uint32_t *offs, uint32_t *kfirst, Counters *cnt, uint32_t cap,
                             const uint32_t *pre_partial, int n_pre, HostCounters *host, uint32_t tag,
                             hipStream_t st) {
    const auto split = [&](auto kernel, int per) {
        kernel<<<(dp.ns + per - 1) / per, kRankThreads, 0, st>>>(d.samples, dp.ns, dp.stride, n, dp.nb,
                                                                 d.splitters, d.fill);
    };
    static_assert(64 * kRankBlocks >= kDepthSamples, "the largest instance ranks every sample");
    if (dp.ns <= 16 * kRankBlocks) split(depth_splitters_kernel<4>, 16);
    else if (dp.ns <= 32 * kRankBlocks) split(depth_splitters_kernel<8>, 32);
    else split(depth_splitters_kernel<16>, 64);
    // about a block per CU: the more blocks, the more adds to each bucket's
    // counter, one after the other
    if (n <= 256 * kScatterThreads * 2) scatter<2>(dp, n, dkey, rect, sat, TX, d, st);
    else if (n <= 256 * kScatterThreads * 4) scatter<4>(dp, n, dkey, rect, sat, TX, d, st);
    else if (n <= 256 * kScatterThreads * 8) scatter<8>(dp, n, dkey, rect, sat, TX, d, st);
    else scatter<16>(dp, n, dkey, rect, sat, TX, d, st);
    const BucketIo io{d.fill, d.entries, dp.nb, dp.cap, sat, TX,  didx,        offs, kfirst,
                      d.srect, cnt,      host,  tag,    cap, pre_partial, n_pre};
    if (dp.cap <= (uint32_t)kBucketSmall) {
        depth_buckets_kernel<kBucketSmall, 0, 512><<<dp.nb, 512, 0, st>>>(io);
    } else if (dp.nb <= 256) {   // a block per CU whatever its LDS
        depth_buckets_kernel<kBucketMost, 0, 1024><<<dp.nb, 1024, 0, st>>>(io);
    } else {
        depth_buckets_kernel<kBucketShort, 0, 1024><<<dp.nb, 1024, 0, st>>>(io);
        depth_buckets_kernel<kBucketMost, kBucketShort, 1024><<<dp.nb, 1024, 0, st>>>(io);
    }
}

}  // namespace tgs

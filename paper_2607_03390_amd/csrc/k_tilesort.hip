// Stable LSD radix sort of a frame's Gaussian-tile keys by tile id
// (Sec. III-A), for grids of up to 65536 tiles whose Gaussian index leaves
// room for half a tile id beside it in 32 bits (tile_sort_plan; other frames
// take the general sort of k_sort.hip).
//
// The tile id is cut into a low and a high digit.  The emission writes, per
// key, the low digit as one byte and the payload (high digit << index bits |
// Gaussian index) as one word: 5 bytes.  The first pass sorts the payloads
// by the low digit, which is then no longer needed; the second by the high
// digit in the payload, and stores the Gaussian index alone.  Per key that is
// 27 bytes written and read over the emission and the two passes instead of
// the 52 of (tile id, index) word pairs and a last read of the sorted ids for
// the tile ranges.  Grids of up to 256 tiles take one pass.
//
// Second pass: its partitions do not straddle the segments of equal low
// digit (one block of the first pass lists them), so the key runs of a
// segment's first and last partition are where the keys of its tiles begin
// and end, and a partition's digit counts are tile counts.  The tile ranges
// are written by the blocks that scatter the keys, and the blend order of the
// tiles, which needs only their lengths, by eight more blocks of that launch.
//
// Each pass: an upsweep counts the digits of every partition (left out in the
// first pass where the emission has counted its blocks of 1024 keys), the
// column scan (k_sort.hip) turns the counts into offsets, the downsweep
// ranks and scatters each partition as k_sort.hip does (64-lane digit match,
// per-wave counters, staging in LDS in digit order).
#include "match.h"
#include "order.h"
#include "radix.h"
#include "tgs_internal.h"

namespace tgs {

namespace {

// Keys per thread: 1024-key partitions for sorts expected up to 2M keys
// (enough blocks to fill the chip), 5120-key ones above (longer runs per
// digit, fewer counts to scan).
constexpr int kIptSmall = 4;
constexpr int kIptLarge = 20;

// What the first pass leaves for the second: its partitions, each the keys
// [x, x + (y >> 8 & 0xffff)) of low digit y & 255; kFirstOf / kLastOf: the
// first and last of their segment.
static_assert(kOrderShares == 8, "one block per XCD");
constexpr uint32_t kFirstOf = 1u << 30, kLastOf = 1u << 31;
struct Segments {
    uint32_t n, pad;
    uint2 part[1];
};

// Digit counts of a partition: first pass from the digit bytes (whole words:
// a partition starts at a multiple of 1024 keys), second pass from the high
// digit of the payloads.
// The second pass's counts are also added to the tiles' lengths (contended
// by a segment's partitions only).
template <int IPT, bool SECOND>
__global__ __launch_bounds__(kSortThreads) void tile_upsweep_kernel(
    const uint8_t *__restrict__ dig, const uint32_t *__restrict__ pay, const uint32_t *n_dev,
    const Segments *seg, int shift, int lo_bits, int n_tiles, uint32_t *counts, uint32_t *tile_len) {
    constexpr uint32_t kTileKeys = kSortThreads * IPT;
    // counters per wave and, in the second pass, per lane & 3: the keys of one
    // tile column or row band share a few high digits, and lanes adding to one
    // address serialise (a street scene's 9.9M keys: 25.0 -> 18.0 us)
    constexpr int kCopies = SECOND ? 4 : 1;
    __shared__ uint32_t s_h[4 * kCopies][kRadix];
    const int tid = threadIdx.x, wave = tid >> 6;
    const int row = wave * kCopies + (tid & (kCopies - 1));
    const uint32_t part = blockIdx.x;
    uint32_t base = part * kTileKeys, n, lo = 0;
    if (SECOND) {
        if (part >= seg->n) return;   // block-uniform
        const uint2 p = seg->part[part];
        base = p.x;
        lo = p.y & 255u;
        n = p.y >> 8 & 0xffffu;
    } else {
        const uint32_t K = *n_dev;
        if (base >= K) return;   // block-uniform
        n = K - base < kTileKeys ? K - base : kTileKeys;
    }
#pragma unroll
    for (int w = 0; w < 4 * kCopies; ++w) s_h[w][tid] = 0u;
    if (SECOND) {
        const uint32_t *src = pay + base;
        uint32_t v[IPT];
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const uint32_t i = (uint32_t)(j * kSortThreads + tid);
            v[j] = src[i < n ? i : n - 1u] >> shift;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPT; ++j)
            if ((uint32_t)(j * kSortThreads + tid) < n) atomicAdd(&s_h[row][v[j]], 1u);
    } else {
        // words past the keys' last one are clamped to it
        const uint32_t *words = reinterpret_cast<const uint32_t *>(dig + base);
        const uint32_t last = (n - 1u) / 4u;
        uint32_t v[IPT / 4];
#pragma unroll
        for (int j = 0; j < IPT / 4; ++j) {
            const uint32_t i = (uint32_t)(j * kSortThreads + tid);
            v[j] = words[i < last ? i : last];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPT / 4; ++j) {
            const uint32_t i = 4u * (uint32_t)(j * kSortThreads + tid);
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (i + b < n) atomicAdd(&s_h[row][(v[j] >> (8 * b)) & 255u], 1u);
        }
    }
    __syncthreads();
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < 4 * kCopies; ++w) c += s_h[w][tid];
    counts[(size_t)part * kRadix + tid] = c;
    if (SECOND && c && tile_len) {
        const uint32_t t = (uint32_t)tid << lo_bits | lo;
        if (t < (uint32_t)n_tiles) atomicAdd(&tile_len[t], c);
    }
}

// Operands of the last pass: tile ranges and blend order.
struct LastIo {
    uint2 *ranges;
    const uint32_t *tile_len;   // lengths of the tiles' lists (NULL: no order)
    int n_tiles;
    OrderK order;
};

// One pass of the sort.  SECOND: the digit is payload >> shift (nbits wide)
// and the partitions are the segments'; else the digit byte.  LAST: the
// values stored are the Gaussian indices (payload's low `shift` bits), the
// first kOrderShares blocks order the tiles (if tile_len is given) and the
// others write the tile ranges; in a first pass of two, block 0 lists the
// second pass's partitions.
template <int IPT, bool SECOND, bool LAST>
__global__ __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(4))) void tile_downsweep_kernel(
    const uint8_t *__restrict__ dig, const uint32_t *__restrict__ pay, uint32_t *__restrict__ out,
    const uint32_t *n_dev, Segments *seg, int shift, int nbits, int lo_bits,
    const uint32_t *__restrict__ offsets, const uint32_t *__restrict__ chunk_sums, LastIo io) {
    constexpr uint32_t kTileKeys = kSortThreads * IPT;
    __shared__ uint32_t s_vals[kTileKeys];
    __shared__ uint8_t s_dig[SECOND ? 1 : kTileKeys];
    __shared__ uint32_t s_wh[4 * kRadix];   // per-wave digit counters, then wave prefixes
    __shared__ uint32_t s_gbase[kRadix];    // global start of the block's digit run, then
                                            // that minus the block-local start
    __shared__ uint32_t s_scan[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the first eight blocks (one per XCD, so block b of the others still
    // runs on XCD b mod 8) take the work beside the sort
    const bool aside = blockIdx.x < (uint32_t)kOrderShares;
    auto tile_at = [&](int i) { return io.order.tile_in ? io.order.tile_in[i] : i; };
    const int n_order = io.order.tile_in ? (int)*io.order.n_dev : io.n_tiles;
    if (SECOND && aside) {   // block-uniform
        if (io.tile_len)
            order_tiles_share<kSortThreads>(io.order, n_order, (int)blockIdx.x, kOrderShares, s_wh, tile_at,
                                            [&](int t) { return length_bucket(io.tile_len[t]); });
        return;
    }
    const uint32_t K = SECOND ? 0u : *n_dev;
    const uint32_t npa = SECOND ? seg->n : (K + kTileKeys - 1) / kTileKeys;
    uint32_t part = 0;
    if (!aside && (!xcd_partition(blockIdx.x - kOrderShares, npa, part) || part >= npa)) return;
    const uint32_t c_mine = part / chunk_len(npa);
    // digit tid: its total over all chunks and its sum over the chunks before this one
    uint32_t tot = 0, pre = 0;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
        const uint32_t v = chunk_sums[c * kRadix + tid];
        tot += v;
        if ((uint32_t)c < c_mine) pre += v;
    }
    const uint32_t first = block_exclusive_scan256<uint32_t>(tot, s_scan);   // start of digit tid
    if (!SECOND && aside) {   // block-uniform; also when there is nothing to sort
        if (LAST) {
            // one pass: a digit is a tile
            if (blockIdx.x == 0 && tid < io.n_tiles && tot > 0u)
                io.ranges[tid] = make_uint2(first, first + tot);
            s_gbase[tid] = tot;
            __syncthreads();
            if (io.tile_len)
                order_tiles_share<kSortThreads>(io.order, n_order, (int)blockIdx.x, kOrderShares, s_wh,
                                                tile_at, [&](int t) { return length_bucket(s_gbase[t]); });
        } else if (blockIdx.x == 0) {
            const uint32_t np = (tot + kTileKeys - 1) / kTileKeys;
            const uint32_t p0 = block_exclusive_scan256<uint32_t>(np, s_scan);
            if (tid == kRadix - 1) seg->n = p0 + np;
            for (uint32_t k = 0; k < np; ++k) {
                const uint32_t left = tot - k * kTileKeys, n = left < kTileKeys ? left : kTileKeys;
                seg->part[p0 + k] = make_uint2(first + k * kTileKeys,
                                               (uint32_t)tid | n << 8 | (k == 0 ? kFirstOf : 0u) |
                                                   (k + 1 == np ? kLastOf : 0u));
            }
        }
        return;
    }
    uint32_t base = part * kTileKeys, n, sp = 0;
    if (SECOND) {
        const uint2 p = seg->part[part];
        base = p.x;
        sp = p.y;
        n = p.y >> 8 & 0xffffu;
    } else {
        n = K - base < kTileKeys ? K - base : kTileKeys;
    }
    // issue every global load of the block before the next barrier (uniform
    // base, 32-bit offsets)
    const uint32_t w0 = (uint32_t)wave * (64u * IPT) + (uint32_t)lane;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    const uint32_t *src = pay + base;
    const uint8_t *src_dig = dig + base;
    uint32_t val[IPT], rank[IPT];   // rank: the digit in the low byte, the rank above
    bool ok[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t i = w0 + 64u * j;
        ok[j] = i < n;
        const uint32_t ic = ok[j] ? i : n - 1u;
        val[j] = src[ic];
        if (!SECOND) rank[j] = src_dig[ic];
    }
    const uint32_t off_mine = offsets[(size_t)part * kRadix + tid];
#pragma unroll
    for (int w = 0; w < 4; ++w) s_wh[w * kRadix + tid] = 0u;
    const uint32_t gstart = first + pre + off_mine;   // global start of the block's digit run
    __syncthreads();
    constexpr int kG = IPT % 5 == 0 ? 5 : 4;
    static_assert(IPT % kG == 0, "items per thread must be a multiple of the group");
#pragma unroll
    for (int j0 = 0; j0 < IPT; j0 += kG) {
        uint32_t dg[kG];
        uint64_t pm[kG];
#pragma unroll
        for (int g = 0; g < kG; ++g) {
            dg[g] = SECOND ? val[j0 + g] >> shift : rank[j0 + g];
            pm[g] = __ballot(ok[j0 + g]);
        }
        match_digits<kG>(dg, nbits, pm);
#pragma unroll
        for (int g = 0; g < kG; ++g) {
            const int j = j0 + g;
            const uint32_t d = dg[g];
            const uint64_t peers = pm[g];
            const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
            uint32_t before = 0;
            if (ok[j]) before = s_wh[wave * kRadix + d];
            __builtin_amdgcn_wave_barrier();
            if (ok[j] && below == 0) s_wh[wave * kRadix + d] = before + (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
            rank[j] = (before + below) << 8 | d;
            // the digit is taken from here again below: kept beside it (and
            // its counter's address) it would cost two more registers an item
            __asm__ volatile("" : "+v"(rank[j]));
        }
    }
    __syncthreads();
    const uint32_t c0 = s_wh[tid], c1 = s_wh[kRadix + tid], c2 = s_wh[2 * kRadix + tid],
                   c3 = s_wh[3 * kRadix + tid];
    const uint32_t total = c0 + c1 + c2 + c3;
    if (SECOND) {
        // tile (tid, low digit): its keys begin in the segment's first
        // partition and end in its last
        const uint32_t t = (uint32_t)tid << lo_bits | (sp & 255u);
        if (tid < (1 << nbits) && t < (uint32_t)io.n_tiles) {
            if (sp & kFirstOf) io.ranges[t].x = gstart;
            if (sp & kLastOf) io.ranges[t].y = gstart + total;
        }
    }
    // (the scan's barriers also order the counter reads above before the
    // writes below)
    const uint32_t dstart = block_exclusive_scan256<uint32_t>(total, s_scan);
    s_wh[tid] = dstart;
    s_wh[kRadix + tid] = dstart + c0;
    s_wh[2 * kRadix + tid] = dstart + c0 + c1;
    s_wh[3 * kRadix + tid] = dstart + c0 + c1 + c2;
    s_gbase[tid] = gstart - dstart;
    __syncthreads();
#pragma unroll
    for (int j0 = 0; j0 < IPT; j0 += kG) {
#pragma unroll
        for (int g = 0; g < kG; ++g) {
            const int j = j0 + g;
            const uint32_t d = rank[j] & 255u;
            const uint32_t pos = s_wh[wave * kRadix + d] + (rank[j] >> 8);
            if (ok[j]) {
                s_vals[pos] = val[j];
                if (!SECOND) s_dig[pos] = (uint8_t)d;
            }
        }
    }
    __syncthreads();
    const uint32_t imask = shift < 32 ? (1u << shift) - 1u : 0xffffffffu;
#pragma unroll 1
    for (int j0 = 0; j0 < IPT; j0 += kG) {
        uint32_t sv[kG], od[kG];
#pragma unroll
        for (int g = 0; g < kG; ++g) {
            const uint32_t i = (uint32_t)((j0 + g) * kSortThreads + tid);
            sv[g] = s_vals[i];
            od[g] = i < n ? (SECOND ? sv[g] >> shift : (uint32_t)s_dig[i]) : 0u;
        }
#pragma unroll
        for (int g = 0; g < kG; ++g) od[g] = s_gbase[od[g]];
#pragma unroll
        for (int g = 0; g < kG; ++g) {
            const uint32_t i = (uint32_t)((j0 + g) * kSortThreads + tid);
            if (i < n) out[od[g] + i] = LAST ? sv[g] & imask : sv[g];
        }
    }
}

template <int IPT>
int run(const TileSortPlan &tp, uint32_t cap, const uint32_t *n_dev, const uint8_t *dig, uint32_t *pay,
        uint32_t *pay_alt, uint32_t *scratch, uint32_t *segments, bool counted, uint2 *ranges,
        uint32_t *tile_len, int n_tiles, const OrderK &order, hipStream_t st) {
    constexpr uint32_t kTileKeys = kSortThreads * IPT;
    uint32_t *sums = scratch, *table = sort_count_rows(scratch);
    Segments *seg = reinterpret_cast<Segments *>(segments);
    const LastIo io{ranges, tile_len, n_tiles, order};
    const uint32_t np = cap ? (cap + kTileKeys - 1) / kTileKeys : 1u;
    if (!counted)
        tile_upsweep_kernel<IPT, false><<<np, kSortThreads, 0, st>>>(dig, pay, n_dev, seg, 0, tp.lo,
                                                                      n_tiles, table, tile_len);
    launch_colscan(n_dev, cap, kTileKeys, np, 1, table, sums, st);
    const uint32_t grid = (np + 7) / 8 * 8 + kOrderShares;   // whole rounds of eight
    if (tp.hi == 0) {
        tile_downsweep_kernel<IPT, false, true><<<grid, kSortThreads, 0, st>>>(
            dig, pay, pay_alt, n_dev, seg, tp.index_bits, tp.lo, tp.lo, table, sums, io);
        return 1;
    }
    tile_downsweep_kernel<IPT, false, false><<<grid, kSortThreads, 0, st>>>(
        dig, pay, pay_alt, n_dev, seg, tp.index_bits, tp.lo, tp.lo, table, sums, io);
    // every low digit may end in a partition of its own
    const uint32_t np2 = np + (1u << tp.lo);
    tile_upsweep_kernel<IPT, true><<<np2, kSortThreads, 0, st>>>(dig, pay_alt, n_dev, seg, tp.index_bits,
                                                                 tp.lo, n_tiles, table, tile_len);
    launch_colscan(&seg->n, np2, 1, np2, 1, table, sums, st);
    tile_downsweep_kernel<IPT, true, true><<<(np2 + 7) / 8 * 8 + kOrderShares, kSortThreads, 0, st>>>(
        dig, pay_alt, pay, n_dev, seg, tp.index_bits, tp.hi, tp.lo, table, sums, io);
    return 0;
}

}  // namespace

TileSortPlan tile_sort_plan(int n, int bits) {
    TileSortPlan p{};
    p.bits = bits;
    while (p.index_bits < 32 && ((uint64_t)1 << p.index_bits) < (uint64_t)(n > 0 ? n : 1)) p.index_bits += 1;
    p.lo = bits <= 8 ? (bits > 0 ? bits : 1) : (bits + 1) / 2;
    p.hi = bits > 8 ? bits - p.lo : 0;
    p.packed = bits <= 16 && p.index_bits + p.hi <= 32;
    return p;
}

size_t tile_sort_segment_words(uint32_t max_keys) {
    const size_t np = ((size_t)max_keys + kSortThreads * kIptSmall - 1) / (kSortThreads * kIptSmall);
    return 2 + 2 * (np + kRadix);
}

bool tile_sort_small(uint32_t cap, uint32_t n_hint) { return (n_hint < cap ? n_hint : cap) <= (2u << 20); }

int launch_tile_sort(const TileSortPlan &tp, uint32_t cap, uint32_t n_hint, const uint32_t *n_dev,
                     const uint8_t *dig, uint32_t *pay, uint32_t *pay_alt, uint32_t *scratch,
                     uint32_t *segments, bool counted, uint2 *ranges, uint32_t *tile_len, int n_tiles,
                     const OrderK &order, hipStream_t st) {
    if (order_apart(n_hint)) tile_len = nullptr;
    if (tile_sort_small(cap, n_hint))
        return run<kIptSmall>(tp, cap, n_dev, dig, pay, pay_alt, scratch, segments, counted, ranges,
                              tile_len, n_tiles, order, st);
    return run<kIptLarge>(tp, cap, n_dev, dig, pay, pay_alt, scratch, segments, counted, ranges, tile_len,
                          n_tiles, order, st);
}

}  // namespace tgs

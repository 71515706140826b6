// Gaussian-tile duplication (Sec. III-A) around the two sorts of a frame:
//  - key emission in depth order, a fixed slice of output keys per block with
//    coalesced stores (owners from a search over the sorted offsets and an
//    LDS max-scan);
//  - per-tile [start, end) ranges of the tile-sorted keys and the blend
//    order of the tiles.
// Counts stay on the device, so nothing here needs a host round trip.
#include "order.h"
#include "tgs_internal.h"

namespace tgs {

namespace {

// Row and column of key r of a rectangle w tiles wide (r < 2^20, w <= 1024:
// the quotient of the hardware reciprocal is off by at most one).
__device__ inline void divide_row(uint32_t r, uint32_t w, uint32_t &row, uint32_t &col) {
    uint32_t q = (uint32_t)((float)r * __builtin_amdgcn_rcpf((float)w));
    int rem = (int)(r - q * w);
    if (rem < 0) {
        q -= 1;
        rem += (int)w;
    } else if (rem >= (int)w) {
        q += 1;
        rem -= (int)w;
    }
    row = q;
    col = (uint32_t)rem;
}

// The keys of one Gaussian in order: its rectangle's tiles row by row, or
// (sat != NULL) the selected ones among them.  seek(r) goes to its r-th key,
// next() to the one after (the Gaussian has it).
struct KeyWalk {
    ushort4 rc;
    int tx, ty;
    int pos, end;   // sat: entries of the row's selected columns, current and last + 1
};

__device__ inline void key_seek(KeyWalk &k, uint32_t r, const uint32_t *sat, const int *sel_cols, int TX) {
    const ushort4 rc = k.rc;
    if (!sat) {
        uint32_t row, col;
        divide_row(r, (uint32_t)(rc.z - rc.x + 1), row, col);
        k.tx = (int)rc.x + (int)col;
        k.ty = (int)rc.y + (int)row;
        return;
    }
    // the row holding the r-th selected tile, by bisection on the summed area
    // table (needles cross hundreds of tile rows)
    const size_t s = (size_t)(TX + 1);
    auto upto = [&](int y) { return sat[y * s + rc.z + 1] - sat[y * s + rc.x]; };   // in rows below y
    const uint32_t base = upto(rc.y);
    int lo = rc.y, hi = rc.w;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (upto(mid + 1) - base > r) hi = mid;
        else lo = mid + 1;
    }
    const uint32_t *row = sat + lo * s, *below = row + s;
    const uint32_t a0 = row[rc.x], a1 = row[rc.z + 1], b0 = below[rc.x], b1 = below[rc.z + 1];
    k.ty = lo;
    k.pos = (int)(b0 - a0 + (r - (a1 - a0 - base)));
    k.end = (int)(b1 - a1);
    k.tx = sel_cols[(size_t)lo * TX + k.pos];
}

__device__ inline void key_next(KeyWalk &k, uint32_t r, const uint32_t *sat, const int *sel_cols, int TX) {
    if (!sat) {
        k.tx += 1;
        if (k.tx > (int)k.rc.z) {
            k.tx = k.rc.x;
            k.ty += 1;
        }
    } else if (k.pos + 1 < k.end) {
        k.pos += 1;
        k.tx = sel_cols[(size_t)k.ty * TX + k.pos];
    } else {
        key_seek(k, r, sat, sel_cols, TX);
    }
}

// Inputs of key generation: the cnt->n_visible Gaussians in emission order
// (didx), the start of each one's keys (offs, strictly increasing: every
// emitted Gaussian has keys), the owner of every kKeyBlock-th key (kfirst),
// and the tile rectangles / selection.
struct DupIo {
    const Counters *cnt;
    const uint32_t *didx;
    const uint32_t *offs;
    const uint32_t *kfirst;
    const ushort4 *rect;
    bool rect_sorted;   // in emission order, not by index
    const uint32_t *sat;
    const int *sel_cols;
    int TX;
    int n_tiles;
    uint2 *ranges;       // cleared by the emission, as the tiles' lengths
    uint32_t *tile_len;  // (packed keys)
    uint32_t *rows;  // optional: counts of the low digit in each block's keys
    int lo_bits;     // packed keys: width of the low digit
    int index_bits;  // packed keys: where the high digit starts in the payload
};

// Window of the Gaussians owning output positions [P0, P1) (P0 a multiple
// of kKeyBlock, P1 - P0 <= KD): from j0, the owner of P0, to the owner of
// P1 (the next block's first key) or, for the block holding the last key K,
// to the last Gaussian.  Entry k >= 1 starts at or after P0 + k (strictly
// increasing offsets), so at most KD entries can start before P1.
template <int KD>
__device__ inline void dup_window(const DupIo &io, uint32_t P0, uint32_t P1, uint32_t K,
                                  uint32_t V, uint32_t &j0, uint32_t &nw) {
    j0 = io.kfirst[P0 / kKeyBlock];
    const uint32_t jn = P1 < K ? io.kfirst[P1 / kKeyBlock] + 1u : V;
    nw = jn - j0 < (uint32_t)KD ? jn - j0 : (uint32_t)KD;
}

// Owners of the output positions [P0, P1) by a block of NT threads: s_off[k]
// / s_g[k] = start and Gaussian index of window entry k (those starting
// before P1), own[i] = the window entry owning position P0 + kPer tid + i
// (kPer consecutive positions per thread; past P1: the last entry), j0 = the
// emission position of entry 0.  The window is read in one step (every load
// in flight at once).
template <int KD, int NT>
__device__ inline void dup_owners(const DupIo &io, uint32_t P0, uint32_t P1, uint32_t K,
                                  uint32_t V, int *s_mark, uint32_t *s_off, uint32_t *s_g,
                                  int *s_wmax, int (&own)[KD / NT], uint32_t &j0) {
    static_assert(KD % NT == 0 && KD % kKeyBlock == 0, "whole steps and key blocks");
    constexpr int kPer = KD / NT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t nw;
    dup_window<KD>(io, P0, P1, K, V, j0, nw);
    // clamped indices, no branches: every load is issued before the first wait
    uint32_t o[kPer], g[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const uint32_t k = (uint32_t)(tid + NT * i), kc = k < nw ? k : nw - 1u;
        o[i] = io.offs[j0 + kc];
        g[i] = io.didx[j0 + kc];
    }
    for (int k = tid; k < KD; k += NT) s_mark[k] = -1;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int k = tid + NT * i;
        if ((uint32_t)k < nw && (k == 0 || o[i] < P1)) {
            s_off[k] = o[i];
            s_g[k] = g[i];
            s_mark[k == 0 ? 0 : (int)(o[i] - P0)] = k;
        }
    }
    __syncthreads();
    // inclusive max-scan of the marks
    int m = -1;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        m = max(m, s_mark[kPer * tid + i]);
        own[i] = m;
    }
    int inc = m;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(inc, d);
        if (lane >= d) inc = max(inc, t);
    }
    int ex = __shfl_up(inc, 1);
    if (lane == 0) ex = -1;
    if (lane == 63) s_wmax[wave] = inc;
    __syncthreads();
    for (int w = 0; w < wave; ++w) ex = max(ex, s_wmax[w]);
#pragma unroll
    for (int i = 0; i < kPer; ++i) own[i] = max(own[i], ex);
}

// Block b emits output keys [1024 b, 1024 b + 1024), four consecutive ones per
// thread (one 16-byte store of indices or payloads, one store of tile ids or
// digits), whatever the Gaussians' key counts: a Gaussian spanning thousands
// of tiles is spread over many blocks instead of holding one wave.  Owners
// of the positions come from the key-block table and the window of Gaussians
// starting inside the block (dup_owners).  A thread finds the tile of its
// first key from the rank inside the owner's rectangle; the next ones of the
// same owner follow it along the row.  Past the key capacity
// (cnt->n_sorted == 0 with keys) nothing is emitted: the host grows the
// buffers and renders the frame again.  With io.rows, the block also counts
// its keys' low digits into row blockIdx.x (LDS counters per wave), so that
// the tile sort's first pass needs no counting launch of its own.
constexpr int kDupKeys = kKeyBlock;

template <bool PACKED>
__global__ __launch_bounds__(256) void duplicate_kernel(DupIo io, uint32_t *tkey, uint32_t *tval) {
    __shared__ int s_mark[kDupKeys];
    __shared__ uint32_t s_off[kDupKeys];
    __shared__ uint32_t s_g[kDupKeys];
    __shared__ int s_wmax[4];
    __shared__ uint32_t s_hist[4][256];
    const int tid = threadIdx.x;
    for (int t = blockIdx.x * blockDim.x + tid; t < io.n_tiles; t += gridDim.x * blockDim.x) {
        io.ranges[t] = make_uint2(0u, 0u);
        if (PACKED) io.tile_len[t] = 0u;
    }
    const uint32_t V = io.cnt->n_visible, K = io.cnt->n_sorted;
    const uint32_t P0 = blockIdx.x * (uint32_t)kDupKeys;
    if (K == 0u || P0 >= K) return;   // block-uniform
    if (PACKED && io.rows) {
#pragma unroll
        for (int w = 0; w < 4; ++w) s_hist[w][tid] = 0u;   // ordered by dup_owners' barriers
    }
    const uint32_t P1 = K - P0 < (uint32_t)kDupKeys ? K : P0 + kDupKeys;
    constexpr int kPer = kDupKeys / 256;
    static_assert(kPer == 4, "four keys per 16-byte store");
    int own[kPer];
    uint32_t j0;
    dup_owners<kDupKeys, 256>(io, P0, P1, K, V, s_mark, s_off, s_g, s_wmax, own, j0);
    // positions past the keys take the last key's (no branch before the
    // stores, so every rectangle load is in flight together)
    const uint32_t p = P0 + (uint32_t)(kPer * tid);
    uint32_t g[kPer], r[kPer], key[kPer];
    ushort4 rc[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t pc = p + k < P1 ? p + k : P1 - 1u;
        g[k] = s_g[own[k]];
        r[k] = pc - s_off[own[k]];
        rc[k] = io.rect[io.rect_sorted ? j0 + (uint32_t)own[k] : g[k]];
    }
    KeyWalk walk;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (k == 0 || own[k] != own[k - 1]) {
            walk.rc = rc[k];
            key_seek(walk, r[k], io.sat, io.sel_cols, io.TX);
        } else if (p + k < P1) {
            key_next(walk, r[k], io.sat, io.sel_cols, io.TX);
        }
        key[k] = (uint32_t)(walk.ty * io.TX + walk.tx);
    }
    const uint32_t lmask = PACKED ? (1u << io.lo_bits) - 1u : 0u;
    uint32_t val[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        val[k] = PACKED ? g[k] | (key[k] >> io.lo_bits) << (io.index_bits & 31) : g[k];
    if (p + kPer <= P1) {
        *reinterpret_cast<uint4 *>(tval + p) = make_uint4(val[0], val[1], val[2], val[3]);
        if (PACKED)
            reinterpret_cast<uint32_t *>(tkey)[p / 4] = (key[0] & lmask) | (key[1] & lmask) << 8 |
                                                        (key[2] & lmask) << 16 | (key[3] & lmask) << 24;
        else
            *reinterpret_cast<uint4 *>(tkey + p) = make_uint4(key[0], key[1], key[2], key[3]);
    } else {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (p + k < P1) {
                tval[p + k] = val[k];
                if (PACKED) reinterpret_cast<uint8_t *>(tkey)[p + k] = (uint8_t)(key[k] & lmask);
                else tkey[p + k] = key[k];
            }
        }
    }
    if (PACKED && io.rows) {
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (p + k < P1) atomicAdd(&s_hist[tid >> 6][key[k] & lmask], 1u);
        __syncthreads();
        io.rows[(size_t)blockIdx.x * 256 + tid] = s_hist[0][tid] + s_hist[1][tid] + s_hist[2][tid] +
                                                  s_hist[3][tid];
    }
}

__global__ __launch_bounds__(256) void ranges_zero_kernel(int n_tiles, uint2 *ranges, uint32_t *tile_len) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_tiles) return;
    ranges[t] = make_uint2(0u, 0u);
    if (tile_len) tile_len[t] = 0u;
}

// Four consecutive sorted keys per thread (one 16-byte load) and the key on
// either side: the thread writes the start / end of every tile run that
// begins / ends among its four.
__global__ __launch_bounds__(256) void ranges_kernel(const Counters *cnt, const uint32_t *keys,
                                                     uint2 *ranges) {
    const uint64_t K = cnt->n_sorted;
    const uint64_t G = (K + 3) / 4;
    for (uint64_t g = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; g < G;
         g += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t k0 = 4 * g;
        uint32_t t[4];
        if (k0 + 4 <= K) {
            const uint4 v = *reinterpret_cast<const uint4 *>(keys + k0);
            t[0] = v.x;
            t[1] = v.y;
            t[2] = v.z;
            t[3] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) t[j] = k0 + j < K ? keys[k0 + j] : 0xffffffffu;
        }
        const uint32_t prev = k0 > 0 ? keys[k0 - 1] : 0xffffffffu;
        const uint32_t next = k0 + 4 < K ? keys[k0 + 4] : 0xffffffffu;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t k = k0 + j;
            if (k >= K) break;
            const uint32_t tp = j == 0 ? prev : t[j - 1];
            const uint32_t tn = j == 3 ? next : t[j + 1];
            if (k == 0 || tp != t[j]) ranges[t[j]].x = (uint32_t)k;
            if (k == K - 1 || tn != t[j]) ranges[t[j]].y = (uint32_t)(k + 1);
        }
    }
}

__global__ __launch_bounds__(256) void order_tiles_kernel(OrderK o) {
    __shared__ uint32_t s_cnt[order_lds_words(256)];
    order_tiles_share<256>(
        o, o.n_dev ? (int)*o.n_dev : o.n_host, (int)blockIdx.x, (int)gridDim.x, s_cnt,
        [&](int i) { return o.tile_in ? o.tile_in[i] : i; },
        [&](int t) {
            const uint2 r = o.ranges[t];
            return length_bucket(r.y - r.x);
        });
}

}  // namespace

void launch_duplicate(int n, uint32_t cap, const Counters *cnt, const uint32_t *didx,
                      const uint32_t *offs, const uint32_t *kfirst, const ushort4 *rect,
                      bool rect_sorted, const uint32_t *sat, const int *sel_cols, int TX, int n_tiles,
                      const TileSortPlan &tp, uint32_t *tkey, uint32_t *tval, uint2 *ranges,
                      uint32_t *tile_len, uint32_t *rows, hipStream_t st) {
    if (n <= 0 || cap == 0) {
        ranges_zero_kernel<<<(n_tiles + 255) / 256, 256, 0, st>>>(n_tiles, ranges,
                                                                 tp.packed ? tile_len : nullptr);
        return;
    }
    const uint32_t blocks = (cap + kDupKeys - 1) / kDupKeys;
    const DupIo io{cnt, didx, offs, kfirst, rect, rect_sorted, sat, sel_cols, TX, n_tiles, ranges,
                   tile_len, rows, tp.lo, tp.index_bits};
    if (tp.packed) duplicate_kernel<true><<<blocks, 256, 0, st>>>(io, tkey, tval);
    else duplicate_kernel<false><<<blocks, 256, 0, st>>>(io, tkey, tval);
}

void launch_ranges(uint32_t cap, const Counters *cnt, const uint32_t *keys, uint2 *ranges,
                   hipStream_t st) {
    // sized for the key capacity (the key count is on the device), at most
    // 65535 blocks, grid-stride beyond
    const uint64_t groups = ((uint64_t)cap + 3) / 4;
    const uint32_t blocks = (uint32_t)((groups + 255) / 256 < 65535u ? (groups + 255) / 256 : 65535u);
    if (cap > 0) ranges_kernel<<<blocks, 256, 0, st>>>(cnt, keys, ranges);
}

void launch_order_tiles(const OrderK &o, hipStream_t st) {
    if (o.n_host > 0) order_tiles_kernel<<<kOrderShares, 256, 0, st>>>(o);
}

}  // namespace tgs

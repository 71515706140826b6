// Temporal kernels of a TemporalGS frame (Sec. III-C..E):
//  - forward warp of the temporal geometry buffer into the current view
//    (Eq. 3): nearest destination pixel, minimum depth and maximum standard
//    deviation by integer atomics on the float bits (both are non-negative,
//    so unsigned order is float order and the result is order-independent);
//  - depth fill, backward correspondence query and unmatched tiles, one
//    block per tile with a block-wide OR (fill_query.h; with the
//    full-resolution geometry buffer the preprocess launch runs it);
//  - occluded tiles of the newly visible Gaussians, one wave per
//    (Gaussian, tile) pair with a wave ballot over the tile's 256 pixels,
//    the pairs of 1024 Gaussians dealt out over the four waves of a block;
//  - tile selection and compaction in one launch, one block per tile row,
//    including the summed area table of the mask used by the key counts.
// (The stitching of the tiles that are not re-rendered, Eq. 4, runs in the
// blend launch: stitch.h.)
// All of these are HBM- or latency-bound; none is a dense contraction.
#include "fill_query.h"
#include "tgs_internal.h"

namespace tgs {

namespace {

__global__ __launch_bounds__(256) void temporal_init_kernel(int n_px, float *dmin, float *smax) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n_px) {
        dmin[k] = kNoHit;
        smax[k] = 0.0f;
    }
}

__global__ __launch_bounds__(256) void forward_warp_kernel(WarpK w, const float *__restrict__ D,
                                                           const float *__restrict__ S, float *dmin,
                                                           float *smax) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= w.W * w.H) return;
    const float d = D[q];
    if (d == kNoHit) return;
    const int x = q % w.W, y = q / w.W;
    const float rx = ((float)x - w.kref[2]) / w.kref[0];
    const float ry = ((float)y - w.kref[3]) / w.kref[1];
    const float Px = d * rx, Py = d * ry, Pz = d;
    const float *M = w.M;
    const float X = ((M[0] * Px + M[1] * Py) + M[2] * Pz) + M[3];
    const float Y = ((M[4] * Px + M[5] * Py) + M[6] * Pz) + M[7];
    const float Z = ((M[8] * Px + M[9] * Py) + M[10] * Pz) + M[11];
    if (!(Z > w.z_near)) return;
    const float u = w.kcur[0] * (X / Z) + w.kcur[2];
    const float v = w.kcur[1] * (Y / Z) + w.kcur[3];
    const float xf = floorf(u + 0.5f), yf = floorf(v + 0.5f);
    if (!(xf >= 0.0f && xf <= (float)(w.W - 1) && yf >= 0.0f && yf <= (float)(w.H - 1))) return;
    const int p = (int)yf * w.W + (int)xf;
    atomicMin(reinterpret_cast<unsigned int *>(dmin + p), __float_as_uint(Z));
    atomicMax(reinterpret_cast<unsigned int *>(smax + p), __float_as_uint(S[q]) & 0x7fffffffu);
}

__global__ __launch_bounds__(256) void fill_query_kernel(FillK f) { fill_query_tile(f, blockIdx.x); }

// value of x in lane j (j uniform across the wave)
__device__ inline float lane_f(float x, int j) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), j));
}

// Tiles that Gaussian i can reach with alpha >= 1/255: its rectangle cut to
// the tiles meeting the box of the alpha >= 1/255 ellipse (enlarged by 0.2%
// + 0.05 px, from the record; negative half extents: alpha < 1/255
// everywhere).  No pixel outside that box can reach the threshold.  Returns
// the number of tiles (0: none) and the first column and row and the column
// count in *box.
__device__ inline uint32_t occ_box(int i, const float4 *g, const ushort4 *rect, int3 *box) {
    const ushort4 r = rect[i];
    const float4 a = g[4 * (size_t)i];
    const float hx = g[4 * (size_t)i + 2].w, hy = g[4 * (size_t)i + 1].w;
    if (r.x > r.z || r.y > r.w || !(hx >= 0.0f)) return 0u;
    const int ex0 = max((int)r.x, (int)ceilf((a.x - hx - 15.0f) * 0.0625f));
    const int ex1 = min((int)r.z, (int)floorf((a.x + hx) * 0.0625f));
    const int ey0 = max((int)r.y, (int)ceilf((a.y - hy - 15.0f) * 0.0625f));
    const int ey1 = min((int)r.w, (int)floorf((a.y + hy) * 0.0625f));
    if (ex0 > ex1 || ey0 > ey1) return 0u;
    *box = make_int3(ex0, ey0, ex1 - ex0 + 1);
    return (uint32_t)((ex1 - ex0 + 1) * (ey1 - ey0 + 1));
}

constexpr int kOccThreads = 256;
constexpr int kOccPer = 4;                                 // consecutive Gaussians per thread
constexpr int kOccBlock = kOccThreads * kOccPer;           // 1024 Gaussians per block
constexpr int kOccWaves = kOccThreads / 64;

// Exclusive scan across a block of kOccThreads threads, one value each;
// *total = the block's sum.
__device__ inline uint32_t occ_block_scan(uint32_t v, uint32_t *s_wave, uint32_t *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int x = 0; x < kOccWaves; ++x) {
        const uint32_t c = s_wave[x];
        if (x < wave) off += c;
        tot += c;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// One block per 1024 Gaussians, four consecutive ones per thread (a launch
// of few waves: most blocks find no newly visible Gaussian).  The newly
// visible ones that can reach a tile are compacted in LDS with the start of
// their (Gaussian, tile) pairs (two block scans, index order).  Wave w takes
// the pairs p = w (mod 4), 64 at a time: lane
// l finds the owner and tile of its pair (the searches run side by side),
// then the wave tests the pairs one after another with their data broadcast
// from the lanes: each lane tests four pixel centres and a ballot marks the
// tile.  Dealing the pairs out one by one spreads a block's pairs, however
// few Gaussians hold them, evenly over its four waves.  Marks are plain
// byte stores of 1, so concurrent writers agree.
__global__ __launch_bounds__(kOccThreads) void occluded_kernel(WarpK w, int n,
                                                               const uint8_t *__restrict__ status,
                                                               const float4 *__restrict__ g,
                                                               const ushort4 *__restrict__ rect,
                                                               uint8_t *oc) {
    __shared__ uint32_t s_idx[kOccBlock];   // compacted Gaussians
    __shared__ uint32_t s_off[kOccBlock];   // start of their pairs
    __shared__ uint32_t s_wave[kOccWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = blockIdx.x * kOccBlock + tid * kOccPer;
    // the four status bytes in one load (their buffer is four-byte aligned)
    uint32_t st = 0u;
    if (i0 + kOccPer <= n) {
        st = *reinterpret_cast<const uint32_t *>(status + i0);
    } else {
#pragma unroll
        for (int k = 0; k < kOccPer; ++k)
            if (i0 + k < n) st |= (uint32_t)status[i0 + k] << (8 * k);
    }
    st &= 0x02020202u;
    if (!__syncthreads_or((int)st)) return;   // most blocks: nothing newly visible
    uint32_t c[kOccPer], na = 0u, np = 0u;
#pragma unroll
    for (int k = 0; k < kOccPer; ++k) {
        c[k] = 0u;
        if (st >> (8 * k) & 2u) {
            int3 box;
            c[k] = occ_box(i0 + k, g, rect, &box);
        }
        na += c[k] ? 1u : 0u;
        np += c[k];
    }
    uint32_t total, n_act;
    uint32_t oa = occ_block_scan(na, s_wave, &n_act);
    uint32_t op = occ_block_scan(np, s_wave, &total);
#pragma unroll
    for (int k = 0; k < kOccPer; ++k) {
        if (c[k]) {
            s_idx[oa] = (uint32_t)(i0 + k);
            s_off[oa] = op;
            ++oa;
            op += c[k];
        }
    }
    __syncthreads();
    const uint32_t mine = total > (uint32_t)wave ? (total - (uint32_t)wave + kOccWaves - 1) / kOccWaves : 0u;
    for (uint32_t r0 = 0; r0 < mine; r0 += 64u) {
        const uint32_t r = r0 + (uint32_t)lane;
        int tx = 0, ty = 0;
        float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
        bool test = false;
        if (r < mine) {
            const uint32_t p = (uint32_t)wave + kOccWaves * r;
            // owner of pair p: the last entry whose start is <= p (starts
            // increase strictly: every entry has a pair)
            uint32_t lo = 0, hi = n_act;
            while (hi - lo > 1u) {
                const uint32_t mid = (lo + hi) >> 1;
                if (s_off[mid] <= p) lo = mid;
                else hi = mid;
            }
            const int gi = (int)s_idx[lo];
            int3 box;
            (void)occ_box(gi, g, rect, &box);
            const int k = (int)(p - s_off[lo]);
            tx = box.x + k % box.z;
            ty = box.y + k / box.z;
            a = g[4 * (size_t)gi];
            b = g[4 * (size_t)gi + 1];
            // Left out: tiles already marked (a mark seen late only costs
            // the test), and tiles whose centre lies farther from the mean
            // than sqrt(k) + m in the norm of the conic (m: the tile's
            // centre-to-corner offset (7.5, +-7.5); k >= 2 ln(255 o) from
            // the record): by the triangle inequality no pixel centre of
            // theirs reaches alpha >= 1/255.  Enlarged by 0.2 % + 0.01 and by
            // the rounding of the exponent (below) at the tile's pixels and of
            // q here: its terms cancel along a needle, eight roundings of
            // at most 2^-24 of their sum, itself at most 2 (T + m^2) at a
            // pixel.  A needle's box has many more tiles than its ellipse
            // meets.
            const float kq = g[4 * (size_t)gi + 3].w;
            const float m2 = 56.25f * (a.z + b.x + 2.0f * fabsf(a.w));
            const float dx = (float)(tx * kTile) + 7.5f - a.x, dy = (float)(ty * kTile) + 7.5f - a.y;
            const float sq = a.z * dx * dx + b.x * dy * dy, cross = 2.0f * a.w * dx * dy;
            const float err = 2e-6f * ((sq + fabsf(cross)) + m2);
            const float rr = (__builtin_amdgcn_sqrtf(kq + err) + __builtin_amdgcn_sqrtf(m2)) * 1.002f + 0.01f;
            test = !((sq + cross) - err > rr * rr) && !oc[ty * w.TX + tx];
        }
        for (uint64_t left = __ballot(test); left != 0ull; left &= left - 1ull) {
            const int j = __ffsll((long long)left) - 1;
            const int jx = __builtin_amdgcn_readlane(tx, j), jy = __builtin_amdgcn_readlane(ty, j);
            const float ax = lane_f(a.x, j), ay = lane_f(a.y, j), az = lane_f(a.z, j),
                        aw = lane_f(a.w, j), bx = lane_f(b.x, j), by = lane_f(b.y, j);
            float amax = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int px = lane + 64 * q;
                const int x = jx * kTile + (px & 15), y = jy * kTile + (px >> 4);
                if (x < w.W && y < w.H) {
                    const float dx = ax - (float)x, dy = ay - (float)y;
                    const float power = -0.5f * (az * dx * dx + bx * dy * dy) - aw * dx * dy;
                    if (!(power > 0.0f)) amax = fmaxf(amax, fminf(kAlphaMax, by * __expf(power)));
                }
            }
            const uint64_t hit = __ballot(!(amax < kAlphaMin));
            if (hit != 0ull && lane == 0) oc[jy * w.TX + jx] = 1;
        }
    }
}

// One block per tile row ty: selected = occluded | unmatched (or every
// tile), row ty + 1 of the mask's summed area table (block 0 also row 0), the
// columns of the row's selected tiles in order, and its entries of the
// ascending list of selected tiles (the tiles not selected fill the list from
// the end, descending).  What lies above the row the block counts itself from
// the flags, per column (threads share out the rows above, a few KB read from
// cache), so no second launch waits for the other rows.  The last row also
// stores the total.
constexpr int kSelThreads = 512;
constexpr int kSelWaves = kSelThreads / 64;

// Exclusive scans across the block of two values per thread; totals in ta, tb.
__device__ inline void select_scan2(uint32_t &a, uint32_t &b, uint2 *s_wave, uint32_t &ta, uint32_t &tb) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t ia = a, ib = b;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t xa = __shfl_up(ia, d), xb = __shfl_up(ib, d);
        if (lane >= d) {
            ia += xa;
            ib += xb;
        }
    }
    if (lane == 63) s_wave[wave] = make_uint2(ia, ib);
    __syncthreads();
    uint32_t oa = 0, ob = 0;
    ta = tb = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        const uint2 x = s_wave[w];
        if (w < wave) {
            oa += x.x;
            ob += x.y;
        }
        ta += x.x;
        tb += x.y;
    }
    __syncthreads();
    a = oa + ia - a;
    b = ob + ib - b;
}

__global__ __launch_bounds__(kSelThreads) void select_kernel(int TX, int TY, int mode, const uint8_t *oc,
                                                             const uint8_t *um, uint8_t *sel,
                                                             uint32_t *sat, int *sel_list, int *sel_cols,
                                                             uint8_t *mask_out, Counters *cnt) {
    __shared__ uint32_t s_col[kSelThreads];
    __shared__ uint2 s_wave[kSelWaves];
    const int ty = blockIdx.x, tid = threadIdx.x;
    // a chunk of 2^cb columns (the grid's width or 512) by 512 >> cb groups of rows
    int cb = 4;
    while (cb < 9 && (1 << cb) < TX) ++cb;
    const int cw = 1 << cb, groups = kSelThreads >> cb;
    const int xi = tid & (cw - 1), grp = tid >> cb;
    // selected tiles of the chunk's columns above the row; valid for tid < cw
    auto above_of = [&](int c0) -> uint32_t {
        const int x = c0 + xi;
        uint32_t part = 0;
        if (x < TX) {
            if (mode) {
                part = grp == 0 ? (uint32_t)ty : 0u;
            } else {
                // clamped rows, no branches: each round's loads are in flight
                // together
                for (int y0 = grp; y0 < ty; y0 += 8 * groups) {
                    uint32_t f[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int y = y0 + k * groups;
                        const size_t t = (size_t)(y < ty ? y : y0) * TX + x;
                        f[k] = (uint32_t)(oc[t] | um[t]);
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k) part += y0 + k * groups < ty ? f[k] : 0u;
                }
            }
        }
        __syncthreads();
        s_col[tid] = part;
        __syncthreads();
        uint32_t a = 0;
        if (tid < cw)
            for (int g = 0; g < groups; ++g) a += s_col[g * cw + tid];
        return a;
    };
    uint32_t off = 0;   // selected tiles above the row
    if (TX > cw) {      // block-uniform; else known from the one chunk's scan
        for (int c0 = 0; c0 < TX; c0 += cw) {
            uint32_t a = above_of(c0), z = 0, ta, tz;
            select_scan2(a, z, s_wave, ta, tz);
            off += ta;
        }
    }
    const uint32_t above = (uint32_t)ty * (uint32_t)TX;
    uint32_t *row = sat + (size_t)(ty + 1) * (TX + 1);
    uint32_t run = 0, run_sat = 0;   // of the chunks before
    for (int c0 = 0; c0 < TX; c0 += cw) {
        const int x = c0 + tid;
        const bool mine = tid < cw && x < TX;
        const int t = ty * TX + x;
        uint32_t a = above_of(c0), f = 0;
        if (mine) {
            f = mode ? 1u : (uint32_t)(oc[t] | um[t]);
            sel[t] = (uint8_t)f;
            if (mask_out) mask_out[t] = (uint8_t)f;
        }
        uint32_t ex = f, exs = a + f, tot, tots;
        select_scan2(ex, exs, s_wave, tot, tots);
        if (TX <= cw) off = tots - tot;
        if (mine) {
            row[x] = run_sat + exs;
            if (ty == 0) sat[x] = 0u;
            if (f) {
                sel_list[off + run + ex] = t;
                sel_cols[(size_t)ty * TX + run + ex] = x;
            } else {
                // the others from the end: tiles not selected above the row,
                // then those of the row before this one
                sel_list[TX * TY - 1 - ((above - off) + ((uint32_t)x - run - ex))] = t;
            }
        }
        run += tot;
        run_sat += tots;
    }
    if (tid == 0) {
        row[TX] = run_sat;
        if (ty == 0) sat[TX] = 0u;
        if (ty == TY - 1) cnt->n_selected = off + run;
    }
}

template <typename T>
__global__ __launch_bounds__(256) void fill_kernel(T *p, size_t n, T v) {
    for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n;
         k += (size_t)gridDim.x * blockDim.x)
        p[k] = v;
}

template <typename T>
void fill(T *p, size_t n, T v, hipStream_t st) {
    if (n == 0) return;
    size_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    fill_kernel<T><<<(unsigned)blocks, 256, 0, st>>>(p, n, v);
}

}  // namespace

void launch_temporal_init(int n_px, float *dmin, float *smax, hipStream_t st) {
    if (n_px > 0) temporal_init_kernel<<<(n_px + 255) / 256, 256, 0, st>>>(n_px, dmin, smax);
}

void launch_forward_warp(const WarpK &w, const float *D, const float *S, float *dmin, float *smax,
                         hipStream_t st) {
    const int n = w.W * w.H;
    forward_warp_kernel<<<(n + 255) / 256, 256, 0, st>>>(w, D, S, dmin, smax);
}

void launch_fill_query(const FillK &f, hipStream_t st) {
    fill_query_kernel<<<f.w.TX * f.w.TY, f.w.tp * f.w.tp, 0, st>>>(f);
}

void launch_occluded(const WarpK &w, int n, const uint8_t *status, const float4 *g,
                     const ushort4 *rect, uint8_t *oc, hipStream_t st) {
    if (n <= 0) return;
    occluded_kernel<<<(n + kOccBlock - 1) / kOccBlock, kOccThreads, 0, st>>>(w, n, status, g, rect,
                                                                            oc);
}

void launch_select(int TX, int TY, int mode, const uint8_t *oc, const uint8_t *um, uint8_t *sel,
                   int *sel_list, uint32_t *sat, int *sel_cols, uint8_t *mask_out,
                   Counters *cnt, hipStream_t st) {
    select_kernel<<<TY, kSelThreads, 0, st>>>(TX, TY, mode, oc, um, sel, sat, sel_list, sel_cols,
                                      mask_out, cnt);
}

void launch_fill_u8(uint8_t *p, size_t n, uint8_t v, hipStream_t st) { fill<uint8_t>(p, n, v, st); }
void launch_fill_f32(float *p, size_t n, float v, hipStream_t st) { fill<float>(p, n, v, st); }
void launch_fill_i32(int *p, size_t n, int v, hipStream_t st) { fill<int>(p, n, v, st); }

}  // namespace tgs

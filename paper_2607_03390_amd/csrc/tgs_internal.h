// Internal declarations shared by the HIP translation units of libtgs.
// Kernel argument structs and the host-side launchers each .hip file exports.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include "depth_plan.h"
#include "tgs.h"

namespace tgs {

constexpr float kNoHit = 1001.0f;           // z_far (1000) + epsilon (1)
constexpr float kZFar = 1000.0f;            // far plane
constexpr float kAlphaMin = 1.0f / 255.0f;
constexpr float kAlphaMax = 0.99f;
constexpr float kTMin = 1e-4f;
constexpr int kTile = 16;
// Key positions are 32-bit; the limit leaves headroom so that block bases
// (partition * tile, block * 1024) and loop strides never wrap.
constexpr uint32_t kMaxKeys = 0xffff0000u;

// Camera constants as the kernels consume them.
struct CamK {
    float V[12];              // rows 0..2 of world->camera
    float fx, fy, cx, cy;
    int W, H, TX, TY;
    float limx, limy;         // 1.3 * tan(half fov) guards of the Jacobian
    float campos[3];          // camera centre in world space
};

// Device scene.  Means and opacities are one float4 per Gaussian in their own
// array (every Gaussian's is read each frame, one coalesced 1 KB request per
// wave).  The rest is read only for Gaussians that survive the culls, often
// a scattered minority of a wave, so each Gaussian's bytes are contiguous:
// two geometry float4s (32 bytes) and sh_slots SH float4s (192 bytes, three
// whole 64-byte lines, at degree 3), and a culled Gaussian's lines are
// never fetched.
struct SceneDev {
    int n, deg, ncoef, sh_slots;
    const float4 *mean_op;    // x, y, z, opacity
    const float4 *geo;        // [2i] = (sx, sy, sz, qw), [2i + 1] = (qx, qy, qz, 0)
    const float4 *sh;         // [i * sh_slots + j]: coefficient-major (k*3 + channel) floats
};

// Per-Gaussian records written by the preprocess.
struct Records {
    // One 64-byte record per Gaussian (one aligned line per gather):
    // g[4i] = (u, v, conic a, conic b), g[4i + 1] = (conic c, opacity,
    // depth, hy), g[4i + 2] = (r, g, b, hx), g[4i + 3] = (qa, qb, qc, k):
    // the blend's constants, computed once per Gaussian instead of once per
    // (Gaussian, tile): q* = conic pre-scaled by -log2(e) (1/2 on the
    // squares), and hx, hy = half extents of the box of the alpha >= 1/255
    // ellipse enlarged by 0.2% + 0.05 px (negative: alpha < 1/255 everywhere);
    // g[4i + 3].w = k >= 2 ln(255 o), the ellipse's bound on the conic form.
    float4 *g;
    ushort4 *rect;            // tile rectangle x0, y0, x1, y1 (x0 > x1: empty)
    uint8_t *status;          // bit0 survivor, bit1 newly visible
    uint32_t *count;          // keys of the Gaussian (tiles of its rectangle)
    uint32_t *dkey;           // float bits of the depth (depth-sort key); kNoDepth: no keys
    uint32_t *partial;        // per 256-Gaussian block: survivors, newly visible
    // optional: the depth keys of one Gaussian per stratum of sample_stride,
    // for the depth order's splitters (sample_magic = ceil(2^40 / stride):
    // i * magic >> 40 is i / stride for i < 2^23)
    uint32_t *samples;
    uint32_t sample_stride;
    uint64_t sample_magic;
};
constexpr uint32_t kNoDepth = 0xffffffffu;
// The sampled Gaussian of stratum q (`stride` consecutive ones): at a place
// hashed from its number, so that no order of the scene is met in step.
__host__ __device__ inline uint32_t depth_sample_at(uint32_t q, uint32_t stride, int n) {
    const uint32_t at = q * stride + (uint32_t)((uint64_t)(q * 0x9e3779b1u) * stride >> 32);
    return at < (uint32_t)(n - 1) ? at : (uint32_t)(n - 1);
}

// Temporal dynamic culling inputs of the preprocess.
struct CullK {
    float z_near;
    int afc, toc;
    const int *fbox;          // ordered-int encoded F_min.x, F_min.y, F_max.x, F_max.y
    const float *dmin, *smax; // warped TGB
    const uint8_t *g_rendered;
    float lambda1, lambda2;
    int footprint;            // tile rectangle: 0 = 3-sigma square, 1 = alpha footprint box
    int tgb_shift;            // dmin/smax grid = image >> tgb_shift (0, or 1: 2x2 blocks)
    int tgb_w;                // width of that grid
    uint8_t *clear_flag;      // optional (reference frames): set to 0 for every Gaussian
                              // (the temporal Gaussian buffer the blend then fills)
};

// Frame counters on the device (read back once per frame).
struct Counters {
    uint32_t n_keys;
    uint32_t n_survivors;
    uint32_t n_newly;
    uint32_t n_selected;
    uint32_t n_visible;       // Gaussians with at least one key
    uint32_t n_sorted;        // keys emitted and sorted: n_keys, or 0 past the key capacity
    uint32_t n_split;         // tiles the blend splits into quadrants (the blend order's first)
    uint32_t pad;
};

// The frame's counters as the host reads them: written by the last counting
// kernel straight into coherent pinned host memory (16-byte aligned), tag
// last (after a system-scope fence), so the host waits for the tag instead of
// a copy.
struct HostCounters {
    uint32_t n_keys, n_survivors, n_newly, n_selected, n_visible, n_sorted;
    uint32_t redo;   // 1: the frame has no keys and is to be rendered again (a bucket of the
                     // sample sort overflowed) with the radix passes
    uint32_t tag;
};

// Writes the frame's counters to the host: the seven values as vector
// stores, a system-scope fence (they are complete and visible), then the tag
// as a relaxed store that nothing waits for.  (A volatile store would wait
// for its own round trip to host memory, one after another.)
__device__ inline void publish_host(HostCounters *h, uint32_t n_keys, uint32_t n_survivors,
                                    uint32_t n_newly, uint32_t n_selected, uint32_t n_visible,
                                    uint32_t n_sorted, uint32_t redo, uint32_t tag) {
    reinterpret_cast<uint4 *>(h)[0] = make_uint4(n_keys, n_survivors, n_newly, n_selected);
    reinterpret_cast<uint2 *>(h)[2] = make_uint2(n_visible, n_sorted);
    h->redo = redo;
    __threadfence_system();
    __hip_atomic_store(&h->tag, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Ordered-int encoding of a float: signed-int order equals float order, so
// integer atomic min/max give exact float min/max.
__device__ inline int float_to_ordered(float f) {
    int i = __float_as_int(f);
    return i >= 0 ? i : i ^ 0x7fffffff;
}
__device__ inline float ordered_to_float(int i) {
    return __int_as_float(i >= 0 ? i : i ^ 0x7fffffff);
}

// Key count of a Gaussian in a selective-rendering frame: the selected tiles
// of its rectangle, from the tile mask's summed area table: sat[y * (TX + 1)
// + x] = selected tiles in rows below y and columns below x (TY + 1 rows), so
// four loads whatever the rectangle's height.  (From prefix sums per row, two
// loads a row, counting 1.5M Gaussians took 11.9 us and 3M needles 66 us.)
__device__ inline uint32_t masked_count(ushort4 r, const uint32_t *sat, int TX) {
    if (r.x > r.z || r.y > r.w) return 0u;
    const uint32_t *top = sat + (size_t)r.y * (TX + 1), *bot = sat + (size_t)(r.w + 1) * (TX + 1);
    const uint32_t t0 = top[r.x], t1 = top[r.z + 1], b0 = bot[r.x], b1 = bot[r.z + 1];
    return (b1 - b0) - (t1 - t0);
}

// ---- launchers (k_preprocess.hip) ----
// Writes the records and, per 256-Gaussian block, the survivor and
// newly-visible counts (summed into cnt by the last depth-sort pass).
// fill (optional): the depth fill / correspondence query of a TemporalGS
// frame (full-resolution geometry buffer) run by blocks of the same launch
// past the Gaussians' (independent work: both read only the forward warp).
// start / stop (may be NULL): events attached to the preprocess dispatch.
struct FillK;
void launch_preprocess(const SceneDev &s, const CamK &cam, const CullK &cull, Records rec,
                       Counters *cnt, const FillK *fill, hipStream_t st, hipEvent_t start = nullptr,
                       hipEvent_t stop = nullptr);
inline int preprocess_blocks(int n) { return (n + 255) / 256; }

// Keys are emitted in blocks of kKeyBlock consecutive positions; kfirst[B]
// (written by whichever kernel produces the key offsets) is the sorted
// position of the Gaussian that owns key B * kKeyBlock, for every block below
// the key capacity.
constexpr int kKeyBlock = 1024;
__host__ __device__ inline size_t key_blocks(size_t cap) { return (cap + kKeyBlock - 1) / kKeyBlock; }
// Records, for a sorted Gaussian at position s with keys [o, o + c), s as
// the owner of every key block that starts inside that range (below nb).
__device__ inline void mark_key_blocks(uint32_t *kfirst, uint32_t nb, uint32_t s, uint64_t o,
                                       uint32_t c) {
    for (uint64_t b = (o + kKeyBlock - 1) / kKeyBlock; b < nb && b * kKeyBlock < o + c; ++b)
        kfirst[b] = s;
}

// ---- launchers (k_keys.hip) ----
// Emits the cnt->n_sorted keys of the cnt->n_visible depth-ordered Gaussians
// (cap bounds n_sorted for the grid; nothing is emitted past the key
// capacity) and clears the tile ranges and lengths (filled by the tile sort, or
// the ranges by launch_ranges after it).  sat / sel_cols are NULL in frames that render every tile.
// rect: by Gaussian index, or (rect_sorted) in the order of didx.
// Keys: tile id to tkey and index to tval, or (tp.packed) the low digit bytes
// to tkey and the payload to tval (launch_tile_sort).  rows (optional): per
// block of kKeyBlock keys, the counts of the low digit in row b of
// rows[b][256].
struct TileSortPlan;
void launch_duplicate(int n, uint32_t cap, const Counters *cnt, const uint32_t *didx,
                      const uint32_t *offs, const uint32_t *kfirst, const ushort4 *rect,
                      bool rect_sorted, const uint32_t *sat, const int *sel_cols, int TX, int n_tiles,
                      const TileSortPlan &tp, uint32_t *tkey, uint32_t *tval, uint2 *ranges,
                      uint32_t *tile_len, uint32_t *rows, hipStream_t st);
// Ranges of the cnt->n_sorted tile-sorted keys; cap bounds n_sorted for the grid.
void launch_ranges(uint32_t cap, const Counters *cnt, const uint32_t *keys, uint2 *ranges,
                   hipStream_t st);
// Tiles to rasterise (tile_in[0..m), or 0..m-1 when tile_in is NULL; m =
// *n_dev when n_dev is given, else n) in blend order, longest lists first,
// into tile_out[0..m).
// max_bucket (optional, host-visible memory) receives floor(log2 of the
// longest list length) + 1, and nothing where all lists are empty.
struct OrderK {
    int n_host;
    const uint32_t *n_dev;
    const int *tile_in;
    const uint2 *ranges;
    int *tile_out;
    uint32_t *max_bucket;
    // optional: the number of tiles the blend splits, the first of the
    // order: those whose list length bucket is at least split_bucket, or, if
    // more than max_split (<= kMaxSplit) are, at least the lowest higher
    // bucket that leaves at most max_split (0: no split)
    // cnt (optional): the frame's counters; split_bucket is then an upper bound
    // and the frame's own is taken from its keys and lists (split_bucket_for)
    uint32_t *n_split;
    int split_bucket;
    int max_split;
    const Counters *cnt;
};
// (kOrderShares blocks, each placing its share of the tiles.)
constexpr int kOrderShares = 8;
void launch_order_tiles(const OrderK &o, hipStream_t st);

// ---- launchers (k_sort.hip) ----
int sort_passes_for_bits(int bits);
// Scratch words of a sort of at most max_keys keys (either kind below).
size_t sort_scratch_words(uint32_t max_keys);
// Stable LSD sort of (key, value) pairs on key bits [begin_bit, begin_bit +
// bits), in ceil(bits / 8) passes of (nearly) equal width; every key must be
// below 2^(begin_bit + bits).  The key count is *n_dev if n_dev is not NULL
// (n_max bounds it), else n_max.  Returns 1 if the result is in the alt buffers.
// n_hint: the expected key count (e.g. a recent frame's); it picks the
// partition size (small partitions fill the chip for small sorts).
int launch_sort_u32(const uint32_t *n_dev, uint32_t n_max, uint32_t n_hint, int begin_bit,
                    int bits, uint32_t *keys, uint32_t *vals, uint32_t *keys_alt,
                    uint32_t *vals_alt, uint32_t *scratch, hipStream_t st);
// The sorts' scratch: chunk sums, then count rows of 256 digits.
uint32_t *sort_count_rows(uint32_t *scratch);
// Column scan of the count rows of ceil(n / tile) partitions (n = *n_dev or
// n_host): offsets within the chunk in place, the chunks' digit sums to sums.
void launch_colscan(const uint32_t *n_dev, uint32_t n_host, uint32_t tile, uint32_t np, int tables,
                    uint32_t *table, uint32_t *sums, hipStream_t st);
// ---- launchers (k_tilesort.hip) ----
// How the keys of a scene of n Gaussians on a grid of tile ids of `bits` bits
// are laid out and sorted: packed (grids of up to 2^16 tiles whose high
// digit fits beside the index), or as (tile id, index) word pairs by
// launch_sort_u32.
struct TileSortPlan {
    int bits;         // of a tile id
    int index_bits;   // of a Gaussian index
    int lo, hi;       // packed: widths of the two digits (hi = 0: one pass)
    bool packed;
};
TileSortPlan tile_sort_plan(int n, int bits);
// Whether the sort takes partitions of kKeyBlock keys (n_hint: the expected
// key count, e.g. a recent frame's): the emission may then count the low
// digits of its blocks of keys into sort_count_rows(scratch).
bool tile_sort_small(uint32_t cap, uint32_t n_hint);
// Stable sort of the *n_dev (<= cap) payloads (high digit << index_bits |
// index) by (high digit, low digit dig), to Gaussian indices; the tile
// ranges (of the tiles with keys; the others stay as the emission cleared
// them) and, unless order_apart(n_hint), the blend order of the tiles (order).
// counted: the emission has counted.  scratch and segments:
// tile_sort_scratch_words(cap) and tile_sort_segment_words(cap) words;
// tile_len: n_tiles words, cleared by the emission.  Returns 1 if the result is in pay_alt, 0 if in pay.
// Sorts of more keys than this leave the order to a launch of its own: a
// tile's length is summed by one add per partition of its low digit, hundreds
// of them to one address (2.27G keys: 1.7 -> 3.9 ms for the counting launch,
// 5.0M keys: 6.4 -> 8.8 us, against a launch of 10 us).
inline bool order_apart(uint32_t n_hint) { return n_hint > (32u << 20); }
size_t tile_sort_scratch_words(uint32_t max_keys);
size_t tile_sort_segment_words(uint32_t max_keys);
int launch_tile_sort(const TileSortPlan &tp, uint32_t cap, uint32_t n_hint, const uint32_t *n_dev,
                     const uint8_t *dig, uint32_t *pay, uint32_t *pay_alt, uint32_t *scratch,
                     uint32_t *segments, bool counted, uint2 *ranges, uint32_t *tile_len, int n_tiles,
                     const OrderK &order, hipStream_t st);

// Depth order of the Gaussians with count[i] > 0 among i < n, stable by index
// (keys dkey[i], the depth's float bits): four passes (dkey -> a -> b -> a ->
// v_b; k_b may alias dkey).  With sat (a selective-rendering frame) the
// first pass first replaces count[i] by the masked count of rect[i].  Writes cnt->n_visible (Gaussians kept), the
// sorted indices to v_b[0..n_visible), offs[s] = exclusive prefix of their
// counts and the key-block owners kfirst[0 .. key_blocks(cap)), then
// cnt->n_keys, cnt->n_sorted (n_keys if <= cap, else 0),
// cnt->n_survivors / n_newly (from the preprocess partials) and, tag last,
// the same counters to `host`.
void launch_depth_sort(int n, uint32_t *count, const ushort4 *rect, const uint32_t *sat, int TX,
                       const uint32_t *dkey, uint32_t *k_a, uint32_t *v_a, uint32_t *k_b,
                       uint32_t *v_b, uint32_t *offs, uint32_t *kfirst, uint32_t *scratch,
                       Counters *cnt, uint32_t cap, const uint32_t *pre_partial, int n_pre,
                       HostCounters *host, uint32_t tag, hipStream_t st);

// ---- launchers (k_depthsort.hip) ----
// Depth order of the Gaussians that have keys by a sample sort (sizes:
// depth_plan.h): the parts of its scratch (entries: 16-byte aligned, used only
// until the sorted order is written) and the sort, with the outputs of
// launch_depth_sort and the sorted Gaussians' rectangles
// (DepthScratch::srect).  Without keys to publish, because a bucket
// overflowed: HostCounters::redo.
struct DepthScratch {
    uint4 *entries;
    uint64_t *splitters, *fill;
    ushort4 *srect;
    uint32_t *samples;
};
DepthScratch depth_scratch(const DepthPlan &dp, int n, void *entries, void *rest);
void launch_depth_samplesort(const DepthPlan &dp, const DepthScratch &d, int n, const uint32_t *dkey,
                             const ushort4 *rect, const uint32_t *sat, int TX, uint32_t *didx,
                             uint32_t *offs, uint32_t *kfirst, Counters *cnt, uint32_t cap,
                             const uint32_t *pre_partial, int n_pre, HostCounters *host, uint32_t tag,
                             hipStream_t st);

// ---- launchers (k_segsort.hip) ----
// Per-tile depth order without the global depth sort: key counts scanned in
// index order (part: 2 words per 1024-Gaussian block), the
// Gaussians with keys compacted in index order into vidx / voffs (the
// duplication's input), the frame's counters published as the depth sort
// does; after the tile sort, each tile's list sorted by (depth bits, index)
// in place (tmp: scratch of the same size as vals).
int count_scan_blocks(int n);
void launch_count_scan(int n, uint32_t *count, const ushort4 *rect, const uint32_t *sat, int TX,
                       uint32_t *part, uint32_t *vidx, uint32_t *voffs, uint32_t *kfirst,
                       Counters *cnt, uint32_t cap, const uint32_t *pre_partial, int n_pre,
                       HostCounters *host, uint32_t tag, hipStream_t st);
// long_lists: lists above 2048 entries are expected (a launch of their own
// for them); otherwise the few there are take a slower in-block path.
void launch_segment_sort(int n_tiles, const uint2 *ranges, uint32_t *vals, uint32_t *tmp,
                         const uint32_t *dkey, bool long_lists, hipStream_t st);
// Length bucket (floor(log2 len) + 1) from which a recent frame's lists make
// the long-list launch worth its cost: lists of 2048 entries and more.
constexpr int kSegLongBucket = 12;
// Longest list the per-tile sort handles in LDS; longer ones take its slower
// in-block path.  Lists of bucket <= kSegBucketMax (floor(log2 len) + 1)
// fit.
constexpr int kSegBucketMax = 12;

// ---- launchers (k_blend.hip) ----
// View pair of a TemporalGS frame (reference -> current) for the temporal
// kernels and stitching.
struct WarpK {
    float M[12];              // reference camera -> current camera
    float Minv[12];           // current camera -> reference camera
    float kref[4], kcur[4];   // fx, fy, cx, cy
    float z_near;
    int W, H, TX, TY;         // grid size (image, or the geometry buffer's) and tiles
    int tp;                   // pixels per tile side on this grid (16, or 8 at half resolution)
};

// Operands of the depth fill / backward query: one block of tp x tp threads
// per tile; also clears oc[tile] and resets this tile's cells of the other
// warp pair (dmin_next = empty depth, smax_next = 0) for the next frame.
struct FillK {
    WarpK w;
    const float *dmin;
    float *dfill;
    float2 *uv;
    uint8_t *um, *oc;
    float *dmin_next, *smax_next;
};

struct BlendArgs {
    int W, H, TX, TY;
    const int *tile_list;     // NULL: blockIdx = tile
    const uint32_t *n_tiles_dev;  // optional: blocks at or past *n_tiles_dev do nothing
    // optional (with tile_list): the first *n_split_dev (<= split_cap) tiles
    // of tile_list are blended as four quadrant blocks each; the launch adds
    // 3 split_cap + 28 blocks (4 ceil8(n_split) quadrant blocks replace
    // n_split tile blocks; n_grid: the launch's tile blocks, set by
    // launch_blend)
    const uint32_t *n_split_dev;
    int split_cap;            // with n_split_dev: *n_split_dev <= split_cap <= kMaxSplit
    int n_grid;
    const uint2 *ranges;
    const uint32_t *vals;
    const float4 *g;          // 64-byte records (Records::g)
    float *rgb;               // [3][H][W]
    float *tab;               // optional second copy of rgb
    float *depth, *sigma, *alpha;       // optional outputs
    float *tgb_depth, *tgb_sigma;       // optional second copies
    float *tgbh_depth, *tgbh_sigma;     // optional: Eq. 1/2 pooled over 2x2 blocks
                                        // (grid ceil(W/2) x ceil(H/2))
    uint8_t *g_flag;          // optional: Gaussian composited somewhere
    float *contrib;           // optional: max weight per Gaussian
    unsigned long long *pairs;  // optional: count of evaluated pixel-Gaussian pairs
    unsigned long long *hits;   // with pairs: count of pairs with alpha >= 1/255 (composited or stopping)
    float empty_depth;        // depth written where no Gaussian is composited
    float bg[3];              // background: rgb = sum of w c + T bg
    uint8_t *mark_sel, *mark_mask;   // optional: set to 1 for every blended tile
    // optional (TGS frames): blocks at or past *n_tiles_dev stitch tile
    // stitch_list[block] from the reference image stitch_tab (Eq. 4)
    // instead of blending, so that stitching overlaps the blend's tail:
    // stitch_mode 1 samples at the per-pixel correspondences stitch_uv,
    // 2 unprojects with the half-resolution repaired depth stitch_dfill
    // (grid width stitch_wg); sw is the full-resolution view pair
    const int *stitch_list;
    int stitch_mode, stitch_wg;
    const float *stitch_tab;
    const float2 *stitch_uv;
    const float *stitch_dfill;
    WarpK sw;
};
// Longest lists split into quadrant blocks by the blend: at most kMaxSplit
// tiles (a scene's cap; the launch adds 3 cap + 28 blocks, for 4 ceil8(n_split)
// quadrant blocks, those without a quadrant exit at once; none when the
// scene does not split), by default those of kSplitBucket (lists of
// 2^(kSplitBucket-1) entries) and up.
constexpr int kMaxSplit = TGS_BLEND_SPLIT_MAX;
constexpr int kSplitBucket = TGS_BLEND_SPLIT_DEFAULT + 1;
// start/stop (may be NULL) are attached to the dispatch itself
// (hipExtLaunchKernelGGL): kernel timing without extra barrier packets.
void launch_blend(const BlendArgs &a, int n_blocks, hipStream_t st, hipEvent_t start = nullptr,
                  hipEvent_t stop = nullptr);
// fbox must hold 4 + 4 * kAfcPartials ints (result, then partials).
constexpr int kAfcPartials = 256;
void launch_afc_bounds(int n, const uint8_t *g_flag, const float4 *g, int W, int H, int *fbox,
                       hipStream_t st);

// ---- launchers (k_temporal.hip) ----
// dmin = empty depth, smax = 0 over n_px cells
void launch_temporal_init(int n_px, float *dmin, float *smax, hipStream_t st);
void launch_forward_warp(const WarpK &w, const float *D, const float *S, float *dmin, float *smax,
                         hipStream_t st);
// Also oc[tile] = 0 and dmin_next / smax_next reset to their initial values
// (the other warp pair, for the next frame).
void launch_fill_query(const FillK &f, hipStream_t st);
void launch_occluded(const WarpK &w, int n, const uint8_t *status, const float4 *g,
                     const ushort4 *rect, uint8_t *oc, hipStream_t st);
// sel_list: the selected tiles ascending in [0, n_selected), the others
// descending from the end (a permutation of all tiles); sat: the mask's
// summed area table ((TY + 1) x (TX + 1), see masked_count);
// sel_cols[ty * TX + k] = column of the k-th selected tile of row ty
void launch_select(int TX, int TY, int mode, const uint8_t *oc, const uint8_t *um, uint8_t *sel,
                   int *sel_list, uint32_t *sat, int *sel_cols, uint8_t *mask_out,
                   Counters *cnt, hipStream_t st);
void launch_fill_u8(uint8_t *p, size_t n, uint8_t v, hipStream_t st);
void launch_fill_f32(float *p, size_t n, float v, hipStream_t st);
void launch_fill_i32(int *p, size_t n, int v, hipStream_t st);

}  // namespace tgs

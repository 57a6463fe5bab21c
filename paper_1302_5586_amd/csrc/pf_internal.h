// Internal declarations shared by the library's translation units.
// Nothing here is part of the C ABI (that is include/pf.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <string>
#include <vector>

#include "pf.h"
#include "pf_check.h"

namespace pf {

// A wave strip is 64 lanes x 4 columns. halo_lanes: neighbouring lanes on
// each side whose columns a lane's window needs. For radii 1 and 2 every
// lane produces outputs (256 columns, 1 KiB of FP32) and lanes 0 and 63
// also load the r columns beyond the strip (r registers per row); for
// larger radii, where those registers would cost occupancy, the outermost
// lanes only load halo columns and do not store.
#ifndef PF_STRIP_ALIGNED
#define PF_STRIP_ALIGNED 1
#endif
#ifndef PF_STRIP_ALIGNED_RMAX
#define PF_STRIP_ALIGNED_RMAX 2
#endif
constexpr int halo_lanes(int r) { return (r + 3) / 4; }
constexpr bool aligned_strip(int r) { return PF_STRIP_ALIGNED && r >= 1 && r <= PF_STRIP_ALIGNED_RMAX; }
constexpr int idle_lanes(int r) { return aligned_strip(r) ? 0 : halo_lanes(r); }
constexpr int strip_width(int r) { return 4 * (64 - 2 * idle_lanes(r)); }
// The uint8 strip keeps its halo lanes at every radius.
constexpr int strip_width_u8(int r) { return 4 * (64 - 2 * halo_lanes(r)); }

// ---- strip geometry of the FP32 strip kernel.

// How a strip loads its rows (uniform over the wave):
//   kStripFast: every lane's 4 columns lie inside the image (a halo lane
//               left of column 0 aside): one 16-byte load per lane;
//   kStripEdge: some columns lie outside; the lane loads the 4 in-bounds
//               columns nearest to its own (w >= 4) and picks each clamped
//               column from them;
//   kStripTiny: one clamped load per column (images narrower than 4
//               columns, and every strip of radii above 4).
constexpr int kStripFast = 0, kStripEdge = 1, kStripTiny = 2;

// Rows per pipelined chunk of the FP32 strip: a multiple of K = 2r+1 (ring
// residues stay compile-time constants) near `chunk` rows (8 measured best).
// Rows past the last whole chunk of a tile are taken in groups of
// 2r+1 with a wait per group, so tile heights that fill whole chunks skip
// that tail (the tuner tries them).
#ifndef PF_CHUNK
#define PF_CHUNK 8
#endif
constexpr int chunk_rows_of(int r, int chunk) {
    return (2 * r + 1) * (chunk / (2 * r + 1) > 0 ? chunk / (2 * r + 1) : 1);
}

constexpr int clamp_int(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// First column of lane `lane` in a strip starting at column x0.
constexpr int lane_col(int r, int x0, int lane) { return x0 + 4 * (lane - idle_lanes(r)); }

// kStripFast needs every lane's columns to end inside the image; for an
// aligned strip also the r columns to its right inside it, or none.
constexpr bool fast_strip(int r, int x0, int w) {
    const int end = x0 + 4 * (64 - idle_lanes(r));
    return aligned_strip(r) ? (end <= w && (end == w || end + r <= w)) : end <= w;
}

constexpr int strip_mode(int r, int x0, int w) {
    return r > 4 ? kStripTiny : (fast_strip(r, x0, w) ? kStripFast : (w >= 4 ? kStripEdge : kStripTiny));
}

// First of the 4 columns the 16-byte load of a lane with first column xs
// reads in kStripFast and kStripEdge (a halo lane left of column 0 reads
// columns 0..3).
constexpr int vec_load_col(int r, int mode, int xs, int w) {
    return mode == kStripFast ? (idle_lanes(r) > 0 ? (xs > 0 ? xs : 0) : xs) : clamp_int(xs, 0, w - 4);
}

// First of the r columns the halo load of an aligned strip reads in
// kStripFast: left of the strip (lanes 0..31) or right of it (lanes 32..63),
// moved inside the image at its edges.
constexpr int halo_load_col(int r, bool left, int x0, int w) {
    return left ? (x0 - r > 0 ? x0 - r : 0) : (x0 + 4 * 64 < w - r ? x0 + 4 * 64 : w - r);
}

// Order of the FP32 kernels' wave tiles inside an image: row-major over the
// image's strips (0) or column-major (1).
#ifndef PF_TILE_COLMAJOR
#define PF_TILE_COLMAJOR 0
#endif
constexpr bool kTileColMajorF32 = PF_TILE_COLMAJOR != 0;

// Tile number -> (strip x, strip y): row-major over the image's strips, or
// column-major (strip by strip down the image).
constexpr void tile_strip(bool colmajor, int t, int strips_x, int strips_y, int &sx, int &sy) {
    if (colmajor) {
        sx = t / strips_y;
        sy = t - sx * strips_y;
    } else {
        sy = t / strips_x;
        sx = t - sy * strips_x;
    }
}

// ---- tile geometry, shared by the FP32 tile kernels and the host-side check
// of batch plans.

// Columns staged left and right of a tile: the radius in whole 16-byte vectors.
constexpr int tile_pad(int r) { return 4 * ((r + 3) / 4); }

// Whether the tw x th tile at (x0, y0) and its staged halo lie inside the
// image, so that it is loaded without clamping (with 32-bit row offsets).
constexpr bool tile_inside(int r, int tw, int th, int x0, int y0, int h, int w) {
    return x0 >= tile_pad(r) && w - x0 >= tw + tile_pad(r) && y0 >= r && h - y0 >= th + r && w <= 1 << 24;
}

// Column, relative to x0, of the 16-byte load that serves columns c .. c+3 of
// a tile at the image's edge: the nearest inside the row (w >= 4).
constexpr int tile_load_col(int c, int x0, int w) { return clamp_int(c, -x0, w - 4 - x0); }

// Tiles of a batch launch, columns x rows.
//  * 64 x 16 while all of the batch's fit on the chip at once (8 workgroups of
//    4 waves on each of 256 CUs), since the time is then one tile's.
//  * 64 x 32 where there are at most 1.8 of them to one of 256 x 20: in images of
//    up to some 200 columns a wide tile is mostly padding, and a tile of 64 x 32
//    takes about half its time even so. us, separable, radius 1, 256 x 20 / 64 x
//    32: 4096 images of 64 x 64 (0.5 to one) 59 / 25, 2000 of 100 x 100 (1.6)
//    40.5 / 36.2, 3000 of 70 x 300 (1.9) 86.5 / 90; sizes log-uniform 16..96 (0.8)
//    41 / 22, 32..512 (1.7) 81 / 67, 64..1024 (2.1) 124 / 148; 2D, radius 4: 64 x
//    64 240 / 56, 32..512 158 / 115, 64..1024 188 / 190.
//  * 256 x 4 for images of a few rows: where there are at most 2 of them to one of
//    256 x 20 and 1.5 to one of 64 x 32 (a tile takes half the time of the former
//    or less, 0.6 of the latter's).
//  * 256 x 20 otherwise. us for 512, 128, 48 and 16 separable images (24600,
//    6300, 2200 and 630 tiles of 256 x 16), windows of 512 tiles: 256 x 20 247,
//    65.9, 23.5, 8.8; 256 x 16 255, 66.2, 23.3, 9.0; 256 x 24 243, 66.0, 23.2,
//    9.7; with windows of 2048 256 x 32 257, 69.8, 25.2, 10.5; 128 x 16 284, 75.7,
//    22.9, 8.8; 64 x 32 312, 82, 24.7, 8.4.
struct BatchShape {
    int w, h;
};
constexpr int kBatchShapeCount = 4;
constexpr BatchShape kBatchShapes[kBatchShapeCount] = {{64, 16}, {64, 32}, {256, 4}, {256, 20}};
constexpr int64_t kBatchSmallTiles = 8 * 256;

// Tiles per window of the launch (window_tile): the images of a batch have few
// rows of tiles each, and a small window keeps the HBM pages in use few (512
// images, 256 x 20: 247 us, windows of 1024 252 us, of 2048 262 us; 128 images
// 65.9, 68.1 and 70.6 us; of 256 244 and 65.5 us, but 48 images 24.1 against
// 23.5 us).
constexpr int kBatchWindow = 512;

// One image of a batch as the batch kernel sees it. `var` is the executed
// variant (PF_VAR_*); its tiles are numbered row by row, tiles_x to a row.
// Element offsets are added to the kernel's base pointers as integers, so a
// descriptor may also carry an absolute address (byte address / 4) with a
// null base.
struct BatchImg {
    int64_t in_off;
    int64_t out_off;
    int64_t filt_off;
    int32_t h, w, r, var;
    int32_t tiles_x, tiles_y;
};

// One entry of a batch's tile list: the image (index into the descriptor
// array) and the tile's number inside the image.
struct BatchTask {
    int32_t img, tile;
};

inline int64_t batch_tiles(int h, int w, int shape) {
    const BatchShape t = kBatchShapes[shape];
    return (((int64_t)w + t.w - 1) / t.w) * (((int64_t)h + t.h - 1) / t.h);
}

// The shape for the images of a batch (h and w set), whose tiles_x and
// tiles_y it fills; *tiles: how many there are.
inline int batch_shape(std::vector<BatchImg> &imgs, int64_t *tiles) {
    int64_t n[kBatchShapeCount] = {};
    for (const BatchImg &d : imgs)
        for (int s = 0; s < kBatchShapeCount; ++s) n[s] += batch_tiles(d.h, d.w, s);
    int shape = 3;
    if (n[0] <= kBatchSmallTiles) shape = 0;
    else if (n[2] <= 2 * n[3] && 2 * n[2] <= 3 * n[1]) shape = 2;
    else if (5 * n[1] <= 9 * n[3]) shape = 1;
    const BatchShape t = kBatchShapes[shape];
    for (BatchImg &d : imgs) {
        d.tiles_x = (int32_t)(((int64_t)d.w + t.w - 1) / t.w);
        d.tiles_y = (int32_t)(((int64_t)d.h + t.h - 1) / t.h);
    }
    *tiles = n[shape];
    return shape;
}

// Appends the tiles of image `img` (descriptor d) to a batch's tile list.
inline void append_tiles(std::vector<BatchTask> &list, int32_t img, const BatchImg &d) {
    const int32_t n = d.tiles_x * d.tiles_y;
    for (int32_t t = 0; t < n; ++t) list.push_back({img, t});
}

// Host tables of a batch plan (batch.cpp): the image descriptors, the flat
// tile list and the shape of its tiles, the variant of each image, and the
// set of variants used (bit v: PF_VAR_*).
struct PlanTables {
    std::vector<BatchImg> imgs;
    std::vector<BatchTask> tasks;
    std::vector<int32_t> variant;
    int shape = 0, used = 0;
};
pf_status build_plan_tables(int32_t n, const int32_t *h, const int32_t *w, const int32_t *r, const int32_t *kind,
                            const int64_t *pix_off, const int64_t *filt_off, int64_t npix, int64_t nfilt,
                            int32_t flags, PlanTables *t);
int64_t check_plan_tables(const PlanTables &t, int64_t npix, std::string *first);

// Workgroups of a batch launch, one per tile: x is kept well inside the 2^32
// work items of a launch dimension.
inline dim3 batch_grid(int64_t ntasks) {
    const int64_t x = std::min<int64_t>(ntasks, 1 << 22);
    return dim3((unsigned)x, (unsigned)((ntasks + x - 1) / x));
}

// Size class used by the tune table.
inline int size_class(int64_t pixels) {
    return pixels < 256 * 256 ? 0 : (pixels > 1024 * 1024 ? 2 : 1);
}

// Device properties the launchers need (cached per device).
struct DevInfo {
    int device = -1;
    int cus = 0;
    std::string arch;
};
const DevInfo &dev_info();

// Thread-local error text.
pf_status fail(pf_status s, const std::string &msg);
pf_status fail_hip(hipError_t e, const char *what);
void clear_error();

// Launchers (kernels.hip). All validate nothing: callers have already.
// Single-image calls on LDS tiles (tile.hip): fa: 2D taps (sep false) or
// fx; fb: fy (ignored for 2D taps); border: PF_BORDER_* (2D; the separable
// kernel clamps); radius 0 goes to launch_point. tile_fits: the grid stays
// within the 2^32 work items a launch dimension holds (images of a few columns
// and hundreds of millions of rows do not; the strip kernel takes those).
constexpr int kTileThreads = 256;
inline bool tile_fits(int r, int h, int w) {
    return r == 0 || ((int64_t)w + 63) / 64 * (((int64_t)h + 15) / 16) * kTileThreads < ((int64_t)1 << 32);
}
hipError_t launch_tile(int r, bool sep, bool exact, const float *in, const float *fa, const float *fb, float *out,
                       int h, int w, int border, hipStream_t s);
// Radius 0 (point.hip): n pixels, `passes` passes with the weight *fa, then one
// with *fb unless it is null.
hipError_t launch_point(bool exact, const float *in, const float *fa, const float *fb, float *out, int64_t n,
                        int passes, hipStream_t s);
// The strip kernel with an explicit shape. fa: 2D taps (PF_VAR_DIRECT) or fx; fb: fy (ignored for PF_VAR_DIRECT).
hipError_t launch_f32(int r, int var, bool exact, const float *in, const float *fa, const float *fb, float *out,
                      int h, int w, int by, int wpg, hipStream_t s);
// var: PF_VAR_DIRECT (v_dot4) or PF_VAR_MFMA (int8 matrix cores, u8_mfma.hip).
hipError_t launch_u8(int r, int var, const uint8_t *in, const int8_t *filt, uint8_t *out, int c, int h,
                     int w, int shift, int by, int wpg, hipStream_t s);
hipError_t launch_u8_mfma(int r, const uint8_t *in, const int8_t *filt, uint8_t *out, int c, int h, int w,
                          int shift, int rpw, int wpg, hipStream_t s);
// Whether the uint8 variant runs at radius r with this launch shape.
bool u8_variant_ok(int var, int r, int by, int wpg);
// Batch kernel over images with r <= PF_BATCH_R_MAX and variants of `used`
// (a set of bits).
hipError_t launch_batch(bool exact, int used, int shape, const BatchImg *imgs, const BatchTask *tasks, int64_t ntasks,
                        const float *in, const float *filt, float *out, hipStream_t s);
// Fused chain of `passes` 2D passes under a border rule (chain.hip); also
// the single-pass filter for borders other than clamp.
hipError_t launch_chain(int r, bool exact, const float *in, const float *filt, float *out, int h, int w, int passes,
                        int border, hipStream_t s);
// Reductions (reduce.hip): workspace sizes and the two-launch sum and
// histogram.
size_t sum_workspace_bytes(int64_t n);
size_t hist_workspace_bytes(int64_t n);
hipError_t launch_sum(const float *x, int64_t n, double *out, void *workspace, hipStream_t s);
// Sub-histograms (1 KiB of workspace each) that an n-byte histogram runs
// fastest with; launch_hist takes as many of them as the workspace holds.
int64_t hist_rows_wanted(int64_t n);
hipError_t launch_hist(const uint8_t *x, int64_t n, int64_t *hist, void *workspace, size_t workspace_bytes,
                       hipStream_t s);
// Reduction requests of a server batch (reduce.hip). in / out are absolute
// device addresses (the input array; double[2] or int64_t[256] result);
// `first` is the request's first slot in the batch workspace: chunk
// partials (double) for sums, span sub-histograms (256 x uint32) for
// histograms; `op` is PF_OP_SUM_F32 or PF_OP_HIST_U8.
struct ReduceReq {
    int64_t in, n, out, first;
    int32_t op, pad;
};
// Part `part` (chunk or span) of request `req`.
struct ReduceTask {
    int32_t req, part;
};
// Chunks (sum) or spans (histogram) of an n-element request.
int64_t reduce_parts(int op, int64_t n);
// All sums, then all histograms of a batch: two launches each.
hipError_t launch_reduce_batch(const ReduceReq *reqs, const int32_t *sum_ids, int nsum, const ReduceTask *sum_tasks,
                               int n_sum_tasks, const int32_t *hist_ids, int nhist, const ReduceTask *hist_tasks,
                               int n_hist_tasks, double *partial, uint32_t *sub, hipStream_t s);
// The sum's static device scratch (reduce.hip): its capacity in elements and
// its address on the current device.
int64_t sum_noalloc_max();
hipError_t sum_scratch(void **ptr);
void *batch_kernel_fn(bool exact, int used, int shape);

// Per-radius FP32 launchers, each defined in its own instantiation unit.
template <int R>
hipError_t launch_f32_radius(int var, bool exact, const float *in, const float *fa, const float *fb, float *out,
                             int h, int w, int by, int wpg, hipStream_t s);
template <int R>
hipError_t launch_tile_radius(bool sep, bool exact, const float *in, const float *fa, const float *fb, float *out,
                              int h, int w, int border, hipStream_t s);
template <int R>
hipError_t launch_chain_radius(bool exact, const float *in, const float *filt, float *out, int h, int w, int passes,
                               int border, hipStream_t s);
#define PF_DECL_STRIP(R)                                                                                   \
    template <>                                                                                            \
    hipError_t launch_f32_radius<R>(int var, bool exact, const float *in, const float *fa, const float *fb, \
                                    float *out, int h, int w, int by, int wpg, hipStream_t s);
#define PF_DECL_RADIUS(R)                                                                                  \
    PF_DECL_STRIP(R)                                                                                       \
    template <>                                                                                            \
    hipError_t launch_tile_radius<R>(bool sep, bool exact, const float *in, const float *fa,               \
                                     const float *fb, float *out, int h, int w, int border,                \
                                     hipStream_t s);                                                       \
    template <>                                                                                            \
    hipError_t launch_chain_radius<R>(bool exact, const float *in, const float *filt, float *out, int h,    \
                                      int w, int passes, int border, hipStream_t s);
PF_DECL_STRIP(0)
PF_DECL_RADIUS(1)
PF_DECL_RADIUS(2)
PF_DECL_RADIUS(3)
PF_DECL_RADIUS(4)
PF_DECL_RADIUS(5)
PF_DECL_RADIUS(6)
PF_DECL_RADIUS(7)
PF_DECL_RADIUS(8)
#undef PF_DECL_RADIUS
#undef PF_DECL_STRIP

// Batch kernels per (exact, variant set), each in its own unit; the shape is
// an index into kBatchShapes. Sets: bit v for variant v: 1 (direct only), 2
// (separable only) and 3 (both). The separable-as-2D variant runs in
// single-image calls only.
template <int E, int M>
void *batch_fn(int shape);
#define PF_DECL_BATCH(E, M) \
    template <>             \
    void *batch_fn<E, M>(int shape);
PF_DECL_BATCH(0, 1)
PF_DECL_BATCH(1, 1)
PF_DECL_BATCH(0, 2)
PF_DECL_BATCH(1, 2)
PF_DECL_BATCH(0, 3)
PF_DECL_BATCH(1, 3)
#undef PF_DECL_BATCH

// Tune table lookup of single-image calls (tune.cpp).
pf_tune_entry tune_lookup(int kind, int r, int64_t pixels);

bool valid_shape(int by, int wpg);

}  // namespace pf

// FP32 single-image filters on LDS tiles: the full 2D and the separable
// kernel behind pf_filter2d_f32 and pf_filter_sep_f32, one radius (PF_R, set
// by the build) per object.
//
// pf_filter2d_f32_border and one-pass chains run the 2D kernel with their
// border rule. The tile itself is in tile_body.h.
//
// What bounds it: the 2D kernel at R >= 4 is bound by FP32 issue (4096 x
// 4096, R = 8: 137 us where (2R+1)^2 multiply-adds take 130 us at the
// measured 37.4 T lane-ops/s), all else by HBM from about 2 M pixels up and
// by the latency of load, barrier, compute, store below that. The strip
// kernel (filter_body.h), which ran these calls before, walks 256 columns per
// wave down the image: on one image that is few waves, each a long serial chain, and above R = 4 its 2R + 1 unrolled
// rows outgrow the instruction cache and its taps the scalar registers.
// Measured, strip -> tile, us, buffers rotated through 1 GiB: 256 x 256 R = 1
// 2.9 -> 2.6, R = 4 20.4 -> 3.5; 1080 x 1920 R = 2 13.3 -> 6.5; 1533 x 2047
// R = 6 84 -> 20.5; 4096 x 4096 R = 1 27.6 -> 25.4, R = 2 28.2 -> 26.0, R = 6
// 202 -> 86; separable 4096 x 4096 R = 2 27.6 -> 25.0, R = 6 56 -> 31; partly
// from the last-level cache (three images reused) 4096 x 4096 R = 2 22.9 ->
// 22.0. The strip won at no size from 64 x 64 to 8192 x 8192; it does on large
// images of a few rows (strip_wins in abi.cpp).
#include "tile_body.h"

#ifndef PF_R
#error "PF_R must be defined"
#endif

namespace pf {
namespace tile {

// Images of few rows and many columns: an XCD's contiguous share of a window's
// tiles would be part of one row of them, whose neighbours above and below are
// in other L2s. They are taken in panels of kPanel columns of tiles instead (64
// to 400 rows of 16000 to 100000 columns, three images reused, us: 100 x 64000 R =
// 1 11.4 -> 9.9, 200 x 32000 11.2 -> 9.8, separable R = 3 12.4 -> 10.0, 400 x
// 16000 11.0 -> 10.2; 800 x 8000 unchanged, 3000 x 12000 would take 57 instead of
// 53). Not in the 2D kernel at R >= 3, which is bound by arithmetic (unchanged
// there, and 1 to 2% slower for the other images).
constexpr int kPanel = 8, kPanelRows = 400;

// This workgroup's tile; panel: tiles of a panel, or 0.
template <bool PANELS>
__device__ __forceinline__ void own_tile(int tiles_x, int panel, int window, int &tx, int &ty) {
    window_tile(blockIdx.x, gridDim.x, tiles_x, window, tx, ty);
    if (!PANELS || panel == 0) return;
    const int t = ty * tiles_x + tx, first = t / panel * kPanel;
    const int in = t - first / kPanel * panel, columns = min(kPanel, tiles_x - first);
    ty = in / columns;
    tx = first + in - ty * columns;
}

template <int R, bool EXACT, int CX, int Q>
__global__ __launch_bounds__(kThreads) void k_tile_2d(const float *__restrict__ in, const float *__restrict__ filt,
                                                      float *__restrict__ out, int h, int w, int tiles_x, int panel,
                                                      int border) {
    __shared__ __align__(16) float buf[rows_of(R, CX, Q) * pitch_of(R, CX)];
    int tx, ty;
    own_tile<R <= 2>(tiles_x, panel, window_of(Q), tx, ty);
    tile_2d<R, EXACT, CX, Q>(buf, in, filt, out, h, w, tx * 4 * CX, ty * (kThreads / CX) * Q, border);
}

template <int R, bool EXACT, int CX, int Q>
__global__ __launch_bounds__(kThreads) void k_tile_sep(const float *__restrict__ in, const float *__restrict__ fx,
                                                       const float *__restrict__ fy, float *__restrict__ out, int h,
                                                       int w, int tiles_x, int panel) {
    __shared__ __align__(16) float buf[rows_of(R, CX, Q) * pitch_of(R, CX)];
    int tx, ty;
    own_tile<true>(tiles_x, panel, window_of(Q), tx, ty);
    tile_sep<R, EXACT, CX, Q>(buf, in, fx, fy, out, h, w, tx * 4 * CX, ty * (kThreads / CX) * Q);
}

template <int R, bool EXACT, bool SEP, int CX, int Q>
hipError_t launch_shape(const float *in, const float *fa, const float *fb, float *out, int h, int w, int border,
                        hipStream_t s) {
    const int64_t tiles_x = dev::cdiv(w, 4 * CX), tiles_y = dev::cdiv(h, kThreads / CX * Q), n = tiles_x * tiles_y;
    // Not the smallest shape, whose tiles are all in flight at once.
    const bool panels = CX * Q > 16 && tiles_y > 1 && h <= kPanelRows && tiles_x >= 4 * kPanel;
    const int panel = panels ? (int)tiles_y * kPanel : 0;
    if constexpr (SEP)
        hipLaunchKernelGGL((k_tile_sep<R, EXACT, CX, Q>), dim3((unsigned)n), dim3(kThreads), 0, s, in, fa, fb, out, h,
                           w, (int)tiles_x, panel);
    else
        hipLaunchKernelGGL((k_tile_2d<R, EXACT, CX, Q>), dim3((unsigned)n), dim3(kThreads), 0, s, in, fa, out, h, w,
                           (int)tiles_x, panel, border);
    return hipGetLastError();
}

// Tiles of 64 x 16 while all of them fit on the chip at once (8 workgroups
// of 4 waves per CU): the time is then one tile's, which a small tile keeps
// short (256 x 256, R = 4: 3.5 us against 4.7 us for the larger one; 1080 x
// 1920, 2040 tiles: 6.3 us against 7.3 us at R = 2). Beyond that a larger
// tile, whose halo weighs less (us; C: three images reused, partly in the
// last-level cache, H: eight or more, from HBM):
//  * 2D up to R = 2 and separable up to R = 3: 256 x 16, whole 1 KiB row
//    pieces (3000 x 4001, separable R = 2: H 21.6, 128 x 16 22.8, 128 x 32
//    23.3, 64 x 32 25.9; 1800 x 2500: C 8.2, 128 x 16 8.9), from 3 tiles per
//    CU; below 128 x 32, which divides among the CUs better (1080 x 1920: C
//    5.0 against 5.9; 1533 x 2047, 3 tiles per CU: both 7.6, 128 x 16 8.2).
//  * Other 2D: 128 x 16 at R = 3 (1800 x 2500: C 11.9, 256 x 16 12.5), 64 x 32
//    above (1533 x 2047, R = 7: C 24.3, 64 x 64 25.0).
//  * Other separable: 128 x 32 (4096 x 4096, R = 6: C 25.1, 64 x 32 26.7,
//    R = 8: H 31.0 against 35.1). With separate multiplies and adds at R >= 5
//    arithmetic weighs more than the halo's loads, and few tiles leave CUs
//    idle at the end: 64 x 32 up to 12 tiles per CU (1800 x 2500, R = 5: C
//    11.0, 128 x 32 12.2), then 64 x 64 (2160 x 3840, R = 6: C 17.1, 64 x 32
//    18.0; 4096 x 4096, R = 8: H 39.4 against 49.6).
// Images thinner than that tile waste it on padding (us, three images reused;
// the tile the rule above names, then the one taken):
//  * Up to 16 rows at R >= 4: 64 x 16 (16 x 10^6: 2D R = 4 81 and 49, R = 6 157
//    and 88; separable R = 6 42 and 34). Up to a few rows the strip kernel is
//    ahead of every tile at most radii; those calls do not come here.
//  * Of columns, where a narrower tile has a quarter less of them: 64 x 32 up to
//    64 and from 129 to 192 (400000 x 16: R = 1 71 and 28, separable R = 3 95
//    and 34; 50000 x 130, separable R = 3 17.2 and 15.1), 128 x 32 up to 128 and
//    from 257 to 384 (50000 x 100, R = 1: 13.9 and 9.9; 50000 x 300 23.0 and
//    21.9).
template <int R, bool EXACT, bool SEP>
hipError_t launch(const float *in, const float *fa, const float *fb, float *out, int h, int w, int border,
                  hipStream_t s) {
    const int64_t cus = dev_info().cus;
    auto tiles = [&](int tw, int th) { return (int64_t)dev::cdiv(w, tw) * dev::cdiv(h, th); };
#define PF_SHAPE(CX, Q) return launch_shape<R, EXACT, SEP, CX, Q>(in, fa, fb, out, h, w, border, s)
    auto columns = [&](int tw) { return (int64_t)dev::cdiv(w, tw) * tw; };  // with the padding
    auto quarter_less = [&](int tw) { return 4 * columns(tw) <= 3 * columns(2 * tw); };
    if (tiles(64, 16) <= 8 * cus || (R >= 4 && h <= 16)) PF_SHAPE(16, 1);
    if constexpr (SEP && EXACT && R >= 5) {
        if (tiles(64, 32) > 12 * cus) PF_SHAPE(16, 4);
        PF_SHAPE(16, 2);
    } else if constexpr (R <= (SEP ? 3 : 2)) {
        if (quarter_less(64)) PF_SHAPE(16, 2);
        if (tiles(256, 16) >= 3 * cus && !quarter_less(128)) PF_SHAPE(64, 4);
        PF_SHAPE(32, 4);
    } else if constexpr (SEP) {
        if (quarter_less(64)) PF_SHAPE(16, 2);
        PF_SHAPE(32, 4);
    } else if constexpr (R <= 3) {
        if (quarter_less(64)) PF_SHAPE(16, 2);
        PF_SHAPE(32, 2);
    } else {
        PF_SHAPE(16, 2);
    }
#undef PF_SHAPE
}

}  // namespace tile

template <>
hipError_t launch_tile_radius<PF_R>(bool sep, bool exact, const float *in, const float *fa, const float *fb,
                                    float *out, int h, int w, int border, hipStream_t s) {
    if (sep)
        return exact ? tile::launch<PF_R, true, true>(in, fa, fb, out, h, w, border, s)
                     : tile::launch<PF_R, false, true>(in, fa, fb, out, h, w, border, s);
    return exact ? tile::launch<PF_R, true, false>(in, fa, fb, out, h, w, border, s)
                 : tile::launch<PF_R, false, false>(in, fa, fb, out, h, w, border, s);
}

}  // namespace pf

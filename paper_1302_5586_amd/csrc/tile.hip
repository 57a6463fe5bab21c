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
// 22.0. The strip won at no size from 64 x 64 to 8192 x 8192.
#include "tile_body.h"

#ifndef PF_R
#error "PF_R must be defined"
#endif

namespace pf {
namespace tile {

template <int R, bool EXACT, int CX, int Q>
__global__ __launch_bounds__(kThreads) void k_tile_2d(const float *__restrict__ in, const float *__restrict__ filt,
                                                      float *__restrict__ out, int h, int w, int tiles_x,
                                                      int border) {
    __shared__ __align__(16) float buf[rows_of(R, CX, Q) * pitch_of(R, CX)];
    int tx, ty;
    window_tile(blockIdx.x, gridDim.x, tiles_x, tx, ty);
    tile_2d<R, EXACT, CX, Q>(buf, in, filt, out, h, w, tx * 4 * CX, ty * (kThreads / CX) * Q, border);
}

template <int R, bool EXACT, int CX, int Q>
__global__ __launch_bounds__(kThreads) void k_tile_sep(const float *__restrict__ in, const float *__restrict__ fx,
                                                       const float *__restrict__ fy, float *__restrict__ out, int h,
                                                       int w, int tiles_x) {
    __shared__ __align__(16) float buf[rows_of(R, CX, Q) * pitch_of(R, CX)];
    int tx, ty;
    window_tile(blockIdx.x, gridDim.x, tiles_x, tx, ty);
    tile_sep<R, EXACT, CX, Q>(buf, in, fx, fy, out, h, w, tx * 4 * CX, ty * (kThreads / CX) * Q);
}

template <int R, bool EXACT, int CX, int Q>
hipError_t launch_shape(bool sep, const float *in, const float *fa, const float *fb, float *out, int h, int w,
                        int border, hipStream_t s) {
    const int64_t tiles_x = dev::cdiv(w, 4 * CX), n = tiles_x * dev::cdiv(h, kThreads / CX * Q);
    if (sep)
        hipLaunchKernelGGL((k_tile_sep<R, EXACT, CX, Q>), dim3((unsigned)n), dim3(kThreads), 0, s, in, fa, fb, out, h,
                           w, (int)tiles_x);
    else
        hipLaunchKernelGGL((k_tile_2d<R, EXACT, CX, Q>), dim3((unsigned)n), dim3(kThreads), 0, s, in, fa, out, h, w,
                           (int)tiles_x, border);
    return hipGetLastError();
}

// Tiles of 64 x 16 while all of them fit on the chip at once (8 workgroups
// of 4 waves per CU): the time is then one tile's, which a small tile keeps
// short (256 x 256, R = 4: 3.5 us against 4.7 us for the larger one; 1080 x
// 1920, 2040 tiles: 6.3 us against 7.3 us at R = 2). Beyond that a larger
// tile, whose halo weighs less: 128 x 16 up to R = 3 (whole 512-byte row
// pieces; 4096 x 4096, R = 1: 25.5 us against 27.5 us for 64 x 32), 64 x 32
// above (half the vertical halo; separable R = 6: 31.6 us against 36.1 us).
template <int R, bool EXACT>
hipError_t launch(bool sep, const float *in, const float *fa, const float *fb, float *out, int h, int w, int border,
                  hipStream_t s) {
    if ((int64_t)dev::cdiv(w, 64) * dev::cdiv(h, 16) <= 8 * (int64_t)dev_info().cus)
        return launch_shape<R, EXACT, 16, 1>(sep, in, fa, fb, out, h, w, border, s);
    if constexpr (R <= 3) return launch_shape<R, EXACT, 32, 2>(sep, in, fa, fb, out, h, w, border, s);
    else return launch_shape<R, EXACT, 16, 2>(sep, in, fa, fb, out, h, w, border, s);
}

}  // namespace tile

template <>
hipError_t launch_tile_radius<PF_R>(bool sep, bool exact, const float *in, const float *fa, const float *fb,
                                    float *out, int h, int w, int border, hipStream_t s) {
    return exact ? tile::launch<PF_R, true>(sep, in, fa, fb, out, h, w, border, s)
                 : tile::launch<PF_R, false>(sep, in, fa, fb, out, h, w, border, s);
}

}  // namespace pf

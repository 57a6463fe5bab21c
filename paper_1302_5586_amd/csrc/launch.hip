// Radius dispatch for the single-image kernels and the uint8 kernels, and the
// batch kernel's launch.
#include "filter_body.h"

namespace pf {

hipError_t launch_f32(int r, int var, bool exact, const float *in, const float *fa, const float *fb, float *out,
                      int h, int w, int by, int wpg, hipStream_t s) {
    switch (r) {
        case 0: return launch_f32_radius<0>(var, exact, in, fa, fb, out, h, w, by, wpg, s);
        case 1: return launch_f32_radius<1>(var, exact, in, fa, fb, out, h, w, by, wpg, s);
        case 2: return launch_f32_radius<2>(var, exact, in, fa, fb, out, h, w, by, wpg, s);
        case 3: return launch_f32_radius<3>(var, exact, in, fa, fb, out, h, w, by, wpg, s);
        case 4: return launch_f32_radius<4>(var, exact, in, fa, fb, out, h, w, by, wpg, s);
        case 5: return launch_f32_radius<5>(var, exact, in, fa, fb, out, h, w, by, wpg, s);
        case 6: return launch_f32_radius<6>(var, exact, in, fa, fb, out, h, w, by, wpg, s);
        case 7: return launch_f32_radius<7>(var, exact, in, fa, fb, out, h, w, by, wpg, s);
        case 8: return launch_f32_radius<8>(var, exact, in, fa, fb, out, h, w, by, wpg, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_tile(int r, bool sep, bool exact, const float *in, const float *fa, const float *fb, float *out,
                       int h, int w, int border, hipStream_t s) {
    switch (r) {
        case 0: return launch_point(exact, in, fa, sep ? fb : nullptr, out, (int64_t)h * w, 1, s);
        case 1: return launch_tile_radius<1>(sep, exact, in, fa, fb, out, h, w, border, s);
        case 2: return launch_tile_radius<2>(sep, exact, in, fa, fb, out, h, w, border, s);
        case 3: return launch_tile_radius<3>(sep, exact, in, fa, fb, out, h, w, border, s);
        case 4: return launch_tile_radius<4>(sep, exact, in, fa, fb, out, h, w, border, s);
        case 5: return launch_tile_radius<5>(sep, exact, in, fa, fb, out, h, w, border, s);
        case 6: return launch_tile_radius<6>(sep, exact, in, fa, fb, out, h, w, border, s);
        case 7: return launch_tile_radius<7>(sep, exact, in, fa, fb, out, h, w, border, s);
        case 8: return launch_tile_radius<8>(sep, exact, in, fa, fb, out, h, w, border, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_chain(int r, bool exact, const float *in, const float *filt, float *out, int h, int w, int passes,
                        int border, hipStream_t s) {
    if (r == 0) return launch_point(exact, in, filt, nullptr, out, (int64_t)h * w, passes, s);
    // One pass has nothing to fuse: the tile kernel (4096 x 4096 reflect, R =
    // 1: 25 us, the chain's own tiles 29 us).
    if (passes == 1 && tile_fits(r, h, w)) return launch_tile(r, false, exact, in, filt, nullptr, out, h, w, border, s);
    switch (r) {
        case 1: return launch_chain_radius<1>(exact, in, filt, out, h, w, passes, border, s);
        case 2: return launch_chain_radius<2>(exact, in, filt, out, h, w, passes, border, s);
        case 3: return launch_chain_radius<3>(exact, in, filt, out, h, w, passes, border, s);
        case 4: return launch_chain_radius<4>(exact, in, filt, out, h, w, passes, border, s);
        case 5: return launch_chain_radius<5>(exact, in, filt, out, h, w, passes, border, s);
        case 6: return launch_chain_radius<6>(exact, in, filt, out, h, w, passes, border, s);
        case 7: return launch_chain_radius<7>(exact, in, filt, out, h, w, passes, border, s);
        case 8: return launch_chain_radius<8>(exact, in, filt, out, h, w, passes, border, s);
        default: return hipErrorInvalidValue;
    }
}

bool u8_variant_ok(int var, int r, int by, int wpg) {
    if (var == PF_VAR_DIRECT) return true;
    return var == PF_VAR_MFMA && r >= 1 && r <= PF_U8_MFMA_R_MAX && by % 16 == 0 && by * wpg <= PF_U8_MFMA_TILE_MAX;
}

hipError_t launch_u8(int r, int var, const uint8_t *in, const int8_t *filt, uint8_t *out, int c, int h, int w,
                     int shift, int by, int wpg, hipStream_t s) {
    if (var == PF_VAR_MFMA) {
        if (!u8_variant_ok(var, r, by, wpg)) return hipErrorInvalidValue;
        return launch_u8_mfma(r, in, filt, out, c, h, w, shift, by, wpg, s);
    }
    if (var != PF_VAR_DIRECT) return hipErrorInvalidValue;
    switch (r) {
        case 0: return dev::launch_u8_t<0>(in, filt, out, c, h, w, shift, by, wpg, s);
        case 1: return dev::launch_u8_t<1>(in, filt, out, c, h, w, shift, by, wpg, s);
        case 2: return dev::launch_u8_t<2>(in, filt, out, c, h, w, shift, by, wpg, s);
        case 3: return dev::launch_u8_t<3>(in, filt, out, c, h, w, shift, by, wpg, s);
        case 4: return dev::launch_u8_t<4>(in, filt, out, c, h, w, shift, by, wpg, s);
        case 5: return dev::launch_u8_t<5>(in, filt, out, c, h, w, shift, by, wpg, s);
        case 6: return dev::launch_u8_t<6>(in, filt, out, c, h, w, shift, by, wpg, s);
        case 7: return dev::launch_u8_t<7>(in, filt, out, c, h, w, shift, by, wpg, s);
        case 8: return dev::launch_u8_t<8>(in, filt, out, c, h, w, shift, by, wpg, s);
        default: return hipErrorInvalidValue;
    }
}

void *batch_kernel_fn(bool exact, int used, int shape) {
    switch (used) {
        case 1: return exact ? batch_fn<1, 1>(shape) : batch_fn<0, 1>(shape);
        case 2: return exact ? batch_fn<1, 2>(shape) : batch_fn<0, 2>(shape);
        default: return exact ? batch_fn<1, 3>(shape) : batch_fn<0, 3>(shape);
    }
}

hipError_t launch_batch(bool exact, int used, int shape, const BatchImg *imgs, const BatchTask *tasks, int64_t ntasks,
                        const float *in, const float *filt, float *out, hipStream_t s) {
    int n = (int)ntasks;
    void *params[] = {&imgs, &tasks, &n, &in, &filt, &out};
    return hipLaunchKernel(batch_kernel_fn(exact, used, shape), batch_grid(ntasks), dim3(kTileThreads), params, 0,
                           s);
}

}  // namespace pf

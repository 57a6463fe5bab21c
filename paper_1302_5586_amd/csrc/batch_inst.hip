// The batch kernel: the tiles (tile_body.h) of all images of a batch in one
// launch. One object per arithmetic and variant set, selected by the build:
//   PF_EXACT: 0 fused multiply-add, 1 separate multiply and add;
//   PF_VMASK: bit v set if variant v (PF_VAR_*) is compiled in.
#include "tile_body.h"

#if !defined(PF_EXACT) || !defined(PF_VMASK)
#error "PF_EXACT and PF_VMASK must be defined"
#endif

namespace pf {
namespace tile {

static_assert(PF_BATCH_R_MAX == 4, "k_batch lists its radii");

// The tile at (x0, y0) of image d, whose radius is R.
template <int R, bool EXACT, int VMASK, int CX, int Q>
__device__ __forceinline__ void one_tile(float *buf, const BatchImg &d, const float *__restrict__ in,
                                         const float *__restrict__ filt, float *__restrict__ out, int x0, int y0) {
    constexpr bool kBoth = VMASK == (1 << PF_VAR_DIRECT | 1 << PF_VAR_SEPARABLE);
    if constexpr ((VMASK >> PF_VAR_DIRECT) & 1)
        if (!kBoth || d.var == PF_VAR_DIRECT)
            tile_2d<R, EXACT, CX, Q>(buf, in, filt, out, d.h, d.w, x0, y0, PF_BORDER_CLAMP);
    if constexpr ((VMASK >> PF_VAR_SEPARABLE) & 1)
        if (!kBoth || d.var == PF_VAR_SEPARABLE)
            tile_sep<R, EXACT, CX, Q>(buf, in, filt, filt + 2 * R + 1, out, d.h, d.w, x0, y0);
}

// One workgroup per tile of the list (which goes image by image, row by row
// inside each), its image's radius and variant picked by a branch that is
// uniform. Bound by HBM with what the halo costs on top: 512 images, 78 M
// pixels, radii 1..4, separable: 247 us (5.05 TB/s) where the card copies the
// bytes in 208 us; rows that start anywhere cost 8%, radius 4 against 1
// another 7%. The strips that a fixed grid of one workgroup per CU walked
// before took 300 us, and on smaller batches, where such a strip is a long
// serial chain: 256 images 160 -> 127, 128 92 -> 66, 48 37.8 -> 23.5, 16 21
// -> 9 us.
template <bool EXACT, int VMASK, int CX, int Q>
__global__ __launch_bounds__(kThreads) void k_batch(const BatchImg *__restrict__ imgs,
                                                    const BatchTask *__restrict__ tasks, int ntasks,
                                                    const float *__restrict__ in, const float *__restrict__ filt,
                                                    float *__restrict__ out) {
    __shared__ __align__(16) float buf[rows_of(PF_BATCH_R_MAX, CX, Q) * pitch_of(PF_BATCH_R_MAX, CX)];
    int zero, at;
    window_tile(blockIdx.x, gridDim.x, 1, kBatchWindow, zero, at);
    // No loop over tiles: the compiler would keep every radius' invariants in
    // registers across it (217 instead of 70).
    const int64_t t = (int64_t)blockIdx.y * gridDim.x + at;
    if (t >= ntasks) return;
    const BatchTask tk = tasks[t];
    const BatchImg d = imgs[tk.img];
    const int ty = tk.tile / d.tiles_x, tx = tk.tile - ty * d.tiles_x;
    const int x0 = tx * 4 * CX, y0 = ty * (kThreads / CX) * Q;
    const float *src = dev::global_at(in, d.in_off);
    float *dst = dev::global_at(out, d.out_off);
    const float *fa = dev::global_at(filt, d.filt_off);
    switch (d.r) {
        case 0: one_tile<0, EXACT, VMASK, CX, Q>(buf, d, src, fa, dst, x0, y0); break;
        case 1: one_tile<1, EXACT, VMASK, CX, Q>(buf, d, src, fa, dst, x0, y0); break;
        case 2: one_tile<2, EXACT, VMASK, CX, Q>(buf, d, src, fa, dst, x0, y0); break;
        case 3: one_tile<3, EXACT, VMASK, CX, Q>(buf, d, src, fa, dst, x0, y0); break;
        case 4: one_tile<4, EXACT, VMASK, CX, Q>(buf, d, src, fa, dst, x0, y0); break;
    }
}

}  // namespace tile

template <>
void *batch_fn<PF_EXACT, PF_VMASK>(int shape) {
    constexpr bool kExact = PF_EXACT != 0;
    switch (shape) {
        case 0: return (void *)tile::k_batch<kExact, PF_VMASK, kBatchShapes[0].w / 4, 1>;
        case 1: return (void *)tile::k_batch<kExact, PF_VMASK, kBatchShapes[1].w / 4, 2>;
        case 2: return (void *)tile::k_batch<kExact, PF_VMASK, kBatchShapes[2].w / 4, 1>;
        default: return (void *)tile::k_batch<kExact, PF_VMASK, kBatchShapes[3].w / 4, 5>;
    }
}

}  // namespace pf

// Chains of 2D filter passes fused in one kernel, under four border rules;
// one radius (PF_R, set by the build) per object.
//
// A chain applies the same (2r+1)^2 filter `passes` times; pass p reads the
// FP32 image pass p-1 produced, with that image extended past its edges by
// the border rule. Composing several stencil passes into one kernel is the
// cross-component optimisation the paper motivates (Sec. II), for the
// image-processing and fluid-dynamics stencil domains it names (Sec. I);
// every pass keeps the independent-iteration semantics of Sec. II-B.3. Only
// the input is read from HBM and only the last pass is written: 8 bytes per
// pixel for the whole chain instead of 8 per pass.
//
// Two forms, the same bits from both:
//
//  * Tiles (k_chain_tiles): a workgroup owns an output tile, stages it with
//    a halo of H = R * passes in LDS, border-extended, and runs the passes
//    between two LDS images. Pass p computes, from the image of pass p-1,
//    every in-image position within H - p R of the tile; a tile at the
//    image's edge then writes the border extension of that result. A thread
//    takes 4 x Q outputs at a time, window rows in registers as in the tile
//    kernel (tile.hip). Any size, radius and pass count.
//  * Streams (k_chain_stream): a wave walks a strip of 256 columns down the
//    image and runs every pass in registers: pass p folds each row of pass
//    p-1 into a ring of 2R+1 row accumulators as the row is completed, so an
//    input row costs each pass its multiply-adds and 2R lane shifts and
//    nothing is staged, exchanged or waited for but the next input row. The
//    strips cover the image but for a frame of at most 64 columns and 32
//    rows, which workgroups at the end of the same launch compute as tiles.
//
// Arithmetic per output: taps in definition order (dy outer, dx inner,
// ascending), one FMA per tap, or with EXACT a separate FP32 multiply and
// add (built with -ffp-contract=off), which reproduces the sequential
// program bit for bit at every pass.
//
// What bounds it: large images, FP32 issue (and at one or two 3 x 3 passes
// HBM); small ones, the passes' latency in one tile, about 0.9 us each at the
// image's edge (LDS reads, a barrier, the extension, a barrier). The chain
// before held one LDS image of 64 x 32 tiles, a pass's results in registers
// over a barrier, 4 x 4 outputs per thread. Before -> now, us, three images
// reused: 4 x (3 x 3) over 4096 x 4096 70 -> 30, over 1080 x 1920 24 -> 13,
// over 64 x 64 20 -> 9; 8 x (5 x 5) over 4096 x 4096 281 -> 154; 5 x (7 x 7)
// over 2160 x 2600 126 -> 90.
#include "filter_body.h"

#ifndef PF_R
#error "PF_R must be defined"
#endif

namespace pf {
namespace chain {

using dev::f4u;
using dev::madd;
using dev::static_for;

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;

__host__ __device__ constexpr int ceil4(int v) { return (v + 3) / 4 * 4; }
constexpr int pad_of(int r) { return ceil4(r); }
constexpr int window_vecs(int r) { return 1 + pad_of(r) / 2; }
// Buffer columns left of the tile: what the first pass's region and its
// window reach. h: halo R * passes.
__host__ __device__ constexpr int left_of(int r, int h) { return ceil4(h > r ? h - r : 0) + pad_of(r); }

// Workgroup barrier that orders LDS only (a plain __syncthreads() also
// waits for every global access in flight).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One tile: outputs [y0, ye) x [x0, xe), at most TY x TX of them. `first`
// (0..3): the wave that takes a pass's first task; a pass of fewer tasks than
// threads leaves whole waves idle, each on its own SIMD, so it moves on past
// the waves the previous pass used. lds: 2 images of (TY + 2H + Q - 1) rows.
template <int R, bool EXACT, int TX, int TY, int Q>
__device__ __forceinline__ void chain_tile(const float *__restrict__ in, const float *__restrict__ filt,
                                           float *__restrict__ out, int h, int w, int passes, int border, int x0,
                                           int y0, int xe, int ye, int first, float *lds) {
    constexpr int K = 2 * R + 1, PAD = pad_of(R), NB = window_vecs(R);
    constexpr bool ALL = K * K <= 49;  // every tap stays in scalar registers
    const int H = R * passes, LEFT = left_of(R, H);
    const int pitch = TX + 2 * LEFT, rows = TY + 2 * H;
    const int image = (rows + Q - 1) * pitch;  // floats of one LDS image
    const bool interior = x0 >= LEFT && w - x0 >= TX + LEFT && y0 >= H && h - y0 >= TY + H;
    float wt[ALL ? 1 : 2][ALL ? K * K : K];
    load_taps(filt, wt[0]);
    {
        // Pass 0: rows y0 - H .., columns x0 - LEFT .., border-extended. LC
        // lanes across a row.
        constexpr int LC = TX + 2 * left_of(R, 16) <= 128 ? 32 : 64, LR = kThreads / LC, DEEP = 6;
        const int c = 4 * (threadIdx.x % LC), r0 = threadIdx.x / LC;
        const bool on = c < pitch;
        if (interior) {
            const float *src = in + (int64_t)(y0 - H) * w + (x0 - LEFT);
            for (int b = 0; b < rows; b += DEEP * LR) {
                f4 v[DEEP];
#pragma unroll
                for (int u = 0; u < DEEP; ++u)
                    if (on && b + r0 + LR * u < rows)
                        v[u] = *reinterpret_cast<const f4u *>(src + (int64_t)(b + r0 + LR * u) * w + c);
#pragma unroll
                for (int u = 0; u < DEEP; ++u)
                    if (on && b + r0 + LR * u < rows)
                        *reinterpret_cast<f4 *>(lds + (b + r0 + LR * u) * pitch + c) = v[u];
            }
        } else {
            int xs[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) xs[k] = border_index(x0 - LEFT + c + k, w, border);
            for (int b = 0; b < rows; b += DEEP * LR) {
                f4 v[DEEP];
#pragma unroll
                for (int u = 0; u < DEEP; ++u) {
                    const int r = b + r0 + LR * u;
                    const int y = border_index(y0 - H + r, h, border);
                    v[u] = f4{0.0f, 0.0f, 0.0f, 0.0f};
                    if (on && r < rows && y >= 0) {
                        const float *src = in + (int64_t)y * w;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (xs[k] >= 0) v[u][k] = src[xs[k]];
                    }
                }
#pragma unroll
                for (int u = 0; u < DEEP; ++u)
                    if (on && b + r0 + LR * u < rows)
                        *reinterpret_cast<f4 *>(lds + (b + r0 + LR * u) * pitch + c) = v[u];
            }
        }
    }
    __syncthreads();
    float *cur = lds, *nxt = lds + image;
    for (int p = 1; p <= passes; ++p) {
        const bool last = p == passes;
        const int m = (passes - p) * R;
        const int ylo = max(y0 - m, 0), yhi = ye + min(m, h - ye);
        const int xlo = max(x0 - m, 0), xhi = xe + min(m, w - xe);
        // Tasks: 4 x Q outputs, rows from ylo in steps of Q, 4-aligned buffer
        // columns covering [xlo, xhi). Window reads stay inside an image: rows
        // from H - m - R >= 0 to at most TY + 2H + Q - 2, columns from
        // LEFT - ceil4(m) - PAD >= 0 to TX + LEFT + ceil4(m) + PAD <= pitch.
        // Outputs past the region are computed from whatever is there: the
        // last pass does not store them, the next one reads none of them but
        // the positions that the extension below rewrites first.
        const int cb0 = (xlo - x0 + LEFT) >> 2, cb1 = (xhi - x0 + LEFT + 3) >> 2;
        const int ncb = cb1 - cb0, ntask = ((yhi - ylo + Q - 1) / Q) * ncb;
        const int v0 = (threadIdx.x - 64 * first) & (kThreads - 1);
        int tr = v0 / ncb, tc = v0 - tr * ncb;
        const int dr = kThreads / ncb, dc = kThreads - dr * ncb;
        for (int t = v0; t < ntask; t += kThreads) {
            const int row = ylo + Q * tr - (y0 - H), col = 4 * (cb0 + tc);
            int at = (row - R) * pitch + col - PAD;
            float acc[Q][4];
#pragma unroll
            for (int j = 0; j < Q; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[j][k] = 0.0f;
            float win[Q + 1][4 * NB];
#pragma unroll
            for (int j = 0; j < Q; ++j) load_window<NB>(cur + at + j * pitch, win[j]);
            at += Q * pitch;
            static_for<0, K>([&](auto dcst) __attribute__((always_inline)) {
                constexpr int dy = decltype(dcst)::value;
                if constexpr (!ALL) load_taps<K>(filt + (dy + 1 < K ? dy + 1 : 0) * K, wt[ALL ? 0 : (dy + 1) & 1]);
                if constexpr (dy + 1 < K) {
                    asm volatile("" : "+v"(at));
                    load_window<NB>(cur + at, win[(dy + Q) % (Q + 1)]);
                    at += pitch;
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int dx = 0; dx < K; ++dx)
#pragma unroll
                    for (int j = 0; j < Q; ++j)
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            acc[j][k] = madd<EXACT>(ALL ? wt[0][ALL ? dy * K + dx : 0] : wt[ALL ? 0 : dy & 1][dx],
                                                    win[(dy + j) % (Q + 1)][PAD - R + k + dx], acc[j][k]);
                end_step<Q>(acc);
            });
            if constexpr (!ALL) {
                // K is odd: the next task's tap row 0 was loaded to slot 1.
#pragma unroll
                for (int i = 0; i < K; ++i) wt[0][i] = wt[1][i];
            }
            if (last) {
                const int y = ylo + Q * tr, x = col - LEFT;  // relative to x0
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    if (y + j >= yhi) continue;
                    float *o = out + (int64_t)(y + j) * w + x0 + x;
                    if (x + 4 <= xhi - x0) {
                        const f4u q = {acc[j][0], acc[j][1], acc[j][2], acc[j][3]};
                        __builtin_nontemporal_store(q, reinterpret_cast<f4u *>(o));
                    } else {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (x + k < xhi - x0) __builtin_nontemporal_store(acc[j][k], o + k);
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const f4 q = {acc[j][0], acc[j][1], acc[j][2], acc[j][3]};
                    *reinterpret_cast<f4 *>(nxt + (row + j) * pitch + col) = q;
                }
            }
            tr += dr;
            tc += dc;
            if (tc >= ncb) {
                tc -= ncb;
                ++tr;
            }
        }
        if (last) break;
        first = (first + ((ntask + 63) >> 6)) & 3;
        lds_barrier();
        if (!interior) {
            // Border extension of this pass's image: the positions outside the
            // image that the next pass reads, those of its region within R of
            // the image: whole rows above and below, then what is left and
            // right of the rows between. Each source lies in the part just
            // written: a rule maps a position within R of an edge to within R
            // of it (m >= R here), or wraps inside an image narrower than a
            // tile, which a single tile covers.
            const int ya = max(y0 - m, -R), yb = ye + min(m, h - ye + R);
            const int xa = max(x0 - m, -R), xb = xe + min(m, w - xe + R);
            auto at = [&](int y, int x) -> float & { return nxt[(y - y0 + H) * pitch + x - x0 + LEFT]; };
            const int nv = (ylo - ya) + (yb - yhi), wv = xb - xa;
            for (int i = threadIdx.x; i < nv * wv; i += kThreads) {
                const int r = i / wv, x = xa + i - r * wv;
                const int y = r < ylo - ya ? ya + r : yhi + r - (ylo - ya);
                const int yy = border_index(y, h, border), xx = border_index(x, w, border);
                at(y, x) = (yy < 0 || xx < 0) ? 0.0f : at(yy, xx);
            }
            const int wc = (xlo - xa) + (xb - xhi), nc = yhi - ylo;
            for (int i = threadIdx.x; i < nc * wc; i += kThreads) {
                const int r = i / wc, c = i - r * wc, y = ylo + r;
                const int x = c < xlo - xa ? xa + c : xhi + c - (xlo - xa);
                const int xx = border_index(x, w, border);
                at(y, x) = xx < 0 ? 0.0f : at(y, xx);
            }
            lds_barrier();
        }
        float *sw = cur;
        cur = nxt;
        nxt = sw;
    }
}

template <int R, bool EXACT, int TX, int TY, int Q>
__global__ __launch_bounds__(kThreads) void k_chain_tiles(const float *__restrict__ in,
                                                          const float *__restrict__ filt, float *__restrict__ out,
                                                          int h, int w, int passes, int border, int tiles_x) {
    extern __shared__ __align__(16) float lds[];
    int tx, ty;
    window_tile(blockIdx.x, gridDim.x, tiles_x, 2048, tx, ty);
    const int x0 = tx * TX, y0 = ty * TY;
    chain_tile<R, EXACT, TX, TY, Q>(in, filt, out, h, w, passes, border, x0, y0, x0 + min(TX, w - x0),
                                    y0 + min(TY, h - y0), blockIdx.x & 3, lds);
}

// ---------------------------------------------------------------- streams

// What a stream launch covers: rows [ya, yb) x columns [xa, xb) in strips x
// bands wave tiles of `by` rows; `frame` workgroups for the rest, fx tiles
// per tile row above and below, then (1 + right) per tile row between.
struct StreamPlan {
    int xa, ya, xb, yb;
    int strips, bands, by;
    int frame, fx;
};
constexpr int kFrameX = 64, kFrameY = 32;  // a frame tile

// DPP wavefront shifts that give 0 to the lane without a source lane (a halo
// lane, whose values are not used): no register is set up first.
__device__ __forceinline__ float from_left0(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right0(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}

// Folds one row of a pass's input, 4 columns per lane, into its ring of row
// accumulators; RES: the row's number modulo K. Output row j collects rows
// j .. j + 2R and lives in slot j mod K; the slot of the row's first tap
// starts from 0.
template <int R, bool EXACT, int RES>
__device__ __forceinline__ void fold(const float (&wk)[(2 * R + 1) * (2 * R + 1)], const float (&v)[4],
                                     float (&acc)[2 * R + 1][4]) {
    constexpr int K = 2 * R + 1;
    static_assert(R <= 4, "a window within the adjacent lanes");
    float win[12];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        win[k] = from_left0(v[k]);
        win[4 + k] = v[k];
        win[8 + k] = from_right0(v[k]);
    }
#pragma unroll
    for (int dy = -R; dy <= R; ++dy) {
        const int slot = ((RES - R - dy) % K + K) % K;
#pragma unroll
        for (int dx = -R; dx <= R; ++dx)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                acc[slot][k] = madd<EXACT>(wk[(dy + R) * K + dx + R], win[4 + k + dx],
                                           dy == -R && dx == -R ? 0.0f : acc[slot][k]);
    }
}

// Passes p .. P - 1 for input row i of the strip (i = S modulo K): v, the row
// pass p reads, becomes the row the last pass completes. A pass starts with
// its first complete input row, 2R rows after the pass before it. One pass
// at a time for the scheduler: interleaved, their windows cost 30 to 90 more
// registers.
template <int R, int P, bool EXACT, int S, int p>
__device__ __forceinline__ void run_passes(const float (&wk)[(2 * R + 1) * (2 * R + 1)], float (&v)[4],
                                           float (&acc)[P][2 * R + 1][4], int i) {
    constexpr int K = 2 * R + 1;
    if (p > 0 && i < 2 * R * p) return;
    constexpr int RES = (S + p) % K;  // row i - 2R p of pass p's input
    fold<R, EXACT, RES>(wk, v, acc[p]);
    constexpr int done = (RES + 1) % K;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = acc[p][done][k];
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (p + 1 < P) run_passes<R, P, EXACT, S, p + 1>(wk, v, acc, i);
}

// Input rows in flight per wave: a multiple of K near 6 (9 at R = 1: 24 more
// registers and 34.6 us against 30.1 us for 4 passes over 4096 x 4096). Each
// row's register is loaded again as soon as its row is folded.
constexpr int stream_rows(int r) { return (2 * r + 1) * (6 / (2 * r + 1) > 0 ? 6 / (2 * r + 1) : 1); }

// One wave: outputs [y0, y0 + rows) x [x0, x0 + 256 - 8 IL), every halo row
// and column inside the image.
template <int R, int P, bool EXACT>
__device__ __forceinline__ void stream_strip(const float *__restrict__ in, const float *__restrict__ filt,
                                             float *__restrict__ out, int w, int x0, int y0, int rows, int lane) {
    constexpr int K = 2 * R + 1, H = R * P, IL = (H + 3) / 4, CH = stream_rows(R);
    float wk[K * K];
    load_taps<K * K>(filt, wk);
    float acc[P][K][4];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int s = 0; s < K; ++s)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[p][s][k] = 0.0f;
    const bool out_lane = lane >= IL && lane < 64 - IL;
    const int nin = rows + 2 * H;
    const float *src = in + (int64_t)(y0 - H) * w + (x0 - 4 * IL);
    float *dst = out + (int64_t)y0 * w + (x0 + 4 * (lane - IL));
    const uint32_t col = 4 * lane;
    f4 q[CH];
#pragma unroll
    for (int s = 0; s < CH; ++s) q[s] = *reinterpret_cast<const f4u *>(src + (int64_t)min(s, nin - 1) * w + col);
    src += (int64_t)min(CH, nin - 1) * w;  // row i + CH, or the last one
    for (int i0 = 0; i0 < nin; i0 += CH) {
        static_for<0, CH>([&](auto sc) __attribute__((always_inline)) {
            constexpr int s = decltype(sc)::value;
            const int i = i0 + s;
            float v[4] = {q[s].x, q[s].y, q[s].z, q[s].w};
            q[s] = *reinterpret_cast<const f4u *>(src + col);
            src += i + CH + 1 < nin ? w : 0;
            run_passes<R, P, EXACT, s, 0>(wk, v, acc, i);
            if (i >= 2 * H && i < nin && out_lane) {
                const f4u t = {v[0], v[1], v[2], v[3]};
                __builtin_nontemporal_store(t, reinterpret_cast<f4u *>(dst + (int64_t)(i - 2 * H) * w));
            }
        });
    }
}

// The strips come first in the grid, four waves per workgroup, so that they
// spread one workgroup per CU; the frame's tiles fill in behind them (frame
// first, two strip workgroups share some CUs and the launch takes up to
// twice as long).
template <int R, int P, bool EXACT>
__global__ __launch_bounds__(kThreads) void k_chain_stream(const float *__restrict__ in,
                                                           const float *__restrict__ filt, float *__restrict__ out,
                                                           int h, int w, int border, StreamPlan pl) {
    extern __shared__ __align__(16) float lds[];
    const int ns = gridDim.x - pl.frame;
    if ((int)blockIdx.x >= ns) {
        int b = blockIdx.x - ns, x0, y0, xe, ye;
        const int below = (h - pl.yb + kFrameY - 1) / kFrameY, right = (w - pl.xb + kFrameX - 1) / kFrameX;
        if (b < pl.fx * (1 + below)) {
            const int r = b / pl.fx;
            x0 = (b - r * pl.fx) * kFrameX;
            xe = min(x0 + kFrameX, w);
            y0 = r == 0 ? 0 : pl.yb + (r - 1) * kFrameY;
            ye = r == 0 ? pl.ya : min(y0 + kFrameY, h);
        } else {
            b -= pl.fx * (1 + below);
            const int r = b / (1 + right), c = b - r * (1 + right);
            y0 = pl.ya + r * kFrameY;
            ye = min(y0 + kFrameY, pl.yb);
            x0 = c == 0 ? 0 : pl.xb + (c - 1) * kFrameX;
            xe = c == 0 ? pl.xa : min(x0 + kFrameX, w);
        }
        chain_tile<R, EXACT, kFrameX, kFrameY, 2>(in, filt, out, h, w, P, border, x0, y0, xe, ye, blockIdx.x & 3, lds);
        return;
    }
    constexpr int IL = (R * P + 3) / 4, SW = 4 * (64 - 2 * IL);
    const int lane = threadIdx.x & 63, wave = dev::uniform(threadIdx.x >> 6);
    const int t = xcd_remap(blockIdx.x, ns) * 4 + wave;
    if (t >= pl.strips * pl.bands) return;
    const int sy = t / pl.strips, sx = t - sy * pl.strips;
    // The last strip is moved left to end at xb: it and its neighbour store
    // the same values to the columns they share.
    const int y0 = pl.ya + sy * pl.by, x0 = min(pl.xa + sx * SW, pl.xb - SW);
    stream_strip<R, P, EXACT>(in, filt, out, w, x0, y0, min(pl.by, pl.yb - y0), lane);
}

// ---------------------------------------------------------------- launch

template <int R>
size_t lds_bytes(int passes, int tx, int ty, int q) {
    const int H = R * passes;
    return (size_t)(ty + 2 * H + q - 1) * (tx + 2 * left_of(R, H)) * sizeof(float) * (passes > 1 ? 2 : 1);
}

template <int R, bool EXACT, int TX, int TY, int Q>
hipError_t launch_tiles(const float *in, const float *filt, float *out, int h, int w, int passes, int border,
                        hipStream_t s) {
    const int64_t tiles_x = dev::cdiv(w, TX), n = tiles_x * dev::cdiv(h, TY);
    if (n > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_chain_tiles<R, EXACT, TX, TY, Q>), dim3((unsigned)n), dim3(kThreads),
                       lds_bytes<R>(passes, TX, TY, Q), s, in, filt, out, h, w, passes, border, (int)tiles_x);
    return hipGetLastError();
}

template <int R, int P, bool EXACT>
hipError_t launch_stream(const float *in, const float *filt, float *out, int h, int w, int border,
                         const StreamPlan &pl, hipStream_t s) {
    const int64_t grid = pl.frame + dev::cdiv((int64_t)pl.strips * pl.bands, 4);
    hipLaunchKernelGGL((k_chain_stream<R, P, EXACT>), dim3((unsigned)grid), dim3(kThreads),
                       lds_bytes<R>(P, kFrameX, kFrameY, 2), s, in, filt, out, h, w, border, pl);
    return hipGetLastError();
}

// Passes a stream is built for: its rings fit in registers (at most 192 of
// them; 15 and 16 passes at R = 1 leave some to the accumulation registers). At
// R = 4 the 81 taps no longer fit in scalar registers beside the rest and the
// tiles are as fast.
constexpr int stream_max(int r) { return r == 1 ? 16 : (r == 2 ? 8 : (r == 3 ? 5 : 0)); }

// The least share of useful work at which a stream is ahead of the tiles. Both
// repeat their halo, the tiles more of it the more passes there are; separate
// multiplies and adds weigh more on a stream, which hides less behind them. us,
// stream / tiles, by share: R = 2, 3 passes 0.39 19.8 / 15.9, 0.49 22.9 / 25.3;
// R = 3, 4 passes 0.39 122 / 114, 0.52 86 / 109; exact R = 2, 5 passes 0.56 103 /
// 89, 0.69 152 / 160; exact R = 3, 4 passes 0.52 160 / 132, 0.66 239 / 243;
// R = 1, 12 passes 0.25 38 / 46, exact 50.0 / 50.3; 16 passes 0.34 218 / 196,
// 0.46 114 / 184.
inline double stream_share(int r, bool exact, int passes) {
    constexpr double one[2][8] = {{0.31, 0.29, 0.25, 0.20, 0.20, 0.20, 0.42, 0.42},  // R = 1, from 9 passes
                                   {0.38, 0.37, 0.34, 0.32, 0.30, 0.28, 0.45, 0.45}};
    constexpr double two[2][9] = {{0, 0, 0.56, 0.47, 0.40, 0.34, 0.31, 0.29, 0.28},  // R = 2
                                  {0, 0, 0.90, 0.80, 0.70, 0.62, 0.54, 0.47, 0.42}};
    if (r == 1) return one[exact][passes - 9];
    return two[exact][passes] * (r == 3 ? 1.2 : 1.0);
}

// The stream's plan, or false where the tiles are faster. Bands are as tall
// as one wave per SIMD makes them (a second one per SIMD repeats 2H more halo
// rows per band), but half that where the bands are still at least 8H tall
// and a pixel costs 27 multiply-adds or more: two waves then hide each
// other's waits (4096 x 4096, us, one / two: R = 1, 4 passes 34.0 / 30.1; 8
// passes 58 / 65; 2 passes 23.9 / 26.3, HBM-bound). R = 1 up to 8 passes: from 8
// rows per band (9 rows, 1300 x 1800, 4 passes 12.5 us, tiles 14.8 us). Else by
// the share of the strips' columns and rows that are outputs of one strip alone.
inline bool stream_plan(int r, bool exact, int passes, int h, int w, StreamPlan &pl) {
    if (passes < 2 || passes > stream_max(r)) return false;
    const int H = r * passes, IL = (H + 3) / 4, SW = 4 * (64 - 2 * IL);
    pl.xa = kFrameX, pl.ya = kFrameY;
    pl.xb = w - 4 * IL, pl.yb = h - H;
    if (pl.xb - pl.xa < SW || pl.yb <= pl.ya) return false;
    const int simds = 4 * std::max(dev_info().cus, 1), rows = pl.yb - pl.ya;
    pl.strips = dev::cdiv(pl.xb - pl.xa, SW);
    pl.by = dev::cdiv(rows, std::max(1, simds / pl.strips));
    const double share = (double)(pl.xb - pl.xa) / (256.0 * pl.strips) * pl.by / (pl.by + 2.0 * H);
    if (r == 1 && passes <= 8 ? pl.by < 8 : share < stream_share(r, exact, passes)) return false;
    if (pl.by >= 16 * H && passes * (2 * r + 1) * (2 * r + 1) >= 27)
        pl.by = dev::cdiv(rows, std::max(1, 2 * simds / pl.strips));
    pl.bands = dev::cdiv(rows, pl.by);
    pl.fx = dev::cdiv(w, kFrameX);
    const int64_t frame = (int64_t)pl.fx * (1 + dev::cdiv(h - pl.yb, kFrameY)) +
                          (int64_t)dev::cdiv(rows, kFrameY) * (1 + dev::cdiv(w - pl.xb, kFrameX));
    if (frame + (int64_t)pl.strips * pl.bands > (1 << 23)) return false;  // grid of 2^32 work items
    pl.frame = (int)frame;
    return true;
}

template <int R, bool EXACT, int P = 2>
hipError_t launch_stream_passes(const float *in, const float *filt, float *out, int h, int w, int passes, int border,
                                const StreamPlan &pl, hipStream_t s) {
    if constexpr (P <= stream_max(R)) {
        if (passes == P) return launch_stream<R, P, EXACT>(in, filt, out, h, w, border, pl, s);
        return launch_stream_passes<R, EXACT, P + 1>(in, filt, out, h, w, passes, border, pl, s);
    }
    return hipErrorInvalidValue;
}

// Tiles of 64 x 32; of 64 x 16 while there are at most two per CU, where a
// tile's latency is the launch's time (400 x 600, 8 x (5 x 5): 19.5 us against
// 23.9 us); of 32 x 16 at one per CU at most (257 x 255: 16.8 us against
// 19.4 us). A thread of a 64 x 32 tile takes two rows at a time, but one at R = 2
// and 3 (3 to 6% faster) and at a halo of 16 there and at R = 1, where the spare
// row in LDS costs the third workgroup per CU (R = 1, 16 passes over 4000 x 4000
// 337 us against 376, R = 2, 8 passes over 2160 x 3840 137 against 164).
template <int R, bool EXACT>
hipError_t launch(const float *in, const float *filt, float *out, int h, int w, int passes, int border,
                  hipStream_t s) {
    StreamPlan pl;
    if (stream_plan(R, EXACT, passes, h, w, pl))
        return launch_stream_passes<R, EXACT>(in, filt, out, h, w, passes, border, pl, s);
    const int64_t cus = std::max(dev_info().cus, 1), rows16 = dev::cdiv(h, 16);
    if (dev::cdiv(w, 32) * rows16 <= cus) return launch_tiles<R, EXACT, 32, 16, 1>(in, filt, out, h, w, passes, border, s);
    if (dev::cdiv(w, 64) * rows16 <= 2 * cus) return launch_tiles<R, EXACT, 64, 16, 1>(in, filt, out, h, w, passes, border, s);
    if constexpr (R <= 3)
        if (R > 1 || passes == 16) return launch_tiles<R, EXACT, 64, 32, 1>(in, filt, out, h, w, passes, border, s);
    return launch_tiles<R, EXACT, 64, 32, 2>(in, filt, out, h, w, passes, border, s);
}

}  // namespace chain

template <>
hipError_t launch_chain_radius<PF_R>(bool exact, const float *in, const float *filt, float *out, int h, int w,
                                     int passes, int border, hipStream_t s) {
    return exact ? chain::launch<PF_R, true>(in, filt, out, h, w, passes, border, s)
                 : chain::launch<PF_R, false>(in, filt, out, h, w, passes, border, s);
}

}  // namespace pf

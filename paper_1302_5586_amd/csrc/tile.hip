// FP32 single-image filters on LDS tiles: the full 2D and the separable
// kernel behind pf_filter2d_f32 and pf_filter_sep_f32, one radius (PF_R, set
// by the build) per object.
//
// pf_filter2d_f32_border and one-pass chains run the 2D kernel with their
// border rule.
//
// A 256-thread workgroup owns a tile of 4 CX columns x (256 / CX) Q rows of
// outputs and a thread 4 columns x Q rows of it. The tile's input rows and
// columns with their halo are staged in LDS once, clamped to the image as
// they are loaded, so nothing after the staging knows about borders.
//
//  * 2D: the thread walks the tap rows dy = 0 .. 2R; the Q + 1 window rows it
//    needs sit in registers (a ring: each step reads one new row, as 16-byte
//    LDS vectors, while the arithmetic runs on the others) and so do the tap
//    row in use and the next one (scalar registers, scalar loads one step
//    ahead). Each output takes its taps in the definition's order.
//  * Separable: the row pass over all staged rows into registers, back to
//    LDS in place, then the column pass from there.
//
// What bounds it: the 2D kernel at R >= 4 is bound by FP32 issue (4096 x
// 4096, R = 8: 137 us where (2R+1)^2 multiply-adds take 130 us at the
// measured 37.4 T lane-ops/s), all else by HBM from about 2 M pixels up and
// by the latency of load, barrier, compute, store below that. The strip
// kernel (filter_body.h), which ran these calls before and remains the batch
// kernel, walks 256 columns per wave down the image: on one image that is
// few waves, each a long serial chain, and above R = 4 its 2R + 1 unrolled
// rows outgrow the instruction cache and its taps the scalar registers.
// Measured, strip -> tile, us, buffers rotated through 1 GiB: 256 x 256 R = 1
// 2.9 -> 2.6, R = 4 20.4 -> 3.5; 1080 x 1920 R = 2 13.3 -> 6.5; 1533 x 2047
// R = 6 84 -> 20.5; 4096 x 4096 R = 1 27.6 -> 25.4, R = 2 28.2 -> 26.0, R = 6
// 202 -> 86; separable 4096 x 4096 R = 2 27.6 -> 25.0, R = 6 56 -> 31. From
// the last-level cache (three images reused) 4096 x 4096 R = 2 takes the same
// 23 us on both. The strip won at no size from 64 x 64 to 8192 x 8192.
#include "filter_body.h"

#ifndef PF_R
#error "PF_R must be defined"
#endif

namespace pf {
namespace tile {

using dev::clampi;
using dev::f4u;
using dev::madd;
using dev::static_for;

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = kTileThreads;

// Staged columns left and right of the tile: the radius rounded up to whole
// 16-byte vectors. NB vectors of a staged row hold a thread's window.
constexpr int pad_of(int r) { return 4 * ((r + 3) / 4); }
constexpr int pitch_of(int r, int cx) { return 4 * cx + 2 * pad_of(r); }
constexpr int rows_of(int r, int cx, int q) { return kThreads / cx * q + 2 * r; }
constexpr int window_vecs(int r) { return 1 + pad_of(r) / 2; }

// Stages image rows y0 - R .. and columns x0 - PAD .. into buf, extended past
// the image by the border rule; all of a thread's loads are in flight before
// any is written. Clamping is relative to the tile's origin, so nothing
// overflows at the largest images.
template <int R, int CX, int Q>
__device__ __forceinline__ void stage(const float *__restrict__ in, float *buf, int h, int w, int x0, int y0,
                                      int border) {
    constexpr int PAD = pad_of(R), PITCH = pitch_of(R, CX), ROWS = rows_of(R, CX, Q), CY = kThreads / CX;
    const int right = w - 1 - x0, below = h - 1 - y0;  // >= 0
    if (x0 >= PAD && right >= 4 * CX + PAD - 1 && y0 >= R && below >= CY * Q + R - 1 && w <= (1 << 24)) {
        // Inside the image: thread (cx, cy) takes the vectors of its own
        // columns, every CY-th row, then one of the halo columns. Row steps
        // are scalar, so a load costs no vector address arithmetic (4096 x
        // 4096, R = 2, images reused: 23.2 us, 25.3 us with a division and a
        // clamp per vector).
        constexpr int NP = (ROWS + CY - 1) / CY, HV = PAD / 2, NH = (ROWS * HV + kThreads - 1) / kThreads;
        const int cx = threadIdx.x % CX, cy = threadIdx.x / CX;
        const float *src = in + (int64_t)(y0 - R) * w + (x0 - PAD);
        f4 v[NP], e[NH > 0 ? NH : 1];
        const uint32_t at = (uint32_t)cy * (uint32_t)w + (uint32_t)(PAD + 4 * cx);
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (CY * (u + 1) <= ROWS || cy + CY * u < ROWS)
                v[u] = *reinterpret_cast<const f4u *>(src + (int64_t)u * CY * w + at);
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            const int i = (int)threadIdx.x + u * kThreads, row = i / HV, c = i - row * HV;
            if (i < ROWS * HV)
                e[u] = *reinterpret_cast<const f4u *>(
                    src + ((uint32_t)row * (uint32_t)w + (uint32_t)(4 * (c < HV / 2 ? c : c + CX))));
        }
        float *dst = buf + cy * PITCH + PAD + 4 * cx;
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (CY * (u + 1) <= ROWS || cy + CY * u < ROWS) *reinterpret_cast<f4 *>(dst + u * CY * PITCH) = v[u];
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            const int i = (int)threadIdx.x + u * kThreads, row = i / HV, c = i - row * HV;
            if (i < ROWS * HV) *reinterpret_cast<f4 *>(buf + row * PITCH + 4 * (c < HV / 2 ? c : c + CX)) = e[u];
        }
        return;
    }
    // At the image's edges: vector i of the staged rows, from the nearest 16
    // bytes inside its row, each clamped column picked from them (rows under
    // 4 columns: one load per column).
    constexpr int V = PITCH / 4, N = ROWS * V, NL = (N + kThreads - 1) / kThreads;
    f4 v[NL];
    if (border != PF_BORDER_CLAMP) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int i = min((int)threadIdx.x + u * kThreads, N - 1);
            const int row = i / V, c = 4 * (i - row * V) - PAD;
            const int y = border_index(y0 + row - R, h, border);
            const float *src = in + (int64_t)y * w;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int x = border_index(x0 + c + k, w, border);
                v[u][k] = 0.0f;
                if (x >= 0 && y >= 0) v[u][k] = src[x];
            }
        }
    } else
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        const int i = min((int)threadIdx.x + u * kThreads, N - 1);
        const int row = i / V, c = 4 * (i - row * V) - PAD;
        const float *src = in + (int64_t)(y0 + clampi(row - R, -y0, below)) * w + x0;
        if (w >= 4) {
            const int ca = clampi(c, -x0, right - 3);
            const f4u t = *reinterpret_cast<const f4u *>(src + ca);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[u][k] = dev::pick4(t, clampi(c + k, -x0, right) - ca);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[u][k] = src[clampi(c + k, -x0, right)];
        }
    }
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        const int i = (int)threadIdx.x + u * kThreads;
        if (i < N) reinterpret_cast<f4 *>(buf)[i] = v[u];
    }
}

// A thread's 4 x Q outputs: columns c .. of the tile at x0, rows y .. of the
// tile at y0, those inside the image.
template <int Q>
__device__ __forceinline__ void store_tile(float *__restrict__ out, int h, int w, int x0, int y0, int c, int y,
                                           const float (&acc)[Q][4]) {
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        if (y + j >= h - y0) continue;
        float *o = out + (int64_t)(y0 + y + j) * w + x0 + c;
        if (c + 4 <= w - x0) {
            f4u t;
            t.x = acc[j][0];
            t.y = acc[j][1];
            t.z = acc[j][2];
            t.w = acc[j][3];
            __builtin_nontemporal_store(t, reinterpret_cast<f4u *>(o));
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (c + k < w - x0) __builtin_nontemporal_store(acc[j][k], o + k);
        }
    }
}

template <int R, bool EXACT, int CX, int Q>
__global__ __launch_bounds__(kThreads) void k_tile_2d(const float *__restrict__ in, const float *__restrict__ filt,
                                                      float *__restrict__ out, int h, int w, int tiles_x,
                                                      int border) {
    constexpr int K = 2 * R + 1, PAD = pad_of(R), PITCH = pitch_of(R, CX), NB = window_vecs(R);
    __shared__ __align__(16) float buf[rows_of(R, CX, Q) * PITCH];
    int tx, ty;
    window_tile(blockIdx.x, gridDim.x, tiles_x, tx, ty);
    const int x0 = tx * 4 * CX, y0 = ty * (kThreads / CX) * Q;
    stage<R, CX, Q>(in, buf, h, w, x0, y0, border);
    float wt[2][K];
    load_taps<K>(filt, wt[0]);
    __syncthreads();
    const int cx = threadIdx.x % CX, cy = threadIdx.x / CX;
    int at = Q * cy * PITCH + 4 * cx;
    float acc[Q][4];
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[j][k] = 0.0f;
    float win[Q + 1][4 * NB];  // window row i of the thread at i mod (Q + 1)
#pragma unroll
    for (int j = 0; j < Q; ++j) load_window<NB>(buf + at + j * PITCH, win[j]);
    static_for<0, K>([&](auto dc) __attribute__((always_inline)) {
        constexpr int dy = decltype(dc)::value;
        if constexpr (dy + 1 < K) {
            asm volatile("" : "+v"(at));  // the next window row's load belongs here
            load_taps<K>(filt + (dy + 1) * K, wt[(dy + 1) & 1]);
            load_window<NB>(buf + at + (dy + Q) * PITCH, win[(dy + Q) % (Q + 1)]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int dx = 0; dx < K; ++dx)
#pragma unroll
            for (int j = 0; j < Q; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    acc[j][k] = madd<EXACT>(wt[dy & 1][dx], win[(dy + j) % (Q + 1)][PAD - R + k + dx], acc[j][k]);
        end_step<Q>(acc);
    });
    store_tile<Q>(out, h, w, x0, y0, 4 * cx, Q * cy, acc);
}

template <int R, bool EXACT, int CX, int Q>
__global__ __launch_bounds__(kThreads) void k_tile_sep(const float *__restrict__ in, const float *__restrict__ fx,
                                                       const float *__restrict__ fy, float *__restrict__ out, int h,
                                                       int w, int tiles_x) {
    constexpr int K = 2 * R + 1, PAD = pad_of(R), PITCH = pitch_of(R, CX), NB = window_vecs(R);
    constexpr int ROWS = rows_of(R, CX, Q), CY = kThreads / CX;
    constexpr int NT = (ROWS + CY - 1) / CY;  // staged rows per thread in the row pass
    __shared__ __align__(16) float buf[ROWS * PITCH];
    int tx, ty;
    window_tile(blockIdx.x, gridDim.x, tiles_x, tx, ty);
    const int x0 = tx * 4 * CX, y0 = ty * CY * Q;
    stage<R, CX, Q>(in, buf, h, w, x0, y0, PF_BORDER_CLAMP);
    float wx[K], wy[K];
    load_taps<K>(fx, wx);
    load_taps<K>(fy, wy);
    __syncthreads();
    const int cx = threadIdx.x % CX, cy = threadIdx.x / CX;
    float t[NT][4];
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        float win[4 * NB];
        load_window<NB>(buf + min(cy + CY * u, ROWS - 1) * PITCH + 4 * cx, win);
#pragma unroll
        for (int k = 0; k < 4; ++k) t[u][k] = 0.0f;
#pragma unroll
        for (int dx = 0; dx < K; ++dx)
#pragma unroll
            for (int k = 0; k < 4; ++k) t[u][k] = madd<EXACT>(wx[dx], win[PAD - R + k + dx], t[u][k]);
    }
    __syncthreads();  // every read of the staged rows is done
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        if (cy + CY * u < ROWS) {
            const f4 q = {t[u][0], t[u][1], t[u][2], t[u][3]};
            *reinterpret_cast<f4 *>(buf + (cy + CY * u) * PITCH + 4 * cx) = q;
        }
    }
    __syncthreads();
    float acc[Q][4];
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[j][k] = 0.0f;
    const float *base = buf + Q * cy * PITCH + 4 * cx;
#pragma unroll
    for (int i = 0; i < Q + 2 * R; ++i) {
        const f4 v = *reinterpret_cast<const f4 *>(base + i * PITCH);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const int dy = i - j;
            if (dy < 0 || dy >= K) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[j][k] = madd<EXACT>(wy[dy], v[k], acc[j][k]);
        }
    }
    store_tile<Q>(out, h, w, x0, y0, 4 * cx, Q * cy, acc);
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

// The tile of the FP32 kernels: one workgroup's outputs through LDS, shared by
// the single-image kernels (tile.hip) and the batch kernel (batch_inst.hip).
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
#pragma once

#include "filter_body.h"

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
constexpr int pad_of(int r) { return tile_pad(r); }
constexpr int pitch_of(int r, int cx) { return 4 * cx + 2 * pad_of(r); }
constexpr int rows_of(int r, int cx, int q) { return kThreads / cx * q + 2 * r; }
constexpr int window_vecs(int r) { return 1 + pad_of(r) / 2; }
// Tiles per window of window_tile: 4 million pixels.
constexpr int window_of(int q) { return (1 << 22) / (4 * kThreads * q); }

// Stages image rows y0 - R .. and columns x0 - PAD .. into buf, extended past
// the image by the border rule; all of a thread's loads are in flight before
// any is written. Clamping is relative to the tile's origin, so nothing
// overflows at the largest images.
template <int R, int CX, int Q>
__device__ __forceinline__ void stage(const float *__restrict__ in, float *buf, int h, int w, int x0, int y0,
                                      int border) {
    constexpr int PAD = pad_of(R), PITCH = pitch_of(R, CX), ROWS = rows_of(R, CX, Q), CY = kThreads / CX;
    const int right = w - 1 - x0, below = h - 1 - y0;  // >= 0
    if (tile_inside(R, 4 * CX, CY * Q, x0, y0, h, w)) {
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
    if (border == PF_BORDER_CLAMP && w >= 4 && w <= (1 << 24)) {
        // At the image's edges, the same split: each vector from the nearest
        // 16 bytes inside the nearest row, and where that moved it, each
        // column picked from them. Row by row over all vectors instead, with a
        // division and four picks for each, took 18.9 us against 16.5 us at
        // 2160 x 3840, separable, R = 6, and 23.0 us against 22.0 us at 4096 x
        // 4096, R = 2 (the workgroups at the edges were the last to end).
        constexpr int NP = (ROWS + CY - 1) / CY, HV = PAD / 2, NH = (ROWS * HV + kThreads - 1) / kThreads;
        const int cx = threadIdx.x % CX, cy = threadIdx.x / CX;
        const float *src = in + (int64_t)y0 * w + x0;
        f4 v[NP], e[NH > 0 ? NH : 1];
        const int c = 4 * cx, ca = tile_load_col(c, x0, w);
#pragma unroll
        for (int u = 0; u < NP; ++u)
            v[u] = *reinterpret_cast<const f4u *>(src + (clampi(cy + CY * u - R, -y0, below) * w + ca));
        int ch[NH > 0 ? NH : 1], eh[NH > 0 ? NH : 1];
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            const int i = (int)threadIdx.x + u * kThreads, row = i / HV, k = i - row * HV;
            ch[u] = 4 * (k < HV / 2 ? k : k + CX) - PAD;
            eh[u] = tile_load_col(ch[u], x0, w);
            e[u] = *reinterpret_cast<const f4u *>(src + (clampi(row - R, -y0, below) * w + eh[u]));
        }
        auto pick = [&](f4 &q, int from, int to) __attribute__((always_inline)) {
            const f4u t = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) q[k] = dev::pick4(t, clampi(to + k, -x0, right) - from);
        };
        if (ca != c) {
#pragma unroll
            for (int u = 0; u < NP; ++u) pick(v[u], ca, c);
        }
        float *dst = buf + cy * PITCH + PAD + 4 * cx;
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (CY * (u + 1) <= ROWS || cy + CY * u < ROWS) *reinterpret_cast<f4 *>(dst + u * CY * PITCH) = v[u];
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            const int i = (int)threadIdx.x + u * kThreads, row = i / HV, k = i - row * HV;
            if (eh[u] != ch[u]) pick(e[u], eh[u], ch[u]);
            if (i < ROWS * HV) *reinterpret_cast<f4 *>(buf + row * PITCH + 4 * (k < HV / 2 ? k : k + CX)) = e[u];
        }
        return;
    }
    // The rest (other border rules, rows under 4 columns or over 2^24): vector
    // i of the staged rows, one load per column or, clamped, from the nearest
    // 16 bytes inside its row.
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

// The outputs of the tile at (x0, y0); buf: rows_of * pitch_of floats of LDS.
template <int R, bool EXACT, int CX, int Q>
__device__ __forceinline__ void tile_2d(float *buf, const float *__restrict__ in, const float *__restrict__ filt,
                                        float *__restrict__ out, int h, int w, int x0, int y0, int border) {
    constexpr int K = 2 * R + 1, PAD = pad_of(R), PITCH = pitch_of(R, CX), NB = window_vecs(R);
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
__device__ __forceinline__ void tile_sep(float *buf, const float *__restrict__ in, const float *__restrict__ fx,
                                         const float *__restrict__ fy, float *__restrict__ out, int h, int w, int x0,
                                         int y0) {
    constexpr int K = 2 * R + 1, PAD = pad_of(R), PITCH = pitch_of(R, CX), NB = window_vecs(R);
    constexpr int ROWS = rows_of(R, CX, Q), CY = kThreads / CX;
    constexpr int NT = (ROWS + CY - 1) / CY;  // staged rows per thread in the row pass
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

}  // namespace tile
}  // namespace pf

// Device helpers shared by the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pf.h"

namespace pf {

// MI355X deals the workgroups of a launch round-robin over its 8 XCDs
// (workgroup b runs on XCD b mod 8), and each XCD has its own L2. The
// remap gives the workgroups of one XCD consecutive logical ids, so tiles
// with neighbouring logical ids (which share halo rows and cache lines)
// meet in the same L2. b: hardware workgroup id; g: workgroups in the grid.
__device__ __forceinline__ int xcd_remap(int b, int g) {
    const int xcd = b & 7, idx = b >> 3;
    const int per = g >> 3, rem = g & 7;
    return xcd * per + min(xcd, rem) + idx;
}

// Workgroup -> tile of a list (an image's tiles row by row, tiles_x per row).
// The launch is taken in windows of about `window` tiles: the tiles in flight
// cover one compact band that advances down the image, and inside a window
// each XCD has a contiguous eighth, so that most of a tile's neighbours are
// in the same L2. Measured on the FP32 tile kernel: one contiguous eighth of
// the whole image per XCD keeps eight windows of HBM pages open: 30.0 us
// against 27.5 us at 4096 x 4096, R = 2 (buffers rotated through 2 GiB; 26 us
// against 25.2 us where three images are reused and partly in the last-level
// cache). Dealt in groups of 32 tiles instead, halo rows cross XCDs: 14.5 us
// against 13.7 us at 2160 x 3840 from that cache. About 4 million pixels per
// window serve single images best (separable 4096 x 4096, R = 2, tiles of 128
// x 32, from HBM: 27.4 us with 1024 tiles, 28.8 with 2048; from the cache
// 22.1 and 22.3; 512 tiles 27.3 and 22.8).
__device__ __forceinline__ void window_tile(int b, int n, int tiles_x, int window, int &tx, int &ty) {
    const int windows = max(1, (n + window / 2) / window);
    const int size = ((n + windows - 1) / windows + 7) / 8 * 8;  // a multiple of 8: workgroup b runs on XCD b mod 8
    const int first = b / size * size;
    const int t = first + xcd_remap(b - first, min(size, n - first));
    ty = t / tiles_x;
    tx = t - ty * tiles_x;
}

// Source index of position i of an axis of n elements under a border rule
// (PF_BORDER_*); -1 where the rule reads a zero.
__device__ __forceinline__ int border_index(int i, int n, int border) {
    if (i >= 0 && i < n) return i;
    if (border == PF_BORDER_CLAMP) return i < 0 ? 0 : n - 1;
    if (border == PF_BORDER_ZERO) return -1;
    if (n == 1) return 0;
    // reflect (edge repeated, period 2n): d c b a | a b c d | d c b a; mirror
    // (edge not repeated, period 2n - 2): d c b | a b c d | c b a. One fold
    // suffices within n of the image; further out the index wraps with the
    // period first.
    const int edge = border == PF_BORDER_REFLECT ? 1 : 0;
    const int p = 2 * n - 2 + 2 * edge;
    if (i <= -n || i >= 2 * n - 1) {
        i %= p;
        if (i < 0) i += p;
        return i < n ? i : p - edge - i;
    }
    return i < 0 ? -i - edge : p - edge - i;
}

// N taps through the scalar cache. The address is opaque to the compiler
// here, so that taps are loaded where they are asked for: hoisted to a
// kernel's start, the taps of a wide filter spill.
template <int N>
__device__ __forceinline__ void load_taps(const float *p, float (&t)[N]) {
    typedef __attribute__((address_space(4))) const float cfloat;
    uint64_t a = (uint64_t)p;
    asm volatile("" : "+s"(a));
    const cfloat *c = (const cfloat *)a;
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = c[i];
}

// NB 16-byte LDS vectors from p as 4 NB floats.
template <int NB>
__device__ __forceinline__ void load_window(const float *p, float (&t)[4 * NB]) {
    typedef float f4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const f4 q = *reinterpret_cast<const f4 *>(p + 4 * b);
        t[4 * b] = q.x;
        t[4 * b + 1] = q.y;
        t[4 * b + 2] = q.z;
        t[4 * b + 3] = q.w;
    }
}

// Ends a step of a thread's Q x 4 accumulators: their updates stay before
// the loads of later steps (left to itself the compiler moves those loads up
// and keeps every window row alive at once).
template <int Q>
__device__ __forceinline__ void end_step(float (&acc)[Q][4]) {
#pragma unroll
    for (int j = 0; j < Q; ++j) asm volatile("" : "+v"(acc[j][0]), "+v"(acc[j][1]), "+v"(acc[j][2]), "+v"(acc[j][3]));
    __builtin_amdgcn_sched_barrier(0);
}

// A device address held as an integer (a descriptor field), as a pointer
// into global memory: cast through the global address space so that the
// compiler emits global accesses rather than flat ones.
template <class T>
__device__ __forceinline__ T *global_ptr(int64_t addr) {
    typedef __attribute__((address_space(1))) T gT;
    return (T *)(gT *)(uintptr_t)addr;
}

}  // namespace pf

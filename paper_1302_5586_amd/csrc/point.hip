// FP32 calls of radius 0: every output is its own pixel times one weight per
// pass (a separable call has two passes, fx then fy), whatever the image's
// shape and border rule, so the image is one array.
//
// Bound by HBM, and by the launch below about a million pixels. On tiles, as a
// filter of any other radius, a chain's passes went through LDS (3 passes over
// 2000 x 2000: 31.6 us, now 10.5 us; over 20000 x 400 56 us, now 11.8 us) and
// images thinner than a tile were computed with its padding (1 x 2^23 38 us,
// now 10.7 us; 2^22 x 1 400 us, now 6.5 us). Buffers reused; 100000 x 200
// 26.4 us, now 25.6 us.
#include "filter_body.h"

namespace pf {
namespace point {

using dev::f4u;
using dev::madd;

constexpr int kThreads = 256;
constexpr int kVecs = 4;  // 16-byte vectors per thread, all in flight at once

template <bool EXACT>
__device__ __forceinline__ float apply(float v, float a, float b, int passes, bool two) {
    for (int p = 0; p < passes; ++p) v = madd<EXACT>(a, v, 0.0f);
    return two ? madd<EXACT>(b, v, 0.0f) : v;
}

// out[i] = in[i] after `passes` passes with weight *fa, then one with *fb if
// there is one. Rows need only 4-byte alignment.
template <bool EXACT>
__global__ __launch_bounds__(kThreads) void k_point(const float *__restrict__ in, const float *__restrict__ fa,
                                                    const float *__restrict__ fb, float *__restrict__ out, int64_t n,
                                                    int passes) {
    const bool two = fb != nullptr;
    const float a = fa[0], b = two ? fb[0] : 0.0f;
    const int64_t nv = n / 4, first = (int64_t)blockIdx.x * kThreads * kVecs + threadIdx.x;
    f4u v[kVecs];
#pragma unroll
    for (int u = 0; u < kVecs; ++u)
        if (first + u * kThreads < nv) v[u] = *reinterpret_cast<const f4u *>(in + 4 * (first + u * kThreads));
#pragma unroll
    for (int u = 0; u < kVecs; ++u) {
        if (first + u * kThreads >= nv) continue;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[u][k] = apply<EXACT>(v[u][k], a, b, passes, two);
        __builtin_nontemporal_store(v[u], reinterpret_cast<f4u *>(out + 4 * (first + u * kThreads)));
    }
    // The last n mod 4 elements.
    if (blockIdx.x == 0 && (int64_t)threadIdx.x < n - 4 * nv) {
        const int64_t i = 4 * nv + threadIdx.x;
        out[i] = apply<EXACT>(in[i], a, b, passes, two);
    }
}

}  // namespace point

hipError_t launch_point(bool exact, const float *in, const float *fa, const float *fb, float *out, int64_t n,
                        int passes, hipStream_t s) {
    constexpr int64_t per = 4 * point::kThreads * point::kVecs;  // n < 2^31: at most 2^19 workgroups
    hipLaunchKernelGGL(exact ? point::k_point<true> : point::k_point<false>, dim3((unsigned)((n + per - 1) / per)),
                       dim3(point::kThreads), 0, s, in, fa, fb, out, n, passes);
    return hipGetLastError();
}

}  // namespace pf

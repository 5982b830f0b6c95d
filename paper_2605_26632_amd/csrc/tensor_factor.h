// TENSOR scope: the single compensation factor of an activation from its rows' sums of squares. One device function
// for the kernel that only does this and for the tile loops that fold it into their start, so that both form
// the same bits: fp64 sums in a fixed order.
#pragma once
#include "rtl_internal.h"

namespace rtl {
namespace {

constexpr int kFactorThreads = 256;      // threads that add rows up; further threads of the workgroup only take the result

// Called by every thread of a workgroup of at least kFactorThreads; contains barriers. rowsums [M][2]: |x|^2 of
// the row, |kept|^2 of the row. Bound by the latency of its loads (eight in flight per thread).
__device__ __forceinline__ float tensor_factor(const float* __restrict__ rowsums, int64_t M, float eps) {
    __shared__ double part[2][kFactorThreads / 64];
    const int tid = threadIdx.x;
    if (tid < kFactorThreads) {
        double n = 0.0, d = 0.0;
        const float2* rs = reinterpret_cast<const float2*>(rowsums);
        int64_t r = tid;
        for (; r + 7 * kFactorThreads < M; r += 8 * kFactorThreads) {
            float2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = rs[r + u * kFactorThreads];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                n += (double)v[u].x;
                d += (double)v[u].y;
            }
        }
        if (r < M) {                                     // at most eight more, absent ones add zero
            float2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t q = r + u * kFactorThreads;
                v[u] = rs[q < M ? q : r];
                if (q >= M) v[u] = make_float2(0.f, 0.f);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                n += (double)v[u].x;
                d += (double)v[u].y;
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            n += __shfl_xor(n, off, 64);
            d += __shfl_xor(d, off, 64);
        }
        if ((tid & 63) == 0) {
            part[0][tid >> 6] = n;
            part[1][tid >> 6] = d;
        }
    }
    __syncthreads();
    double n = part[0][0], d = part[1][0];
#pragma unroll
    for (int w = 1; w < kFactorThreads / 64; ++w) {
        n += part[0][w];
        d += part[1][w];
    }
    __syncthreads();
    return (float)sqrt(n / (d + (double)eps));
}

}  // namespace
}  // namespace rtl

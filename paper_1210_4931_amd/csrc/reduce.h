// Sums of per-block partials, the last step of every diagnostic: one workgroup of kSumT threads
// per result, each thread adding a strided share in order, then a tree in LDS (a fixed order,
// so results repeat bit for bit).  What bounds them is latency: one thread walking all the
// partials waited for each load in turn (nside 512: 55 us a pixel sum of 1024 partials, 112 us the
// three harmonic sums over m, 465 us for 64 maps, where these take 2.4, 5 and 5 us).
#pragma once

#include "mfwf_internal.h"

namespace mfwf {

static constexpr int kSumT = 256;

// out[k] = sum over i < n of p[K i + k], in thread 0
template <int K>
__device__ __forceinline__ void sum_strided(const double *__restrict__ p, int n, double (&out)[K]) {
    __shared__ double sh[K][kSumT];
#pragma unroll
    for (int k = 0; k < K; k++) out[k] = 0.0;
    for (int i = threadIdx.x; i < n; i += kSumT)
#pragma unroll
        for (int k = 0; k < K; k++) out[k] += p[(long)K * i + k];
#pragma unroll
    for (int k = 0; k < K; k++) sh[k][threadIdx.x] = out[k];
    __syncthreads();
    for (int w = kSumT / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
#pragma unroll
            for (int k = 0; k < K; k++) sh[k][threadIdx.x] += sh[k][threadIdx.x + w];
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < K; k++) out[k] = sh[k][0];
}

}  // namespace mfwf

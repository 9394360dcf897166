// What the kernels of the log-likelihood share: a workgroup's sum in a fixed tree, and the term of a
// count.
#pragma once

#include "common.hpp"

namespace lda {

__device__ __forceinline__ double block_sum_f64(double v, double* wtot)
{
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
    const int nw = (blockDim.x + kWave - 1) >> 6;
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    __syncthreads();
    if (lane == 0) wtot[wv] = v;
    __syncthreads();
    double s = 0.0;
    for (int i = 0; i < nw; ++i) s += wtot[i];
    return s;
}

// The terms of counts below kTermTable, by count: lgG(v + a) - lgG(a).  They depend on the
// context's alpha and beta alone and are made once, by the same fp64 expression that larger
// counts are computed with, so a sum does not depend on where a term comes from.  Nearly every
// count is small, and lgamma is some 200 fp64 instructions that a wave runs if any of its lanes
// needs it.
constexpr int32_t kTermTable = 4096;

__device__ __forceinline__ double count_term(int32_t v, double a, double lg_a, const double* __restrict__ table)
{
    return v < kTermTable ? table[v] : lgamma((double)v + a) - lg_a;
}

}  // namespace lda

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

// acc plus the terms of U counts, zero where there is none.  The look-ups are all in flight together; a
// test for each of them made them wait for one another (10^8 counts, a fifth of them not zero, 339 us).
template <int U>
__device__ __forceinline__ double add_terms(double acc, const int32_t (&v)[U], double a, double lg_a,
                                            const double* __restrict__ table)
{
    double t[U];
    bool large = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        t[u] = table[v[u] < kTermTable ? v[u] : 0];
        large = large || v[u] >= kTermTable;
    }
    if (__any(large)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (v[u] >= kTermTable) t[u] = lgamma((double)v[u] + a) - lg_a;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc += v[u] > 0 ? t[u] : 0.0;
    return acc;
}

// A wave's terms of the counts [k0, k1) of a dense row, lane by lane, eight loads in flight.  AHEAD: the next
// eight while the terms of eight are looked up.
// (30 000 rows of 16 000 counts, lists kernel: 810 us without and pieces of 2048 counts, 754 with, 727 with pieces
// of 4096.  The implied kernel, whose rows are few and workgroups large: 102 us without, 109 with.)
template <bool AHEAD>
__device__ __forceinline__ double row_terms(const int32_t* __restrict__ row, int32_t k0, int32_t k1, double beta,
                                            double lg_beta, const double* __restrict__ terms)
{
    const int lane = threadIdx.x & (kWave - 1);
    double acc = 0.0;
    auto load = [&](int32_t kb, int32_t (&v)[8]) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int32_t k = kb + u * kWave + lane;
            v[u] = k < k1 ? row[k] : 0;
        }
    };
    int32_t v[8], next[8];
    if constexpr (AHEAD) load(k0, next);
    for (int32_t kb = k0; kb < k1; kb += 8 * kWave) {
        if constexpr (AHEAD) {
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = next[u];
            load(kb + 8 * kWave, next);
        } else {
            load(kb, v);
        }
        acc = add_terms<8>(acc, v, beta, lg_beta, terms);
    }
    return acc;
}

}  // namespace lda

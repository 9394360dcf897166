// The alias table (LightLDA Sec. 4.2, Fig. 2) and what its two builders share.
//
// The table is defined on integers so that a parallel build is exact.  Given the
// quantised weights q0_i = floor(weight_i * 2^40) of n entries:
//   Q0 = sum q0_i,  sh = smallest shift with (Q0 >> sh) < n * 2^31
//   q_i = max(1, q0_i >> sh), Q = sum q_i, C = ceil(Q / n), pad = n*C - Q
//   m_i = q_i + (i < pad)                                    (sum m_i = n*C)
// Entries with m_i < C ("lights", ascending i, exclusive deficit sums Delta_a) are
// topped up by entries with m_i >= C ("heavies", ascending i, inclusive excess sums
// X_b).  Pairing the two ascending lists greedily has the closed form
//   light a : split = m,  alias = heavy b with b = min{b : X_b > Delta_a}
//   heavy b : a = min{a : Delta_a >= X_b}, split = C + X_b - Delta_a,
//             alias = next heavy if split < C, else itself
// so the build is prefix sums over the two lists and a merge of them (alias_regs.hpp: tables
// whose lists fit one workgroup's LDS) or bounded searches (alias_split.hpp: larger tables,
// many workgroups each).
//
// An Io describes one kind of table to both: Raw load(k) and void load2(Raw&) fetch what entry
// k's weight comes from, q0(Raw) is the weight, Loaded load(k, alias, raw) gathers what the
// entry's output needs and store(k, split, alias, raw, loaded) writes it, once per entry.
// kListed: the entries are those of a list among n that differ from each other little: mass(k) is
// entry k's weight if it is not in the list, patch(weights, thread, threads) writes those in it, Q0()
// and Q() are the sums known beforehand; load() reads an array of n ints in LDS, made by
// clear(array, n, thread, threads) and fill(array, thread, threads), and is called late.
// kMassesFirst: see alias_regs.hpp, build_table_workgroup.
#pragma once

#include "common.hpp"

namespace lda {

constexpr int kMaxWaves = 16;

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v)
{
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)v, d, kWave);
        const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), d, kWave);
        v += ((uint64_t)hi << 32) | lo;
    }
    return v;
}

// Inclusive prefix sum over the 64 lanes with DPP row shifts and row broadcasts
// (no LDS traffic): shifts by 1, 2, 3 of the input, then 4 and 8 inside each row of
// 16 lanes, then the last lane of row 0 / 2 into row 1 / 3 and lane 31 into rows 2, 3.
__device__ __forceinline__ uint32_t wave_inclusive_scan_u32(uint32_t v)
{
    const int x = (int)v;
    int r = x;
    r += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    r += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    r += __builtin_amdgcn_update_dpp(0, x, 0x113, 0xf, 0xf, false);  // row_shr:3
    r += __builtin_amdgcn_update_dpp(0, r, 0x114, 0xf, 0xe, false);  // row_shr:4, lanes 4..15
    r += __builtin_amdgcn_update_dpp(0, r, 0x118, 0xf, 0xc, false);  // row_shr:8, lanes 8..15
    r += __builtin_amdgcn_update_dpp(0, r, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1, 3
    r += __builtin_amdgcn_update_dpp(0, r, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2, 3
    return (uint32_t)r;
}

// 64-bit inclusive prefix sum of values < 2^46: the low 26 bits and the rest are
// summed separately (64 terms cannot overflow 32 bits) and recombined.
__device__ __forceinline__ uint64_t wave_inclusive_scan_u64(uint64_t v)
{
    const uint32_t lo = wave_inclusive_scan_u32((uint32_t)v & 0x3FFFFFFu);
    const uint32_t hi = wave_inclusive_scan_u32((uint32_t)(v >> 26));
    return ((uint64_t)hi << 26) + (uint64_t)lo;
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane)
{
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// First index in [lo, hi] at which the monotone predicate holds; pred(hi) is known
// to hold.  lo, hi are wave-uniform and all 64 lanes take part: a window of 64
// consecutive indices first (partners of neighbouring bins are close), then 64-ary
// narrowing of what is left.
template <class Pred>
__device__ __forceinline__ uint32_t wave_first_true(uint32_t lo, uint32_t hi, int lane, Pred pred)
{
    {
        const uint32_t top = (hi - lo > 63u) ? lo + 63u : hi;
        uint32_t idx = lo + (uint32_t)lane;
        if (idx > top) idx = top;
        const uint64_t mask = __ballot(pred(idx));
        if (mask != 0) return lo + (uint32_t)(__ffsll((unsigned long long)mask) - 1);
        lo = top + 1;  // top < hi here, because pred(hi) holds
    }
    for (;;) {
        const uint32_t step = (hi - lo) / 63u + 1u;
        uint32_t idx = lo + (uint32_t)lane * step;
        if (idx > hi) idx = hi;
        const uint64_t mask = __ballot(pred(idx));  // lane 63 sits on hi: never empty
        const uint32_t f = (uint32_t)(__ffsll((unsigned long long)mask) - 1);
        const uint32_t cand = lo + f * step;
        if (step == 1u) return cand < hi ? cand : hi;
        hi = cand < hi ? cand : hi;
        if (f > 0) lo = lo + (f - 1u) * step + 1u;
    }
}

// number of set bits of `mask` below this lane
__device__ __forceinline__ uint32_t rank_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

}  // namespace lda

// Alias-table builder for tables too large for one workgroup's LDS (LightLDA Sec. 4.2, Fig. 2):
// the table alias_build.hpp defines, built by as many workgroups as it has chunks of
// kBigChunk entries, in five launches over all chunks of all tables:
//
//   big_mass     sum of the quantised weights q0 per chunk
//   big_shift    the shift from the table's sum; per chunk the sum of the shifted weights
//   big_counts   C and pad; per chunk the number of lights, their deficit, the heavies' excess
//   big_lists    the two ascending lists with their running sums, in global memory
//   big_pairs    every entry's partner, and the output in entry order
//
// Each launch starts from per-chunk sums the one before it wrote (a workgroup adds up those of
// its own table: at most 2^20 / kBigChunk = 512).  The weights are computed anew in every launch
// instead of stored: the counts they come from are 4 to 12 bytes of streaming reads per entry.
//
// Pairing: the partners of a chunk's lights are a contiguous run of heavies and the other way
// round (both lists ascend).  Four waves find the four ends of the two runs by 64-way searches,
// the runs are copied to LDS, and every lane bisects there, all its entries in step.
//
// What bounds it: the five passes over the entries (about 80 bytes read and written per entry
// all told).  The form it replaced gave a table to one workgroup, four passes with the
// lists in memory: a table of 10^6 entries took 5.5 to 10 ms whatever else the chip did.  Whole
// iterations: K = 10^6 with 10^8 tokens 23.5 -> 16.3 ms, the same streamed with 4 * 10^7 tokens
// 26.5 -> 17.5 ms, K = 10^5 with 1.5 * 10^8 tokens 19.0 -> 18.5 ms.
#pragma once

#include "alias_build.hpp"

namespace lda {

constexpr int kBigE = 8;                        // entries per thread
constexpr int kBigThreads = 256;
constexpr int kBigWaves = kBigThreads / kWave;
constexpr int32_t kBigChunk = kBigE * kBigThreads;
constexpr int32_t kBigWindow = 2 * kBigChunk;   // list entries kept in LDS while pairing: 32 KB

// What every kernel below gets: where the chunks, the per-chunk sums and the lists are.
struct BigWork {
    const int2* chunks;      // (table, first entry) of chunk c
    const uint32_t* first;   // first chunk of table t
    const uint64_t* list;    // first list entry of table t in dx and hidx
    BigSums* sums;           // per chunk
    BigState* state;         // per table
    uint64_t* dx;            // of table t, n + 1 entries: [0..A] Delta_a, [n - b] X_b
    uint32_t* hidx;          // [b] entry of heavy b
    uint32_t c0;             // first chunk of the launch
};

// The chunk of a workgroup and the entries of its lanes: wave v holds the contiguous entries
// [k0 + v * 64 E, ...), lane l of it the entries l, l + 64, ...
template <class Tables>
struct BigChunkView {
    uint32_t c;       // chunk
    int32_t t, k0;    // table, first entry of the chunk
    int32_t n;        // entries of the table
    int32_t kw;       // first entry of the wave
    int lane, wv;
    __device__ __forceinline__ BigChunkView(const Tables& tab, const BigWork& W)
    {
        c = W.c0 + blockIdx.x;
        const int2 ch = W.chunks[c];
        t = ch.x;
        k0 = ch.y;
        n = tab.entries(t);
        lane = threadIdx.x & (kWave - 1);
        wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        kw = k0 + wv * (kBigE * kWave);
    }
    __device__ __forceinline__ int32_t entry(int e) const { return kw + e * kWave + lane; }
    __device__ __forceinline__ uint32_t table_chunks() const { return (uint32_t)((n + kBigChunk - 1) / kBigChunk); }
};

template <class Io>
__device__ __forceinline__ void big_load(const Io& io, int32_t kw, int lane, int32_t n,
                                         typename Io::Raw (&raw)[kBigE])
{
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        const int32_t k = kw + e * kWave + lane;
        raw[e] = io.load(k < n ? k : n - 1);
    }
#pragma unroll
    for (int e = 0; e < kBigE; ++e) io.load2(raw[e]);
}

// sum over the workgroup (every thread gets it); two barriers
__device__ __forceinline__ uint64_t big_block_sum(uint64_t v, uint64_t* buf)
{
    v = wave_sum_u64(v);
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) buf[threadIdx.x >> 6] = v;
    __syncthreads();
    uint64_t s = 0;
#pragma unroll
    for (int i = 0; i < kBigWaves; ++i) s += buf[i];
    return s;
}

template <class Tables>
__global__ __launch_bounds__(kBigThreads) void big_mass_kernel(Tables tab, BigWork W)
{
    __shared__ uint64_t buf[kBigWaves];
    const BigChunkView<Tables> v(tab, W);
    if (v.k0 >= v.n) return;  // uniform: the table has fewer entries than it may have
    const auto io = tab.io(v.t);
    typename decltype(tab.io(0))::Raw raw[kBigE];
    big_load(io, v.kw, v.lane, v.n, raw);
    uint64_t p0 = 0, p1 = 0;
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        const uint64_t q = io.q0(raw[e]);
        if (v.entry(e) < v.n) {
            p0 += q;
            p1 += q < 1 ? 1 : q;
        }
    }
    p0 = big_block_sum(p0, buf);
    p1 = big_block_sum(p1, buf);
    if (threadIdx.x == 0) {
        W.sums[v.c].q0 = p0;
        W.sums[v.c].q = p1;  // of no shift; big_shift replaces it if there is one
    }
}

template <class Tables>
__global__ __launch_bounds__(kBigThreads) void big_shift_kernel(Tables tab, BigWork W)
{
    __shared__ uint64_t buf[kBigWaves];
    const BigChunkView<Tables> v(tab, W);
    if (v.k0 >= v.n) return;
    const uint32_t c_first = W.first[v.t];
    uint64_t Q0 = 0;
    for (uint32_t i = threadIdx.x; i < v.table_chunks(); i += kBigThreads) Q0 += W.sums[c_first + i].q0;
    Q0 = big_block_sum(Q0, buf);
    int sh = 0;
    while ((Q0 >> sh) >= ((uint64_t)v.n << 31)) ++sh;
    if (v.k0 == 0 && threadIdx.x == 0) {
        W.state[v.t].Q0 = Q0;
        W.state[v.t].sh = (uint32_t)sh;
    }
    if (sh == 0) return;  // uniform
    const auto io = tab.io(v.t);
    typename decltype(tab.io(0))::Raw raw[kBigE];
    big_load(io, v.kw, v.lane, v.n, raw);
    uint64_t p1 = 0;
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        const uint64_t q = io.q0(raw[e]) >> sh;
        if (v.entry(e) < v.n) p1 += q < 1 ? 1 : q;
    }
    p1 = big_block_sum(p1, buf);
    if (threadIdx.x == 0) W.sums[v.c].q = p1;
}

// m of the lane's entries (entries past the end: C, neither light nor counted)
template <class Io>
__device__ __forceinline__ void big_masses(const Io& io, const typename Io::Raw (&raw)[kBigE], int32_t kw,
                                           int lane, int32_t n, uint32_t sh, uint64_t C, uint64_t pad,
                                           uint64_t (&m)[kBigE])
{
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        const int32_t k = kw + e * kWave + lane;
        uint64_t q = io.q0(raw[e]) >> sh;
        if (q < 1) q = 1;
        if ((uint64_t)k < pad) q += 1;
        m[e] = k < n ? q : C;
    }
}

template <class Tables>
__global__ __launch_bounds__(kBigThreads) void big_counts_kernel(Tables tab, BigWork W)
{
    __shared__ uint64_t buf[kBigWaves];
    const BigChunkView<Tables> v(tab, W);
    if (v.k0 >= v.n) return;
    const auto io = tab.io(v.t);
    typename decltype(tab.io(0))::Raw raw[kBigE];
    big_load(io, v.kw, v.lane, v.n, raw);
    const uint32_t c_first = W.first[v.t];
    uint64_t Q = 0;
    for (uint32_t i = threadIdx.x; i < v.table_chunks(); i += kBigThreads) Q += W.sums[c_first + i].q;
    Q = big_block_sum(Q, buf);
    // ceil(Q / n) through fp64: exact, see build_table_regs
    const uint64_t C = (uint64_t)((double)(Q + (uint64_t)v.n - 1) / (double)v.n);
    const uint64_t pad = (uint64_t)v.n * C - Q;
    uint64_t m[kBigE];
    big_masses(io, raw, v.kw, v.lane, v.n, W.state[v.t].sh, C, pad, m);
    uint64_t lc = 0, df = 0, ex = 0;
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        if (m[e] < C) { lc += 1; df += C - m[e]; } else ex += m[e] - C;
    }
    lc = big_block_sum(lc, buf);
    df = big_block_sum(df, buf);
    ex = big_block_sum(ex, buf);
    if (threadIdx.x == 0) {
        W.sums[v.c].df = df;
        W.sums[v.c].ex = ex;
        W.sums[v.c].lights = (uint32_t)lc;
        if (v.k0 == 0) {
            W.state[v.t].C = C;
            W.state[v.t].pad = pad;
        }
    }
}

template <class Tables>
__global__ __launch_bounds__(kBigThreads) void big_lists_kernel(Tables tab, BigWork W)
{
    __shared__ uint64_t buf[kBigWaves], w_df[kBigWaves], w_ex[kBigWaves];
    __shared__ uint32_t w_lc[kBigWaves];
    const BigChunkView<Tables> v(tab, W);
    if (v.k0 >= v.n) {
        // a table without entries is never drawn from
        if (v.k0 == 0 && threadIdx.x == 0) tab.done(v.t, 0, 0, 0);
        return;
    }
    const auto io = tab.io(v.t);
    typename decltype(tab.io(0))::Raw raw[kBigE];
    big_load(io, v.kw, v.lane, v.n, raw);
    // lights, deficit and excess of the chunks before this one; lights and deficit of all
    const uint32_t c_first = W.first[v.t], mine = v.c - c_first;
    uint64_t lights = 0, a_before = 0, d_tot = 0, d_before = 0, x_before = 0;
    for (uint32_t i = threadIdx.x; i < v.table_chunks(); i += kBigThreads) {
        const BigSums s = W.sums[c_first + i];
        lights += s.lights;
        d_tot += s.df;
        if (i < mine) { a_before += s.lights; d_before += s.df; x_before += s.ex; }
    }
    lights = big_block_sum(lights, buf);
    d_tot = big_block_sum(d_tot, buf);
    a_before = big_block_sum(a_before, buf);
    d_before = big_block_sum(d_before, buf);
    x_before = big_block_sum(x_before, buf);
    const BigState st = W.state[v.t];
    const uint64_t C = st.C;
    uint64_t* __restrict__ dx = W.dx + W.list[v.t];
    uint32_t* __restrict__ hidx = W.hidx + W.list[v.t];
    if (threadIdx.x == 0) {
        W.sums[v.c].a_before = (uint32_t)a_before;
        if (v.k0 == 0) {
            W.state[v.t].A = (uint32_t)lights;
            dx[lights] = d_tot;
            tab.done(v.t, v.n, st.Q0, (uint32_t)C);
        }
    }
    uint64_t m[kBigE];
    big_masses(io, raw, v.kw, v.lane, v.n, st.sh, C, st.pad, m);
    uint32_t lc = 0;
    uint64_t df = 0, ex = 0;
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        lc += (uint32_t)__popcll(__ballot(m[e] < C));
        if (m[e] < C) df += C - m[e]; else ex += m[e] - C;
    }
    df = wave_sum_u64(df);
    ex = wave_sum_u64(ex);
    if (v.lane == 0) { w_lc[v.wv] = lc; w_df[v.wv] = df; w_ex[v.wv] = ex; }
    __syncthreads();
    uint32_t a_run = (uint32_t)a_before;
    uint64_t d_run = d_before, x_run = x_before;
    for (int i = 0; i < v.wv; ++i) { a_run += w_lc[i]; d_run += w_df[i]; x_run += w_ex[i]; }
    uint32_t b_run = (uint32_t)(v.kw < v.n ? v.kw : v.n) - a_run;
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        const int32_t k = v.entry(e);
        const bool light = m[e] < C, heavy = k < v.n && !light;
        const uint64_t lmask = __ballot(light), hmask = __ballot(heavy);
        const uint32_t la = rank_below(lmask);
        const uint64_t dinc = wave_inclusive_scan_u64(light ? C - m[e] : 0ull);
        const uint64_t xinc = wave_inclusive_scan_u64(heavy ? m[e] - C : 0ull);
        if (light) dx[a_run + la] = d_run + dinc - (C - m[e]);
        if (heavy) {
            const uint32_t b = b_run + rank_below(hmask);
            dx[(uint32_t)v.n - b] = x_run + xinc;
            hidx[b] = (uint32_t)k;
        }
        d_run += readlane_u64(dinc, kWave - 1);
        x_run += readlane_u64(xinc, kWave - 1);
        a_run += (uint32_t)__popcll(lmask);
        b_run += (uint32_t)__popcll(hmask);
    }
}

template <class Tables>
__global__ __launch_bounds__(kBigThreads) void big_pairs_kernel(Tables tab, BigWork W)
{
    __shared__ uint64_t win[kBigWindow];
    __shared__ uint32_t w_lc[kBigWaves], ends[4];
    const BigChunkView<Tables> v(tab, W);
    if (v.k0 >= v.n) return;
    const auto io = tab.io(v.t);
    using Io = decltype(tab.io(0));
    typename Io::Raw raw[kBigE];
    big_load(io, v.kw, v.lane, v.n, raw);
    const BigState st = W.state[v.t];
    const uint64_t C = st.C;
    const uint32_t n = (uint32_t)v.n, A = st.A, B = n - A;
    const uint64_t* __restrict__ dx = W.dx + W.list[v.t];
    const uint32_t* __restrict__ hidx = W.hidx + W.list[v.t];
    uint64_t m[kBigE];
    big_masses(io, raw, v.kw, v.lane, v.n, st.sh, C, st.pad, m);
    uint32_t lc = 0;
#pragma unroll
    for (int e = 0; e < kBigE; ++e) lc += (uint32_t)__popcll(__ballot(m[e] < C));
    if (v.lane == 0) w_lc[v.wv] = lc;
    __syncthreads();
    const uint32_t a0 = W.sums[v.c].a_before, b0 = (uint32_t)v.k0 - a0;  // the chunk's first light, heavy
    uint32_t a_run = a0, lights = 0;
#pragma unroll
    for (int i = 0; i < kBigWaves; ++i) {
        if (i < v.wv) a_run += w_lc[i];
        lights += w_lc[i];
    }
    const uint32_t here = n - (uint32_t)v.k0 < (uint32_t)kBigChunk ? n - (uint32_t)v.k0 : (uint32_t)kBigChunk;
    const uint32_t heavies = here - lights;
    uint32_t b_run = (uint32_t)(v.kw < v.n ? v.kw : v.n) - a_run;
    // ends[0..1]: heavies that the first and the last light of the chunk alias to;
    // ends[2..3]: lights at whose turn the first and the last heavy give out
    if (v.wv < 2) {
        uint32_t r = 0;
        if (lights > 0) {
            const uint64_t delta = dx[v.wv == 0 ? a0 : a0 + lights - 1];
            r = wave_first_true(0u, B - 1, v.lane, [&](uint32_t i) { return dx[n - i] > delta; });
        }
        if (v.lane == 0) ends[v.wv] = r;
    } else {
        uint32_t r = 0;
        if (heavies > 0) {
            const uint64_t x = dx[n - (v.wv == 2 ? b0 : b0 + heavies - 1)];
            r = wave_first_true(0u, A, v.lane, [&](uint32_t i) { return dx[i] >= x; });
        }
        if (v.lane == 0) ends[v.wv] = r;
    }
    __syncthreads();
    const uint32_t bl = ends[0], bh = ends[1], al_ = ends[2], ah = ends[3];
    const uint32_t nx = bh - bl + 1, nd = ah - al_ + 1;
    const bool staged = nx <= (uint32_t)kBigWindow && nd <= (uint32_t)kBigWindow - nx;  // uniform
    if (staged) {
        for (uint32_t i = threadIdx.x; i < nx + nd; i += kBigThreads)
            win[i] = i < nx ? dx[n - (bl + i)] : dx[al_ + (i - nx)];
        __syncthreads();
    }
    // light: first b in [bl, bh] with X_b > own; heavy: first a in [al, ah] with Delta_a >= own.
    // The upper end is known to satisfy its test, so a lane that is done changes nothing.
    uint64_t own[kBigE];
    uint32_t lo[kBigE], hi[kBigE], rank[kBigE];
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        const bool valid = v.entry(e) < v.n, light = m[e] < C;
        const uint64_t lmask = __ballot(light), hmask = __ballot(valid && !light);
        rank[e] = light ? a_run + rank_below(lmask) : b_run + rank_below(hmask);
        if (!valid) rank[e] = b0;  // some heavy or light of the table: the result is dropped
        own[e] = dx[light ? rank[e] : n - rank[e]];
        lo[e] = light ? bl : al_;
        hi[e] = light ? bh : ah;
        a_run += (uint32_t)__popcll(lmask);
        b_run += (uint32_t)__popcll(hmask);
    }
    const uint32_t span = (nx > nd ? nx : nd) - 1;
    const int steps = 32 - __clz((int)span);  // span < 2^21; 0 for one candidate
    if (staged) {
        for (int s = 0; s < steps; ++s) {
#pragma unroll
            for (int e = 0; e < kBigE; ++e) {
                const bool light = m[e] < C;
                const uint32_t mid = (lo[e] + hi[e]) >> 1;
                const uint64_t x = win[light ? mid - bl : nx + (mid - al_)];
                const bool ok = light ? x > own[e] : x >= own[e];
                hi[e] = ok ? mid : hi[e];
                lo[e] = ok ? lo[e] : (mid < hi[e] ? mid + 1 : mid);
            }
        }
    } else {
        for (int s = 0; s < steps; ++s) {
#pragma unroll
            for (int e = 0; e < kBigE; ++e) {
                const bool light = m[e] < C;
                const uint32_t mid = (lo[e] + hi[e]) >> 1;
                const uint64_t x = dx[light ? n - mid : mid];
                const bool ok = light ? x > own[e] : x >= own[e];
                hi[e] = ok ? mid : hi[e];
                lo[e] = ok ? lo[e] : (mid < hi[e] ? mid + 1 : mid);
            }
        }
    }
    uint32_t split[kBigE], al[kBigE];
#pragma unroll
    for (int e = 0; e < kBigE; ++e) {
        const int32_t k = v.entry(e);
        split[e] = al[e] = 0;
        if (k >= v.n) continue;
        if (m[e] < C) {
            split[e] = (uint32_t)m[e];
            al[e] = hidx[lo[e]];
        } else {
            const uint64_t delta = staged ? win[nx + (lo[e] - al_)] : dx[lo[e]];
            const uint64_t sp = C + own[e] - delta;
            split[e] = (uint32_t)sp;
            al[e] = sp < C ? hidx[rank[e] + 1] : (uint32_t)k;
        }
    }
    typename Io::Loaded got[kBigE];
#pragma unroll
    for (int e = 0; e < kBigE; ++e)
        if (v.entry(e) < v.n) got[e] = io.load(v.entry(e), al[e], raw[e]);
#pragma unroll
    for (int e = 0; e < kBigE; ++e)
        if (v.entry(e) < v.n) io.store(v.entry(e), split[e], al[e], raw[e], got[e]);
}

}  // namespace lda

// Alias-table builder for tables of up to kRegsMaxEntries entries (LightLDA Sec. 4.2, Fig. 2).
// The table is the one alias_build.hpp defines; this form of its construction keeps a lane's
// entries in registers from the first read of the counts to the stores, and pairs the two
// lists by merging them instead of by a search per entry.
//
//   1  quantise: q0 of the thread's entries, sum over the workgroup
//   2  C and pad; the masses, number of lights, their deficit and the heavies' excess
//   3  the two ascending lists with their running sums, in LDS (prefix sums)
//   4  merge: light a precedes heavy b exactly when Delta_a < X_b.  A thread takes a run of
//      consecutive positions of the merged order, finds its start by one bisection along the
//      diagonal and then advances one list or the other per step.  What an entry needs is the
//      place of the other list at its turn: b(a) for a light, a(b) for a heavy.
//   5  output, in entry order: coalesced stores
//
// LDS: 12 bytes per entry (8 of running sums, 2 for the heavies' entries, 2 for the result of
// the merge).
//
// What bounds it: instruction issue and LDS round trips, not memory.  Tables of K = 10 000, one
// workgroup per CU, 141 000 of them: 20.0 ms when the partner of every entry was searched and the
// weights were kept in LDS, 13.9 ms with the merge and a scan for every 64 entries in steps 2 to 5
// (vector units busy for 54 % of the time), 11.2 ms with a run of entries per thread there (2.5
// TB/s).  30 000 tables of 333 bins: 247, 84, 71 us; the lists of a K = 1000 corpus (257 to 1024
// entries) 83 -> 68 us for the last change.
// Four waves per table of 1000 bins, not sixteen: eight tables per CU overlap their phases.
#pragma once

#include "alias_build.hpp"

namespace lda {

constexpr int32_t kRegsMaxEntries = 12 * 1024;  // 1024 threads of 12 entries; 144 KB of lists

__host__ __device__ inline size_t alias_regs_lds_bytes(size_t n)
{
    return (sizeof(uint64_t) * (n + 1) + sizeof(uint16_t) * 2 * n + 7) / 8 * 8;
}

// Sum over the wave of values < 2^51
__device__ __forceinline__ uint64_t wave_total_u64(uint64_t v)
{
    return readlane_u64(wave_inclusive_scan_u64(v), kWave - 1);
}

// Step 4: thread t's run of Em positions of the merged order, an odd number, which spreads the
// threads' reads over the LDS banks.  pq[a]: b(a) of light a; pq[n-1-b]: a(b) of heavy b.  The ends
// need no test: dx[A] is the total of both lists, so past the lights no heavy is preceded by
// "light A", and "heavy B" (also dx[n-B] = dx[A]) precedes no light.
__device__ __forceinline__ void merge_run(const uint64_t* dx, uint16_t* pq, int32_t n, int32_t A, int32_t t,
                                          int32_t Em)
{
    const int32_t B = n - A;
    const int32_t q0 = t * Em;
    const int32_t q1 = q0 + Em < n ? q0 + Em : n;
    if (q0 >= n) return;
    int32_t lo = q0 > B ? q0 - B : 0, hi = q0 < A ? q0 : A;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (dx[mid] < dx[n - (q0 - 1 - mid)]) lo = mid + 1; else hi = mid;
    }
    int32_t a = lo, b = q0 - lo;
    uint64_t da = dx[a], xb = dx[n - b];
    for (int32_t q = q0; q < q1; ++q) {
        const bool lt = da < xb;
        pq[lt ? a : n - 1 - b] = (uint16_t)(lt ? b : a);
        a += lt ? 1 : 0;
        b += lt ? 0 : 1;
        const uint64_t v = dx[lt ? a : n - b];
        da = lt ? v : da;
        xb = lt ? xb : v;
    }
}

// The workgroup's form: all its threads build one table of n <= E * threads entries.  Entries are
// read and written in lane order (coalesced), but steps 2, 3 and 5 work on a run of consecutive
// entries per thread: the prefix sums are then additions in a thread and one scan over the wave
// instead of a scan for every 64 entries.  The masses and the results change between the two
// orders through the LDS that holds the running sums before and after.
template <int E, class Src, class Sink>
__device__ __forceinline__ void build_table_workgroup(int32_t n, const Src& src, const Sink& sink,
                                                      unsigned char* lists, uint64_t& Q0_out,
                                                      uint32_t& C_out)
{
    // dx[0..A]   : Delta_a (exclusive deficit sums of the lights, dx[A] = total)
    // dx[n-b]    : X_b     (inclusive excess sums of the heavies), b = 0..B-1, A + B = n
    uint64_t* const dx = reinterpret_cast<uint64_t*>(lists);
    uint16_t* const hidx = reinterpret_cast<uint16_t*>(dx + (n + 1));  // entry of heavy b
    uint16_t* const pq = hidx + n;  // [a]: b(a) of light a; [n-1-b]: a(b) of heavy b
    __shared__ uint64_t w_a[kMaxWaves], w_b[kMaxWaves], w_q[kMaxWaves], w_q2[kMaxWaves];
    __shared__ uint32_t w_c[kMaxWaves];

    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nw = (int)(blockDim.x >> 6);
    const int32_t T = (int32_t)blockDim.x, t = (int32_t)threadIdx.x;
    // entries of a thread: an odd number where it fits, which spreads the threads' accesses over
    // the LDS banks
    const int32_t per = (n + T - 1) / T;
    const int32_t R = (per | 1) <= E ? (per | 1) : per;
    const int32_t r0 = t * R;
    const int32_t rn = r0 >= n ? 0 : (n - r0 < R ? n - r0 : R);

    // 1: the loads of all entries of a thread are in flight together
    typename Src::Raw raw[E];
    uint64_t m[E];
    uint64_t p0 = 0, p1 = 0, Q0, Q;
    if constexpr (Src::kListed) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int32_t k = e * T + t;
            m[e] = src.mass(k < n ? k : n - 1);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int32_t k = e * T + t;
            if (k < n) dx[k] = m[e];
        }
        __syncthreads();
        src.patch(dx, t, T);
        __syncthreads();
        Q0 = src.Q0();
        Q = src.Q();
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int32_t k = e * T + t;
            raw[e] = src.load(k < n ? k : n - 1);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) src.load2(raw[e]);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int32_t k = e * T + t;
            if (k < n) {
                const uint64_t q = src.q0(raw[e]);
                dx[k] = q;
                p0 += q;
                p1 += q < 1 ? 1 : q;
            }
        }
        Q0 = wave_total_u64(p0);
        Q = wave_total_u64(p1);
        if (lane == 0) { w_a[wv] = Q0; w_q[wv] = Q; }
        __syncthreads();
    }
    auto own_masses = [&]() {
#pragma unroll
        for (int e = 0; e < E; ++e) m[e] = e < rn ? dx[r0 + e] : 0ull;
    };
    // Before the sums or after them: the order decides the registers.  Dense tables of 8 entries a thread 66 or
    // 74 VGPRs, seven or six waves (2006 tables of 3495 bins 57 or 64 us), mixture tables 92 or 72.
    constexpr bool first = Src::kMassesFirst && E > 4;
    if constexpr (first) own_masses();
    if constexpr (!Src::kListed) {
        Q0 = Q = 0;
        for (int i = 0; i < nw; ++i) { Q0 += w_a[i]; Q += w_q[i]; }
    }
    if constexpr (!first) own_masses();
    int sh = 0;
    while ((Q0 >> sh) >= ((uint64_t)n << 31)) ++sh;
    if (sh > 0) {  // uniform
        p1 = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            m[e] >>= sh;
            if (e < rn) p1 += m[e] < 1 ? 1 : m[e];
        }
        Q = wave_total_u64(p1);
        if (lane == 0) w_q2[wv] = Q;
        __syncthreads();
        Q = 0;
        for (int i = 0; i < nw; ++i) Q += w_q2[i];
    }
    // ceil(Q / n) through fp64: Q + n < 2^53, and a quotient below 2^32 that is not a whole
    // number is at least 1/n > 2^-20 away from the next one, more than its rounding error
    const uint64_t C = (uint64_t)((double)(Q + (uint64_t)n - 1) / (double)n);
    const uint64_t pad = (uint64_t)n * C - Q;

    // 2: masses; lights, deficit and excess of the thread's run, and of all runs before it
    uint32_t lc = 0;
    uint64_t df = 0, ex = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e < rn) {
            if (m[e] < 1) m[e] = 1;
            if ((uint64_t)(r0 + e) < pad) m[e] += 1;
            const bool light = m[e] < C;
            lc += light ? 1u : 0u;
            df += light ? C - m[e] : 0ull;
            ex += light ? 0ull : m[e] - C;
        }
    }
    const uint32_t lc_inc = wave_inclusive_scan_u32(lc);
    const uint64_t df_inc = wave_inclusive_scan_u64(df), ex_inc = wave_inclusive_scan_u64(ex);
    __syncthreads();  // w_a of step 1 is no longer read, and neither are the weights in dx
    if (lane == kWave - 1) { w_a[wv] = df_inc; w_b[wv] = ex_inc; w_c[wv] = lc_inc; }
    __syncthreads();
    uint32_t a0 = lc_inc - lc, A = 0;
    uint64_t d0 = df_inc - df, x0 = ex_inc - ex, d_tot = 0;
    for (int i = 0; i < nw; ++i) {
        if (i < wv) { a0 += w_c[i]; d0 += w_a[i]; x0 += w_b[i]; }
        A += w_c[i];
        d_tot += w_a[i];
    }
    if (t == 0) dx[A] = d_tot;

    // 3: the lists
    uint32_t a_run = a0, b_run = (uint32_t)(r0 < n ? r0 : n) - a0;
    const uint32_t b0 = b_run;
    uint64_t d_run = d0, x_run = x0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e < rn) {
            const bool light = m[e] < C;
            const uint64_t x_inc = x_run + (m[e] - C);
            dx[light ? a_run : (uint32_t)n - b_run] = light ? d_run : x_inc;
            if (!light) hidx[b_run] = (uint16_t)(r0 + e);
            d_run += light ? C - m[e] : 0ull;
            x_run = light ? x_run : x_inc;
            a_run += light ? 1u : 0u;
            b_run += light ? 0u : 1u;
        }
    }
    __syncthreads();

    // 4: merge
    merge_run(dx, pq, n, (int32_t)A, t, per | 1);
    __syncthreads();

    // 5: output, brought back into lane order
    a_run = a0;
    b_run = b0;
    x_run = x0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e < rn) {
            const bool light = m[e] < C;
            x_run += light ? 0ull : m[e] - C;
            const uint32_t other = pq[light ? a_run : (uint32_t)n - 1 - b_run];
            uint32_t split, al;
            if (light) {
                split = (uint32_t)m[e];
                al = hidx[other];
            } else {
                const uint64_t sp = C + x_run - dx[other];
                split = (uint32_t)sp;
                al = sp < C ? hidx[b_run + 1] : (uint32_t)(r0 + e);
            }
            a_run += light ? 1u : 0u;
            b_run += light ? 0u : 1u;
            m[e] = ((uint64_t)al << 32) | split;
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e < rn) dx[r0 + e] = m[e];
    if constexpr (Src::kListed) {  // hidx and pq, 4 bytes an entry, are no longer read
        sink.clear(reinterpret_cast<int32_t*>(hidx), n, t, T);
        __syncthreads();
        sink.fill(reinterpret_cast<int32_t*>(hidx), t, T);
    }
    __syncthreads();
    if constexpr (Src::kListed) {
#pragma unroll
        for (int e = 0; e < E; ++e) raw[e] = src.load(e * T + t < n ? e * T + t : n - 1);
    }
    typename Sink::Loaded got[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int32_t k = e * T + t;
        if (k < n) {
            m[e] = dx[k];
            got[e] = sink.load(k, (uint32_t)(m[e] >> 32), raw[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int32_t k = e * T + t;
        if (k < n) sink.store(k, (uint32_t)m[e], (uint32_t)(m[e] >> 32), raw[e], got[e]);
    }
    Q0_out = Q0;
    C_out = (uint32_t)C;
}

// One wave's form: entry e * 64 + lane is in the lane's registers throughout, so lists and results
// need no change of order; the prefix sums are scans over the wave, 64 entries at a time.
template <int E, class Src, class Sink>
__device__ __forceinline__ void build_table_wave(int32_t n, const Src& src, const Sink& sink,
                                                 unsigned char* lists, uint64_t& Q0_out,
                                                 uint32_t& C_out)
{
    // dx[0..A]   : Delta_a (exclusive deficit sums of the lights, dx[A] = total)
    // dx[n-b]    : X_b     (inclusive excess sums of the heavies), b = 0..B-1, A + B = n
    uint64_t* const dx = reinterpret_cast<uint64_t*>(lists);
    uint16_t* const hidx = reinterpret_cast<uint16_t*>(dx + (n + 1));  // entry of heavy b
    uint16_t* const pq = hidx + n;  // [a]: b(a) of light a; [n-1-b]: a(b) of heavy b

    const int lane = threadIdx.x & (kWave - 1);

    // 1: the loads of all entries of a lane are in flight together
    typename Src::Raw raw[E];
    uint64_t m[E];
    uint64_t p0 = 0, p1 = 0, Q0, Q;
    if constexpr (Src::kListed) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int32_t k = e * kWave + lane;
            m[e] = src.mass(k < n ? k : n - 1);
            if (k < n) dx[k] = m[e];
        }
        wave_lds_order();
        src.patch(dx, lane, kWave);
        wave_lds_order();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int32_t k = e * kWave + lane;
            m[e] = dx[k < n ? k : n - 1];
        }
        wave_lds_order();
        Q0 = src.Q0();
        Q = src.Q();
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int32_t k = e * kWave + lane;
            raw[e] = src.load(k < n ? k : n - 1);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) src.load2(raw[e]);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            m[e] = src.q0(raw[e]);
            if (e * kWave + lane < n) {
                p0 += m[e];
                p1 += m[e] < 1 ? 1 : m[e];
            }
        }
        Q0 = wave_total_u64(p0);
        Q = wave_total_u64(p1);
    }
    int sh = 0;
    while ((Q0 >> sh) >= ((uint64_t)n << 31)) ++sh;
    if (sh > 0) {  // uniform
        p1 = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            m[e] >>= sh;
            if (e * kWave + lane < n) p1 += m[e] < 1 ? 1 : m[e];
        }
        Q = wave_total_u64(p1);
    }
    // ceil(Q / n) through fp64: Q + n < 2^53, and a quotient below 2^32 that is not a whole
    // number is at least 1/n > 2^-20 away from the next one, more than its rounding error
    const uint64_t C = (uint64_t)((double)(Q + (uint64_t)n - 1) / (double)n);
    const uint64_t pad = (uint64_t)n * C - Q;

    // 2: masses, the lights and their deficit
    uint32_t lc = 0;
    uint64_t df = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int32_t k = e * kWave + lane;
        if (m[e] < 1) m[e] = 1;
        if ((uint64_t)k < pad) m[e] += 1;
        const bool valid = k < n;
        const bool light = valid && m[e] < C;
        lc += (uint32_t)__popcll(__ballot(light));
        if (light) df += C - m[e];
    }
    df = wave_total_u64(df);
    const uint32_t A = lc;
    uint32_t a_run = 0;
    uint64_t d_run = 0, x_run = 0;
    if (lane == 0) dx[A] = df;

    // 3: the lists
    uint32_t b_run = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int32_t k0 = e * kWave;
        if (k0 < n) {  // uniform over the wave
            const bool valid = k0 + lane < n;
            const bool light = valid && m[e] < C;
            const bool heavy = valid && !light;
            const uint64_t lmask = __ballot(light), hmask = __ballot(heavy);
            const uint32_t la = rank_below(lmask);
            if (lmask != 0) {
                const uint64_t dinc = wave_inclusive_scan_u64(light ? C - m[e] : 0ull);
                if (light) dx[a_run + la] = d_run + dinc - (C - m[e]);
                d_run += readlane_u64(dinc, kWave - 1);
            }
            if (hmask != 0) {
                const uint64_t xinc = wave_inclusive_scan_u64(heavy ? m[e] - C : 0ull);
                if (heavy) {
                    const uint32_t b = b_run + ((uint32_t)lane - la);
                    dx[n - b] = x_run + xinc;
                    hidx[b] = (uint16_t)(k0 + lane);
                }
                x_run += readlane_u64(xinc, kWave - 1);
            }
            a_run += (uint32_t)__popcll(lmask);
            b_run += (uint32_t)__popcll(hmask);
        }
    }
    wave_lds_order();

    // 4: merge
    merge_run(dx, pq, n, (int32_t)A, lane, ((n + kWave - 1) / kWave) | 1);
    wave_lds_order();

    // 5: output
    uint32_t split[E], al[E];
    a_run = 0;
    b_run = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        split[e] = al[e] = 0;
        const int32_t k0 = e * kWave;
        if (k0 < n) {
            const int32_t k = k0 + lane;
            const bool valid = k < n;
            const bool light = valid && m[e] < C;
            const uint64_t lmask = __ballot(light);
            const uint32_t la = rank_below(lmask);
            if (light) {
                split[e] = (uint32_t)m[e];
                al[e] = hidx[pq[a_run + la]];
            } else if (valid) {
                const uint32_t b = b_run + ((uint32_t)lane - la);
                const uint64_t sp = C + dx[n - b] - dx[pq[n - 1 - b]];
                split[e] = (uint32_t)sp;
                al[e] = sp < C ? hidx[b + 1] : (uint32_t)k;
            }
            const uint32_t nl = (uint32_t)__popcll(lmask);
            a_run += nl;
            b_run += (uint32_t)((n - k0 < kWave) ? n - k0 : kWave) - nl;
        }
    }
    if constexpr (Src::kListed) {  // hidx and pq, 4 bytes an entry, are no longer read
        wave_lds_order();
        sink.clear(reinterpret_cast<int32_t*>(hidx), n, lane, kWave);
        wave_lds_order();
        sink.fill(reinterpret_cast<int32_t*>(hidx), lane, kWave);
        wave_lds_order();
#pragma unroll
        for (int e = 0; e < E; ++e) raw[e] = src.load(e * kWave + lane < n ? e * kWave + lane : n - 1);
    }
    typename Sink::Loaded got[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int32_t k = e * kWave + lane;
        if (k < n) got[e] = sink.load(k, al[e], raw[e]);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int32_t k = e * kWave + lane;
        if (k < n) sink.store(k, split[e], al[e], raw[e], got[e]);
    }
    Q0_out = Q0;
    C_out = (uint32_t)C;
}

// Builds one table of n entries, n <= E * (threads that build it): one wave (ONE, n <= 64 E; no
// workgroup barrier, so the waves of a workgroup can build tables of their own) or the whole
// workgroup.  lists: alias_regs_lds_bytes(n) bytes, 8-byte aligned.  Src: Raw load(k), void
// load2(Raw&) for what is addressed by the first load, uint64_t q0(Raw).  Sink: Loaded
// load(k, alias, raw), store(k, split, alias, raw, loaded), once per entry.  Returns the
// pre-shift sum Q0 and the capacity C.
// A workgroup that builds another table in the same LDS synchronises first.
template <int E, bool ONE, class Src, class Sink>
__device__ __forceinline__ void build_table_regs(int32_t n, const Src& src, const Sink& sink,
                                                 unsigned char* lists, uint64_t& Q0_out,
                                                 uint32_t& C_out)
{
    if constexpr (ONE) build_table_wave<E>(n, src, sink, lists, Q0_out, C_out);
    else build_table_workgroup<E>(n, src, sink, lists, Q0_out, C_out);
}

}  // namespace lda

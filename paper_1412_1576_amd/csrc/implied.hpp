// Implied tables: the dense K-bin table of a word with few tokens, without its bins.
//
// A word with few tokens has counts for few topics.  The mass of every other bin is that of a
// topic the word has no token of, q_k = max(1, floor(beta / (n_k + betabar) * 2^40)), the same for
// all words; what differs between the words is the capacity C and pad, and the bins of the
// topics they do have.  If all bins without tokens are lights (alias_build.hpp), their exclusive
// deficit sum follows from one prefix sum over q that all words share,
//
//   Delta(k) = k C - PZ[k] - min(k, pad) - corr(k)      PZ[k] = sum of q_j over j < k
//
// where corr(k) sums over the word's own topics below k what they take away from it: q_k's deficit,
// and the deficit of the bin's true mass instead if that is a light too.  The heavies are among
// the word's own topics.  So a word's table is its topics in ascending order with two running sums
// each, corr and the excess X, and a bin's split and alias -- the very ones the closed form of
// alias_build.hpp gives -- are found when a draw needs them:
//
//   no tokens    split = q_k + (k < pad); alias = the first topic with X > Delta(k)
//   a light      split = its mass, which corr holds; alias likewise
//   a heavy      split = C + X - min{Delta : Delta >= X}, by bisection; alias = the next heavy
//
// A word whose sums do not fit that (a bin without tokens would be heavy, or the weights need a
// shift) gets its dense table, as before, and is marked.
#pragma once

#include "common.hpp"

namespace lda {

constexpr int32_t kImpliedTokens = 1024;  // most tokens of such a word, and of a piece of the word pass
constexpr int32_t kImpliedWords = 512;    // words of a piece
constexpr uint32_t kImpliedDense = 0x80000000u;  // in a word's n: it draws from its dense table

// The words whose sums do not fit are put on kMisfitLists lists in turn, whose lengths are a cache line
// apart: with one length for all, 41 000 such words took 490 us, the atomics on it 12 ns each.
constexpr int32_t kMisfitLists = 64, kMisfitStride = 32;
inline int32_t misfit_list_words(int32_t n_implied) { return (n_implied + kMisfitLists - 1) / kMisfitLists; }

// An entry's key: topic << 17 | light << 16 | count (K <= 12 288 < 2^14, count <= 1024)
constexpr int kImpliedTopicShift = 17;
constexpr uint32_t kImpliedLight = 1u << 16;
constexpr uint32_t kImpliedCount = 0xFFFFu;

// A word's header: (n | kImpliedDense, C, pad, unused)
struct ImpliedWord {
    const uint32_t* key;    // [n] in LDS
    const uint64_t* corr;   // [n] inclusive
    const uint64_t* x;      // [n] inclusive excess
    int32_t n;
    uint32_t C, pad;
};

// entries with a topic below t
__device__ __forceinline__ int32_t implied_below(const ImpliedWord& w, uint32_t t)
{
    int32_t lo = 0, len = w.n;
    while (len > 0) {
        const int32_t half = len >> 1;
        const bool less = (w.key[lo + half] >> kImpliedTopicShift) < t;
        lo = less ? lo + half + 1 : lo;
        len = less ? len - half - 1 : half;
    }
    return lo;
}

__device__ __forceinline__ int32_t implied_count(const ImpliedWord& w, int32_t t)
{
    const int32_t i = implied_below(w, (uint32_t)t);
    if (i >= w.n) return 0;
    const uint32_t k = w.key[i];
    return (k >> kImpliedTopicShift) == (uint32_t)t ? (int32_t)(k & kImpliedCount) : 0;
}

// first entry with X > d; there is one for every d below the sum of all deficits
__device__ __forceinline__ int32_t implied_heavy_above(const ImpliedWord& w, uint64_t d)
{
    int32_t lo = 0, hi = w.n - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        const bool above = w.x[mid] > d;
        hi = above ? mid : hi;
        lo = above ? lo : mid + 1;
    }
    return lo;
}

// Delta(k) with `i` of the word's topics below k
__device__ __forceinline__ uint64_t implied_delta(const ImpliedWord& w, const uint64_t* __restrict__ pz,
                                                  uint32_t k, int32_t i)
{
    const uint64_t full = (uint64_t)k * w.C - pz[k] - (k < w.pad ? k : w.pad);
    return i > 0 ? full - w.corr[i - 1] : full;
}

// A draw: bin `bin`, height rr < C.  One that hits a heavy needs a search in memory, which a wave
// makes for all its lanes' draws together (implied_heavy), so it is left pending.
struct ImpliedDraw {
    uint32_t bin, rr;
    int32_t i;      // the word's topics below bin
    bool pending;
};

// The topic, and the word's count of it, unless the draw is left pending
__device__ __forceinline__ ImpliedDraw implied_draw(const ImpliedWord& w, const uint64_t* __restrict__ pz,
                                                    uint32_t q, uint32_t bin, uint32_t rr, int32_t& t, int32_t& nw)
{
    const int32_t i = implied_below(w, bin);
    uint32_t split = (q < 1u ? 1u : q) + (bin < w.pad ? 1u : 0u);
    uint32_t own = 0u;  // key of the bin's own topic
    if (i < w.n) {
        const uint32_t k = w.key[i];
        if ((k >> kImpliedTopicShift) == bin) {
            if ((k & kImpliedLight) == 0u) return ImpliedDraw{bin, rr, i, true};
            own = k;
            split += (uint32_t)(w.corr[i] - (i > 0 ? w.corr[i - 1] : 0ull));
        }
    }
    t = (int32_t)bin;
    nw = (int32_t)(own & kImpliedCount);
    if (rr >= split) {
        const uint32_t k = w.key[implied_heavy_above(w, implied_delta(w, pz, bin, i))];
        t = (int32_t)(k >> kImpliedTopicShift);
        nw = (int32_t)(k & kImpliedCount);
    }
    return ImpliedDraw{bin, rr, i, false};
}

// A pending draw.  The split is C + X - (the smallest Delta that is not below X), found from an estimate
// with the mean mass in the place of PZ: topics of even sizes leave two or three looks at PZ to each of
// the two searches, where bisections took some fifteen, one after the other.
__device__ __forceinline__ void implied_heavy(const ImpliedWord& w, const uint64_t* __restrict__ pz, uint32_t K,
                                              const ImpliedDraw& d, int32_t& t, int32_t& nw)
{
    const uint64_t x = w.x[d.i];
    const uint32_t own = w.key[d.i];
    const double step = (double)w.C - (double)pz[K] / (double)K;  // (positive: every q is below C)
    // the first of the word's topics with Delta >= X (n: none, but Delta(K) is)
    int32_t lo = 0, hi = w.n;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        const double est = (double)(w.key[mid] >> kImpliedTopicShift) * step - (double)(mid > 0 ? w.corr[mid - 1] : 0ull);
        const bool ge = est >= (double)x;
        hi = ge ? mid : hi;
        lo = ge ? lo : mid + 1;
    }
    int32_t e = lo;
    {
        // bracket [el, eh): Delta(topic el - 1) < X <= Delta(topic eh), by doubling steps from the estimate
        auto reaches = [&](int32_t i) { return implied_delta(w, pz, w.key[i] >> kImpliedTopicShift, i) >= x; };
        int32_t el = 0, eh = w.n;
        if (e < w.n && !reaches(e)) {
            el = e + 1;
            for (int32_t s = 1; el < eh; s *= 2) {
                const int32_t at = el + s - 1 < eh ? el + s - 1 : eh - 1;
                if (reaches(at)) { eh = at; break; }
                el = at + 1;
            }
        } else {
            eh = e;
            for (int32_t s = 1; el < eh; s *= 2) {
                const int32_t at = eh - s > el ? eh - s : el;
                if (!reaches(at)) { el = at + 1; break; }
                eh = at;
            }
        }
        while (el < eh) {
            const int32_t mid = (el + eh) >> 1;
            if (reaches(mid)) eh = mid; else el = mid + 1;
        }
        e = el;
    }
    // and the first bin up to it: Delta(below) < X <= Delta(b)
    uint32_t a = e > 0 ? (w.key[e - 1] >> kImpliedTopicShift) + 1u : 0u;
    uint32_t b = e < w.n ? w.key[e] >> kImpliedTopicShift : K;
    uint64_t da = implied_delta(w, pz, a, e), db = da;
    if (da < x) {
        db = implied_delta(w, pz, b, e);
        for (int tries = 0; b - a > 1u; ++tries) {
            uint32_t mid = (a + b) >> 1;
            if (tries < 4) {
                const double g = (double)a + ceil((double)(x - da) / step);
                mid = g < (double)b ? (uint32_t)g : b - 1u;
                mid = mid > a ? mid : a + 1u;
            }
            const uint64_t dm = implied_delta(w, pz, mid, e);
            if (dm >= x) { b = mid; db = dm; } else { a = mid; da = dm; }
        }
    }
    t = (int32_t)d.bin;
    nw = (int32_t)(own & kImpliedCount);
    // (a split of C keeps every rr, so the last heavy never looks for a next one)
    if ((uint64_t)d.rr + (db - x) >= (uint64_t)w.C) {
        int32_t j = d.i + 1;
        while (j < w.n - 1 && (w.key[j] & kImpliedLight)) ++j;
        const uint32_t k = w.key[j];
        t = (int32_t)(k >> kImpliedTopicShift);
        nw = (int32_t)(k & kImpliedCount);
    }
}

}  // namespace lda

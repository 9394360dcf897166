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

// The topic that bin `bin` and height rr < C give, and the word's count of it
__device__ __forceinline__ void implied_draw(const ImpliedWord& w, const uint64_t* __restrict__ pz,
                                             const uint32_t* __restrict__ qz, uint32_t K, uint32_t bin,
                                             uint32_t rr, int32_t& t, int32_t& nw)
{
    const int32_t i = implied_below(w, bin);
    const uint32_t q = qz[bin];
    uint32_t split = (q < 1u ? 1u : q) + (bin < w.pad ? 1u : 0u);
    uint32_t own = 0u;  // key of the bin's own topic
    bool heavy = false;
    if (i < w.n) {
        const uint32_t k = w.key[i];
        if ((k >> kImpliedTopicShift) == bin) {
            own = k;
            heavy = (k & kImpliedLight) == 0u;
            if (!heavy) split += (uint32_t)(w.corr[i] - (i > 0 ? w.corr[i - 1] : 0ull));
        }
    }
    int32_t j;
    if (heavy) {
        // the smallest Delta that is not below X: first between which topics, then at which bin
        const uint64_t x = w.x[i];
        int32_t lo = 0, hi = w.n;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            const bool ge = implied_delta(w, pz, w.key[mid] >> kImpliedTopicShift, mid) >= x;
            hi = ge ? mid : hi;
            lo = ge ? lo : mid + 1;
        }
        const int32_t e = lo;  // Delta >= x holds at topic e (or, past the last one, at K)
        uint32_t a = e > 0 ? (w.key[e - 1] >> kImpliedTopicShift) + 1u : 0u;
        uint32_t b = e < w.n ? w.key[e] >> kImpliedTopicShift : K;
        while (a < b) {
            const uint32_t mid = (a + b) >> 1;
            const bool ge = implied_delta(w, pz, mid, e) >= x;
            b = ge ? mid : b;
            a = ge ? a : mid + 1u;
        }
        const uint64_t past = implied_delta(w, pz, a, e) - x;
        // (a split of C keeps every rr, so the last heavy never looks for a next one)
        if ((uint64_t)rr + past < (uint64_t)w.C) {
            t = (int32_t)bin;
            nw = (int32_t)(own & kImpliedCount);
            return;
        }
        for (j = i + 1; j < w.n - 1 && (w.key[j] & kImpliedLight); ++j) {}
    } else {
        if (rr < split) {
            t = (int32_t)bin;
            nw = (int32_t)(own & kImpliedCount);
            return;
        }
        j = implied_heavy_above(w, implied_delta(w, pz, bin, i));
    }
    const uint32_t k = w.key[j];
    t = (int32_t)(k >> kImpliedTopicShift);
    nw = (int32_t)(k & kImpliedCount);
}

}  // namespace lda

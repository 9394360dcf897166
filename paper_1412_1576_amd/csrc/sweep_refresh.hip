// Sweep with the doc side refreshed after every token (LightLDA Sec. 4.2, footnote 4: the
// doc-proposal is not frozen during a document but follows its assignments token by token) and the word side -- n_kw, n_k, the word-proposal tables -- kept at the snapshot
// (Sec. 6, the immutable model slice).  Selected by lda_options.doc_refresh.
//
// The tokens of a document are visited in order, so a document is a sequential chain; the
// documents are independent.  Two forms.  Where K is large against the documents, one wave per
// document: the document's current assignment sits
// in the wave's part of the LDS, n_kd of a topic is a ballot count over it, and everything
// that does not depend on the document's state -- the Philox numbers of every step, the
// word-proposal draws with their n_kw and n_k -- is computed 64 tokens at a time, one token
// per lane, before those tokens take their turns one after the other.
#include <algorithm>

#include "common.hpp"

namespace lda {

namespace {

constexpr int kRefreshWaves = 4;           // documents per workgroup
constexpr int32_t kRefreshMaxDoc = 4096;   // tokens of the longest document (16 KB of LDS per wave)

struct RefreshArgs {
    const int32_t* word;
    const int32_t* z;
    int32_t* znew;
    const int32_t* doff;
    const int32_t* nkw;
    const int32_t* nk;
    const uint4* alias;  // (split, alias, n_kw[bin], n_kw[alias]) per bin
    const uint32_t* cap;
    int32_t D, K, mode;
    int32_t lds_doc;     // ints of a document in LDS
    int32_t lds_counts;  // of them the n_kd counters (the form with counters)
    double alpha, beta, alphabar, betabar;
    uint32_t seed_lo, seed_hi, sweep;
};

// n_kd of topic k in the document whose current assignment is zs[0..L): every lane gets it
__device__ __forceinline__ int32_t doc_count(const int32_t* zs, int32_t L, int lane, int32_t k)
{
    int32_t c = 0;
    for (int32_t b = 0; b < L; b += 64) {
        const int32_t v = (b + lane < L) ? zs[b + lane] : -1;
        c += (int32_t)__popcll(__ballot(v == k));
    }
    return c;
}

template <int M>
__global__ __launch_bounds__(64 * kRefreshWaves) void sweep_doc_refresh_kernel(RefreshArgs A)
{
#pragma clang fp contract(off)
    extern __shared__ int32_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int32_t d = (int32_t)blockIdx.x * kRefreshWaves + wave;
    if (d >= A.D) return;  // a whole wave leaves; no workgroup barrier follows
    const int32_t b = A.doff[d], L = A.doff[d + 1] - b;
    if (L == 0) return;
    int32_t* __restrict__ zs = smem + (size_t)wave * A.lds_doc;
    for (int32_t i = lane; i < L; i += 64) zs[i] = A.z[b + i];
    wave_lds_order();
    const int32_t K = A.K;
    const double Ld = (double)L;
    for (int32_t base = 0; base < L; base += 64) {
        // ---- one token per lane: what its chain needs from the snapshot ----
        const int32_t i = (base + lane < L) ? base + lane : L - 1;  // lanes past the end: a clone
        const uint32_t g = (uint32_t)(b + i);
        const int32_t w = A.word[g];
        const int32_t z0 = A.z[g];
        const size_t wk = (size_t)w * (size_t)K;
        const uint32_t capw = A.cap[w];
        const int32_t nw_z0 = A.nkw[wk + (size_t)z0];
        const int32_t nk_z0 = A.nk[z0];
        uint32_t x0[M], x1[M], x2[M];
        int32_t tw[M], nwt[M], nkt[M];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const bool word_step = (A.mode == 0) ? ((j & 1) == 0) : (A.mode == 1);
            uint32_t x[4];
            philox4x32_10(g, 0u, A.sweep, (uint32_t)j, A.seed_lo, A.seed_hi, x);
            x0[j] = x[0]; x1[j] = x[1]; x2[j] = x[2];
            tw[j] = 0; nwt[j] = 0; nkt[j] = 0;
            if (word_step) {  // Fig. 2: uniform bin, uniform height, keep the bin or take its alias
                const uint32_t bin = mulhi32(x[0], (uint32_t)K);
                const uint32_t rr = mulhi32(x[1], capw);
                const uint4 e = A.alias[wk + bin];
                const bool keep = rr < e.x;
                tw[j] = keep ? (int32_t)bin : (int32_t)e.y;
                nwt[j] = keep ? (int32_t)e.z : (int32_t)e.w;
                nkt[j] = A.nk[tw[j]];
            }
        }
        // ---- the tokens take their turns ----
        const int32_t turns = (L - base < 64) ? L - base : 64;
        for (int32_t q = 0; q < turns; ++q) {
            const int32_t z0q = __shfl(z0, q, 64);
            const size_t wkq = (size_t)__shfl(w, q, 64) * (size_t)K;
            int32_t s = z0q;
            int32_t nds = doc_count(zs, L, lane, z0q);
            int32_t nws = __shfl(nw_z0, q, 64);
            int32_t nks = __shfl(nk_z0, q, 64);
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const bool word_step = (A.mode == 0) ? ((j & 1) == 0) : (A.mode == 1);
                int32_t t, nw_t, nk_t;
                if (word_step) {
                    t = __shfl(tw[j], q, 64);
                    nw_t = __shfl(nwt[j], q, 64);
                    nk_t = __shfl(nkt[j], q, 64);
                } else {  // Eq. (9), (12) on the document as it stands now
                    const double u0 = unit_open(__shfl(x0[j], q, 64));
                    const uint32_t x1q = __shfl(x1[j], q, 64);
                    if (u0 * (Ld + A.alphabar) < Ld) t = zs[mulhi32(x1q, (uint32_t)L)];
                    else t = (int32_t)mulhi32(x1q, (uint32_t)K);
                    nw_t = A.nkw[wkq + (size_t)t];
                    nk_t = A.nk[t];
                }
                const int32_t nd_t = doc_count(zs, L, lane, t);
                const int32_t ms = (s == z0q) ? 1 : 0;
                const int32_t mt = (t == z0q) ? 1 : 0;
                // Eq. (4) ratio p(t)/p(s), the token removed at its snapshot topic
                double num = (double)(nd_t - mt) + A.alpha;
                num = num * ((double)(nw_t - mt) + A.beta);
                num = num * ((double)(nks - ms) + A.betabar);
                double den = (double)(nds - ms) + A.alpha;
                den = den * ((double)(nws - ms) + A.beta);
                den = den * ((double)(nk_t - mt) + A.betabar);
                if (word_step) {  // Eq. (8): times p_w(s)/p_w(t)
                    num = num * ((double)nws + A.beta);
                    num = num * ((double)nk_t + A.betabar);
                    den = den * ((double)nw_t + A.beta);
                    den = den * ((double)nks + A.betabar);
                } else {          // Eq. (11): times p_d(s)/p_d(t)
                    num = num * ((double)nds + A.alpha);
                    den = den * ((double)nd_t + A.alpha);
                }
                const double uu = unit_open(__shfl(x2[j], q, 64));
                const bool accept = (t != s) && (uu * den < num);
                s = accept ? t : s;
                nds = accept ? nd_t : nds;
                nws = accept ? nw_t : nws;
                nks = accept ? nk_t : nks;
            }
            if (lane == 0) {
                zs[base + q] = s;  // the rest of the document sees the move
                A.znew[b + base + q] = s;
            }
            wave_lds_order();
        }
    }
}

// The same sweep with n_kd of a document kept as K 16-bit counters in the LDS and G lanes to a
// document, 64 / G documents to a wave.  In a round every lane prepares its own token as above,
// and also looks up n_kw and n_k for the topics its doc steps would copy from the document as it
// stands when the round begins; when its turn comes it reads those positions again and repeats
// the look-ups only if an earlier token of the round moved (about G / 2L of the doc steps).
// A turn is one lane's work, on its own registers: two LDS round trips and the accept tests,
// for 64 / G documents in step, where the form above spends a whole wave's instructions on one
// token and counts a topic by L / 64 LDS reads.  Bound by the latency of a turn times the
// documents that fit the LDS (60 000 documents of 332 tokens, K = 1000: 7.7 -> 1.4 ms).
template <int M, int G>
__global__ __launch_bounds__(64) void sweep_doc_refresh_counts_kernel(RefreshArgs A)
{
#pragma clang fp contract(off)
    extern __shared__ int32_t smem[];
    const int lane = (int)threadIdx.x, sub = lane % G;
    const int64_t d = (int64_t)blockIdx.x * (64 / G) + lane / G;
    const int32_t b = d < A.D ? A.doff[d] : 0, L = d < A.D ? A.doff[d + 1] - b : 0;
    int32_t* __restrict__ mine = smem + (size_t)(lane / G) * A.lds_doc;
    uint16_t* cnt = reinterpret_cast<uint16_t*>(mine);
    uint16_t* zs = reinterpret_cast<uint16_t*>(mine + A.lds_counts);
    if (L > 0) {
        for (int32_t i = sub; i < A.lds_counts / 4; i += G)
            reinterpret_cast<int4*>(mine)[i] = make_int4(0, 0, 0, 0);
    }
    wave_lds_order();
    for (int32_t i = sub; i < L; i += G) {
        const uint32_t k = (uint32_t)A.z[b + i];
        zs[i] = (uint16_t)k;
        atomicAdd(reinterpret_cast<uint32_t*>(mine) + (k >> 1), 1u << (16 * (k & 1)));
    }
    wave_lds_order();
    const int32_t K = A.K;
    const double Ld = (double)L;
    int32_t w_next = L > 0 ? A.word[b + (sub < L ? sub : L - 1)] : 0;
    for (int32_t base = 0; base < L; base += G) {
        // ---- one token per lane: all that does not depend on this round's moves ----
        const int32_t i = (base + sub < L) ? base + sub : L - 1;  // lanes past the end: a clone
        const uint32_t g = (uint32_t)(b + i);
        const int32_t w = w_next;
        if (base + G < L) w_next = A.word[b + ((base + G + sub < L) ? base + G + sub : L - 1)];
        const int32_t z0 = (int32_t)zs[i];  // not moved before its turn
        const size_t wk = (size_t)w * (size_t)K;
        const uint32_t capw = A.cap[w];
        const int32_t nw_z0 = A.nkw[wk + (size_t)z0];
        const int32_t nk_z0 = A.nk[z0];
        uint32_t x2[M];
        int32_t tt[M], nwt[M], nkt[M], from[M];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const bool word_step = (A.mode == 0) ? ((j & 1) == 0) : (A.mode == 1);
            uint32_t x[4];
            philox4x32_10(g, 0u, A.sweep, (uint32_t)j, A.seed_lo, A.seed_hi, x);
            x2[j] = x[2];
            from[j] = -1;
            if (word_step) {  // Fig. 2: uniform bin, uniform height, keep the bin or take its alias
                const uint32_t bin = mulhi32(x[0], (uint32_t)K);
                const uint32_t rr = mulhi32(x[1], capw);
                const uint4 e = A.alias[wk + bin];
                const bool keep = rr < e.x;
                tt[j] = keep ? (int32_t)bin : (int32_t)e.y;
                nwt[j] = keep ? (int32_t)e.z : (int32_t)e.w;
            } else {  // Eq. (9), (12)
                const double u0 = unit_open(x[0]);
                if (u0 * (Ld + A.alphabar) < Ld) {
                    from[j] = (int32_t)mulhi32(x[1], (uint32_t)L);
                    tt[j] = (int32_t)zs[from[j]];
                } else {
                    tt[j] = (int32_t)mulhi32(x[1], (uint32_t)K);
                }
                nwt[j] = A.nkw[wk + (size_t)tt[j]];
            }
            nkt[j] = A.nk[tt[j]];
        }
        // ---- the tokens take their turns ----
        const int32_t turns = (L - base < G) ? L - base : G;
        int32_t s = z0;
        for (int32_t q = 0; q < turns; ++q) {
            if (sub == q) {
                int32_t nd[M];
                const int32_t nd_z0 = (int32_t)cnt[z0];
#pragma unroll
                for (int j = 0; j < M; ++j) {
                    const bool word_step = (A.mode == 0) ? ((j & 1) == 0) : (A.mode == 1);
                    if (!word_step && from[j] >= 0) {
                        const int32_t t = (int32_t)zs[from[j]];
                        if (t != tt[j]) {
                            tt[j] = t;
                            nwt[j] = A.nkw[wk + (size_t)t];
                            nkt[j] = A.nk[t];
                        }
                    }
                    nd[j] = (int32_t)cnt[tt[j]];
                }
                int32_t nds = nd_z0, nws = nw_z0, nks = nk_z0;
#pragma unroll
                for (int j = 0; j < M; ++j) {
                    const bool word_step = (A.mode == 0) ? ((j & 1) == 0) : (A.mode == 1);
                    const int32_t t = tt[j], nw_t = nwt[j], nk_t = nkt[j], nd_t = nd[j];
                    const int32_t ms = (s == z0) ? 1 : 0;
                    const int32_t mt = (t == z0) ? 1 : 0;
                    // Eq. (4) ratio p(t)/p(s), the token removed at its snapshot topic
                    double num = (double)(nd_t - mt) + A.alpha;
                    num = num * ((double)(nw_t - mt) + A.beta);
                    num = num * ((double)(nks - ms) + A.betabar);
                    double den = (double)(nds - ms) + A.alpha;
                    den = den * ((double)(nws - ms) + A.beta);
                    den = den * ((double)(nk_t - mt) + A.betabar);
                    if (word_step) {  // Eq. (8): times p_w(s)/p_w(t)
                        num = num * ((double)nws + A.beta);
                        num = num * ((double)nk_t + A.betabar);
                        den = den * ((double)nw_t + A.beta);
                        den = den * ((double)nks + A.betabar);
                    } else {          // Eq. (11): times p_d(s)/p_d(t)
                        num = num * ((double)nds + A.alpha);
                        den = den * ((double)nd_t + A.alpha);
                    }
                    const double uu = unit_open(x2[j]);
                    const bool accept = (t != s) && (uu * den < num);
                    s = accept ? t : s;
                    nds = accept ? nd_t : nds;
                    nws = accept ? nw_t : nws;
                    nks = accept ? nk_t : nks;
                }
                if (s != z0) {  // the rest of the document sees the move
                    cnt[z0] = (uint16_t)(nd_z0 - 1);
                    cnt[s] = (uint16_t)(nds + 1);
                    zs[i] = (uint16_t)s;
                }
            }
            wave_lds_order();
        }
        if (base + sub < L) A.znew[g] = s;
    }
}

// LDS ints of a document's counters (two to an int, cleared 16 bytes at a time) and of the
// document, whose assignment follows them as 16-bit topics
int32_t counter_ints(int32_t K) { return (K + 7) / 8 * 4; }
int32_t counts_doc_ints(int32_t K, int32_t longest_doc) { return counter_ints(K) + (longest_doc + 7) / 8 * 4; }

// Lanes of a document in the form with counters, 0 for the form without.
//
// Fewer lanes put more documents into a turn, but the documents of a wave share its LDS: the
// counters of 64 / G documents should leave room for 8 waves on a CU, and there should be 2 waves
// per CU at all.  Sweep of two steps, us, as it was (one wave counting) and with 8 / 16 / 32 / 64
// lanes, 2 * 10^7 tokens: K = 100, 332 tokens to a document 7416, 808 / 987 / 1665 / 2968; K = 1000
// 7666, 1390 / 1363 / 1808 / 2951; 10^7 tokens: K = 4000, 330 tokens 4046, 1872 / 1590 / 1385 / 1794;
// 12 tokens, K = 333 2360, 382 / 551 / 937 / 1600; 100 documents of 300 tokens, K = 500 587,
// 213 / 178 / 159 / 152.
// Clearing K counters has to pay: K = 12 000 with documents of 20 tokens 986 without, 1520 with 64
// lanes; of 400 tokens 4318 and 3121; K = 8000, 100 tokens 2605 and 2274.  The line lies at 256
// counters per token of a mean document.
int refresh_lanes(const lda_ctx* c, int32_t longest_doc)
{
    if ((double)c->K * (double)c->D > 256.0 * (double)c->N) return 0;
    // (at most 32 KB: the all-dense store has K <= 12 288, and a document 4096 tokens)
    const size_t bytes = sizeof(int32_t) * (size_t)counts_doc_ints(c->K, longest_doc);
    const size_t lds = 160 * 1024;
    int g = 8;
    while (g < 64 && (lds / (bytes * (size_t)(64 / g)) < 8 || c->D * g / 64 < 512)) g *= 2;
    return g;
}

template <int M, int G>
int launch_refresh_counts_as(lda_ctx* c, const RefreshArgs& A)
{
    const auto kern = sweep_doc_refresh_counts_kernel<M, G>;
    const size_t lds = sizeof(int32_t) * (size_t)(64 / G) * (size_t)A.lds_doc;  // (less than 48 KB)
    hipLaunchKernelGGL(kern, dim3((unsigned)((c->D + 64 / G - 1) / (64 / G))), dim3(64), lds, c->stream, A);
    LDA_HIP(c, hipGetLastError());
    return LDA_OK;
}

template <int G>
int launch_refresh_counts(lda_ctx* c, const RefreshArgs& A, int32_t mh_steps)
{
    if (mh_steps == 1) return launch_refresh_counts_as<1, G>(c, A);
    if (mh_steps == 2) return launch_refresh_counts_as<2, G>(c, A);
    if (mh_steps == 3) return launch_refresh_counts_as<3, G>(c, A);
    return launch_refresh_counts_as<4, G>(c, A);
}

}  // namespace

int refresh_sweep_max_doc() { return kRefreshMaxDoc; }

int launch_sweep_doc_refresh(lda_ctx* c, int32_t mh_steps, int32_t longest_doc)
{
    if (c->hybrid)
        return fail(c, LDA_ERR_UNSUPPORTED, "lda_sweep with doc_refresh needs the all-dense store");
    if (mh_steps > 4)
        return fail(c, LDA_ERR_UNSUPPORTED, "lda_sweep with doc_refresh: at most 4 steps");
    RefreshArgs A{};
    A.word = c->d_word; A.z = c->d_z; A.znew = c->d_znew; A.doff = c->d_doff;
    A.nkw = c->d_nkw; A.nk = c->d_nk; A.alias = c->d_alias; A.cap = c->d_cap;
    A.D = (int32_t)c->D; A.K = c->K; A.mode = c->opt.proposal_mode;
    A.lds_doc = std::max(64, (longest_doc + 63) / 64 * 64);
    A.alpha = c->alpha; A.beta = c->beta; A.alphabar = c->alphabar; A.betabar = c->betabar;
    A.seed_lo = (uint32_t)c->seed; A.seed_hi = (uint32_t)(c->seed >> 32); A.sweep = c->sweep_index;
    const size_t lds = sizeof(int32_t) * (size_t)kRefreshWaves * (size_t)A.lds_doc;
    const dim3 grid((unsigned)((c->D + kRefreshWaves - 1) / kRefreshWaves)), block(64 * kRefreshWaves);
    const int G = refresh_lanes(c, longest_doc);
    if (G > 0) {
        A.lds_counts = counter_ints(c->K);
        A.lds_doc = counts_doc_ints(c->K, longest_doc);
        if (G == 8) return launch_refresh_counts<8>(c, A, mh_steps);
        if (G == 16) return launch_refresh_counts<16>(c, A, mh_steps);
        if (G == 32) return launch_refresh_counts<32>(c, A, mh_steps);
        return launch_refresh_counts<64>(c, A, mh_steps);
    }
#define LDA_REFRESH(M)                                                                              \
    do {                                                                                            \
        if (lds > 48 * 1024)                                                                        \
            LDA_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(sweep_doc_refresh_kernel<M>), \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));  \
        hipLaunchKernelGGL(sweep_doc_refresh_kernel<M>, grid, block, lds, c->stream, A);            \
    } while (0)
    if (mh_steps == 1) LDA_REFRESH(1);
    else if (mh_steps == 2) LDA_REFRESH(2);
    else if (mh_steps == 3) LDA_REFRESH(3);
    else LDA_REFRESH(4);
#undef LDA_REFRESH
    LDA_HIP(c, hipGetLastError());
    return LDA_OK;
}

}  // namespace lda

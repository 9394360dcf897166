// Implied tables (implied.hpp): which words get one, the sums they share, and their build from the
// dense n_kw rows.  All-dense store.
#include <algorithm>

#include "alias_regs.hpp"
#include "common.hpp"
#include "implied.hpp"

namespace lda {

namespace {

// Bins that the words' dense tables must have together; below, one launch for all tables (11 us for
// 5000 words of 100 topics) is as quick as the launches of this form.
constexpr int64_t kImpliedLeastBins = (int64_t)1 << 21;
// A word's table is implied if it has at most K / kImpliedShare tokens (and kImpliedTokens).
constexpr int32_t kImpliedShare = 2;

__device__ __forceinline__ uint64_t quantise40(double a)
{
    return (uint64_t)floor(a * 1099511627776.0);
}

// Shared by all words: q[k] = floor(beta / (n_k + betabar) * 2^40), saturated at 32 bits; pz[k] = sum of
// max(1, q) below k; sum = (sum of the q, sum of max(1, q), largest max(1, q)).  One workgroup, a
// run of consecutive topics per thread.  *n_dense starts the list of dense tables at its fixed part.
constexpr int kSumThreads = 1024;

__global__ __launch_bounds__(kSumThreads) void implied_sums_kernel(const int32_t* __restrict__ nk, int32_t K,
                                                                   double beta, double betabar,
                                                                   uint32_t* __restrict__ qz,
                                                                   uint64_t* __restrict__ pz,
                                                                   uint64_t* __restrict__ sum,
                                                                   int32_t* __restrict__ n_dense, int32_t n_fixed)
{
#pragma clang fp contract(off)
    constexpr int E = kRegsMaxEntries / kSumThreads;
    __shared__ uint64_t w_q0[kMaxWaves], w_q[kMaxWaves], w_max[kMaxWaves];
    const int32_t t = (int32_t)threadIdx.x;
    const int lane = t & (kWave - 1), wv = t >> 6;
    const int32_t R = (K + kSumThreads - 1) / kSumThreads, r0 = t * R;
    int32_t n[E];
    uint64_t q[E], q0s = 0, qs = 0, most = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) n[e] = e < R ? nk[r0 + e < K ? r0 + e : K - 1] : 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        q[e] = 0;
        if (e < R && r0 + e < K) {
            const uint64_t v = quantise40(beta / ((double)n[e] + betabar));
            q0s += v;
            q[e] = v < 1 ? 1 : v;
            qs += q[e];
            most = q[e] > most ? q[e] : most;
            qz[r0 + e] = v > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)v;
        }
    }
    const uint64_t inc = wave_inclusive_scan_u64(qs);
    const uint64_t q0t = wave_total_u64(q0s);
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)most, d, kWave), hi = __shfl_xor((uint32_t)(most >> 32), d, kWave);
        const uint64_t o = ((uint64_t)hi << 32) | lo;
        most = o > most ? o : most;
    }
    if (lane == kWave - 1) { w_q0[wv] = q0t; w_q[wv] = inc; w_max[wv] = most; }
    __syncthreads();
    uint64_t before = inc - qs, q0_all = 0, q_all = 0, max_all = 0;
    for (int i = 0; i < kSumThreads / kWave; ++i) {
        if (i < wv) before += w_q[i];
        q0_all += w_q0[i];
        q_all += w_q[i];
        max_all = w_max[i] > max_all ? w_max[i] : max_all;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e < R && r0 + e < K) {
            pz[r0 + e] = before;
            before += q[e];
        }
    }
    if (t == 0) {
        pz[K] = q_all;
        sum[0] = q0_all;
        sum[1] = q_all;
        sum[2] = max_all;
        *n_dense = n_fixed;
    }
}

struct ImpliedArgs {
    const int32_t* __restrict__ words;
    int32_t n_words, K;
    const int32_t* __restrict__ nkw;
    const int32_t* __restrict__ nk;
    double beta, betabar;
    const uint32_t* __restrict__ qz;
    const uint64_t* __restrict__ sum;
    const uint32_t* __restrict__ off;
    uint4* __restrict__ head;
    uint32_t* __restrict__ key;
    uint64_t* __restrict__ corr;
    uint64_t* __restrict__ x;
    int32_t* __restrict__ dense_words;
    int32_t* __restrict__ n_dense;
    int32_t cap;  // keys of a wave in LDS
};

// A wave per word: its topics out of the dense row, the sums of their weights, and the two running
// sums.  Bound by reading the rows (4 K bytes per word): 137 000 rows of 10 000 counts 1.22 ms, 4.5
// TB/s, where the tables of their bins took 10.6 (16 bytes written per bin).
__global__ __launch_bounds__(256) void implied_tables_kernel(ImpliedArgs a)
{
#pragma clang fp contract(off)
    extern __shared__ uint32_t keys_all[];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int32_t i = (int32_t)blockIdx.x * 4 + wv;
    if (i >= a.n_words) return;
    uint32_t* const keys = keys_all + wv * a.cap;
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t w = a.words[i], K = a.K;
    const int32_t* __restrict__ row = a.nkw + (size_t)w * (size_t)K;
    uint32_t n = 0;
    constexpr int U = 8;  // loads of a lane in flight
    for (int32_t k0 = 0; k0 < K; k0 += U * kWave) {
        int32_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t k = k0 + u * kWave + lane;
            v[u] = row[k < K ? k : K - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t k = k0 + u * kWave + lane;
            const bool has = k < K && v[u] > 0;
            const uint64_t mask = __ballot(has);
            if (mask == 0) continue;
            if (has) keys[n + rank_below(mask)] = ((uint32_t)k << kImpliedTopicShift) | (uint32_t)v[u];
            n += (uint32_t)__popcll(mask);
        }
    }
    wave_lds_order();
    const size_t off = a.off[w];
    auto entry = [&](uint32_t key, uint64_t& q0, uint64_t& z0) {
        const uint32_t t = key >> kImpliedTopicShift;
        q0 = quantise40(((double)(int32_t)(key & kImpliedCount) + a.beta) / ((double)a.nk[t] + a.betabar));
        z0 = a.qz[t];
    };
    uint64_t dq0 = 0, dq = 0;
    for (uint32_t e0 = 0; e0 < n; e0 += kWave) {
        const uint32_t e = e0 + lane;
        if (e < n) {
            uint64_t q0, z0;
            entry(keys[e], q0, z0);
            dq0 += q0 - z0;
            dq += (q0 < 1 ? 1 : q0) - (z0 < 1 ? 1 : z0);
        }
    }
    const uint64_t most = a.sum[2];
    const uint64_t Q0 = a.sum[0] + wave_total_u64(dq0), Q = a.sum[1] + wave_total_u64(dq);
    const uint64_t C = (uint64_t)((double)(Q + (uint64_t)K - 1) / (double)K);  // as in alias_regs.hpp
    const uint64_t pad = (uint64_t)K * C - Q;
    // (q saturates beyond 2^32, but then `most` does not pass)
    const bool fits = most < (1ull << 31) && Q0 < ((uint64_t)K << 31) && most + 1 < C;
    uint64_t c_run = 0, x_run = 0;
    for (uint32_t e0 = 0; e0 < n; e0 += kWave) {
        const uint32_t e = e0 + lane;
        const uint32_t key = e < n ? keys[e] : 0u;
        if (!fits) {  // looked up by topic all the same
            if (e < n) a.key[off + e] = key;
            continue;
        }
        uint64_t cor = 0, exc = 0;
        bool light = false;
        if (e < n) {
            uint64_t q0, z0;
            entry(key, q0, z0);
            const uint64_t p = (key >> kImpliedTopicShift) < pad ? 1 : 0;
            const uint64_t m = (q0 < 1 ? 1 : q0) + p, mz = (z0 < 1 ? 1 : z0) + p;
            light = m < C;
            cor = light ? m - mz : C - mz;
            exc = light ? 0 : m - C;
        }
        const uint64_t ci = wave_inclusive_scan_u64(cor), xi = wave_inclusive_scan_u64(exc);
        if (e < n) {
            a.key[off + e] = key | (light ? kImpliedLight : 0u);
            a.corr[off + e] = c_run + ci;
            a.x[off + e] = x_run + xi;
        }
        c_run += readlane_u64(ci, kWave - 1);
        x_run += readlane_u64(xi, kWave - 1);
    }
    if (lane == 0) {
        if (fits) {
            a.head[w] = make_uint4(n, (uint32_t)C, (uint32_t)pad, 0u);
        } else {
            a.head[w] = make_uint4(n | kImpliedDense, 0u, 0u, 0u);
            a.dense_words[atomicAdd(a.n_dense, 1)] = w;
        }
    }
}

}  // namespace

// Classes by the tokens of a word, which bound its topics: the LDS of a wave's keys.
static constexpr int32_t kImpliedClassCap[lda_ctx::kImpliedClasses] = {256, kImpliedTokens};

int setup_implied(lda_ctx* c, const std::vector<int32_t>& woff)
{
    const int32_t V = c->V, K = c->K;
    const bool two_pass = c->opt.proposal_mode != 2 &&
                          (c->chunk_tokens + c->sweep_block - 1) / c->sweep_block <= 4;
    if (c->hybrid || c->opt.doc_refresh || c->opt.stream_block_tokens > 0 || !two_pass) return LDA_OK;
    const int32_t most = std::min(kImpliedTokens, K / kImpliedShare);
    std::vector<int32_t> words[lda_ctx::kImpliedClasses], fixed;
    std::vector<uint32_t> off((size_t)V + 1);
    std::vector<uint8_t> form((size_t)V);
    uint64_t entries = 0;
    int64_t n = 0;
    for (int32_t w = 0; w < V; ++w) {
        const int32_t cw = woff[w + 1] - woff[w];
        off[w] = (uint32_t)entries;
        form[w] = cw == 0 ? 2 : (cw <= most ? 1 : 0);
        if (form[w] == 0) fixed.push_back(w);
        if (form[w] != 1) continue;
        words[cw <= kImpliedClassCap[0] ? 0 : 1].push_back(w);
        entries += (uint64_t)cw;
        ++n;
    }
    off[V] = (uint32_t)entries;
    if (n * K < kImpliedLeastBins) return LDA_OK;
    std::vector<int32_t> all(words[0]);
    all.insert(all.end(), words[1].begin(), words[1].end());
    fixed.resize((size_t)(c->n_dense_fixed = (int32_t)fixed.size()) + all.size());
    LDA_ALLOC(c, &c->d_im_words, all.size(), "implied tables");
    LDA_ALLOC(c, &c->d_im_off, off.size(), "implied tables");
    LDA_ALLOC(c, &c->d_im_head, (size_t)V, "implied tables");
    LDA_ALLOC(c, &c->d_im_key, entries, "implied tables");
    LDA_ALLOC(c, &c->d_im_corr, entries, "implied tables");
    LDA_ALLOC(c, &c->d_im_x, entries, "implied tables");
    LDA_ALLOC(c, &c->d_im_qz, (size_t)K, "implied tables");
    LDA_ALLOC(c, &c->d_im_pz, (size_t)K + 1, "implied tables");
    LDA_ALLOC(c, &c->d_im_sum, 3, "implied tables");
    LDA_ALLOC(c, &c->d_dense_words, fixed.size(), "implied tables");
    LDA_ALLOC(c, &c->d_n_dense, 1, "implied tables");
    LDA_HIP(c, hipMemcpy(c->d_im_words, all.data(), sizeof(int32_t) * all.size(), hipMemcpyHostToDevice));
    LDA_HIP(c, hipMemcpy(c->d_im_off, off.data(), sizeof(uint32_t) * off.size(), hipMemcpyHostToDevice));
    LDA_HIP(c, hipMemcpy(c->d_dense_words, fixed.data(), sizeof(int32_t) * fixed.size(), hipMemcpyHostToDevice));
    LDA_HIP(c, hipMemset(c->d_im_head, 0, sizeof(uint4) * (size_t)V));  // words without tokens
    for (int i = 0; i < lda_ctx::kImpliedClasses; ++i) c->n_im_class[i] = (int32_t)words[i].size();
    c->n_implied = (int32_t)n;
    c->h_table_form = std::move(form);
    return LDA_OK;
}

// The implied tables, and in d_dense_words the list of the words that have dense ones
int launch_implied_tables(lda_ctx* c)
{
    hipLaunchKernelGGL(implied_sums_kernel, dim3(1), dim3(kSumThreads), 0, c->stream, c->d_nk, c->K, c->beta,
                       c->betabar, c->d_im_qz, c->d_im_pz, c->d_im_sum, c->d_n_dense, c->n_dense_fixed);
    LDA_HIP(c, hipGetLastError());
    ImpliedArgs a{};
    a.K = c->K; a.nkw = c->d_nkw; a.nk = c->d_nk; a.beta = c->beta; a.betabar = c->betabar;
    a.qz = c->d_im_qz; a.sum = c->d_im_sum; a.off = c->d_im_off; a.head = c->d_im_head; a.key = c->d_im_key;
    a.corr = c->d_im_corr; a.x = c->d_im_x; a.dense_words = c->d_dense_words; a.n_dense = c->d_n_dense;
    a.words = c->d_im_words;
    for (int i = 0; i < lda_ctx::kImpliedClasses; ++i) {
        a.n_words = c->n_im_class[i];
        a.cap = kImpliedClassCap[i];
        if (a.n_words > 0)
            hipLaunchKernelGGL(implied_tables_kernel, dim3((a.n_words + 3) / 4), dim3(256),
                               sizeof(uint32_t) * 4 * (size_t)a.cap, c->stream, a);
        LDA_HIP(c, hipGetLastError());
        a.words += a.n_words;
    }
    return LDA_OK;
}

}  // namespace lda

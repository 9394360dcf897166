// Implied tables (implied.hpp): which words get one, the sums they share, the words' lists out of the
// word-major assignment, and the tables out of the lists or, where those are kept, the n_kw rows.
// All-dense store.
#include <algorithm>
#include <cmath>

#include "alias_regs.hpp"
#include "common.hpp"
#include "implied.hpp"
#include "loglik_terms.hpp"

namespace lda {

namespace {

// Bins that the words' dense tables must have together; below, one launch for all tables (11 us for
// 5000 words of 100 topics) is as quick as the launches of this form.
// (Six iterations of 3.1 * 10^5 tokens, 7600 words, K = 544, 4 * 10^6 bins: 0.62 ms with bins, 0.75 implied;
// of 1.8 * 10^6, 30 011 words, K = 333, 10^7 bins, five iterations: 1.12 and 0.94.)
constexpr int64_t kImpliedLeastBins = (int64_t)1 << 23;
static_assert(kImpliedLeastBins / kRegsMaxEntries >= 512, "beta / (V beta) * 2^40 is below 2^31");
// A word's table is implied if it has at most K / kImpliedShare tokens (and kImpliedTokens).
constexpr int32_t kImpliedShare = 2;

__device__ __forceinline__ uint64_t quantise40(double a)
{
    return (uint64_t)floor(a * 1099511627776.0);
}

// Shared by all words: q[k] = floor(beta / (n_k + betabar) * 2^40), below 2^31 as betabar is beta times more than
// 512 words; pz[k] = sum of max(1, q) below k; sum = (sum of the q, sum of max(1, q), largest max(1, q)).  One workgroup, a
// run of consecutive topics per thread.  The lists of misfits start empty.
constexpr int kSumThreads = 1024;

__global__ __launch_bounds__(kSumThreads) void implied_sums_kernel(const int32_t* __restrict__ nk, int32_t K,
                                                                   double beta, double betabar,
                                                                   uint32_t* __restrict__ qz,
                                                                   uint64_t* __restrict__ pz,
                                                                   uint64_t* __restrict__ sum,
                                                                   int32_t* __restrict__ n_misfits)
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
            qz[r0 + e] = (uint32_t)v;
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
    }
    if (t < kMisfitLists) n_misfits[t * kMisfitStride] = 0;
}

// A wave per word: its tokens' topics, ascending, with their counts.  The topics are marked in a
// bitmap of K bits; a topic's place is the number of marks below it.
// (A histogram of K counters per word, written as a row of K counts, took 4 K bytes of LDS and of
// memory for a word however few its tokens: 137 000 words of 1.7 * 10^7 tokens, K = 10 000, 1.0 ms; lists 0.09.)
template <int E>
__global__ __launch_bounds__(256) void implied_lists_kernel(const int32_t* __restrict__ words, int32_t n_words,
                                                            int32_t K, const int32_t* __restrict__ woff,
                                                            const int32_t* __restrict__ zw, int32_t sh,
                                                            uint32_t zmask, const int32_t* __restrict__ xmap,
                                                            const uint32_t* __restrict__ off,
                                                            uint32_t* __restrict__ key, int32_t* __restrict__ n_out)
{
    extern __shared__ uint32_t lds[];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int32_t i = (int32_t)blockIdx.x * 4 + wv;
    if (i >= n_words) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t W = (K + 31) / 32;  // words of the bitmap
    uint32_t* const bits = lds + wv * (2 * W + E * kWave);
    uint32_t* const below = bits + W;  // marks in the words before this one
    uint32_t* const keys = below + W;
    const int32_t w = words[i], b = woff[w], n = woff[w + 1] - b;
    size_t q[E];
    uint32_t t[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int32_t p = b + (e * kWave + lane < n ? e * kWave + lane : n - 1);  // (n >= 1)
        if (e * kWave < n) q[e] = xmap ? (size_t)xmap[p] : (size_t)p;
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e * kWave < n) t[e] = (uint32_t)__builtin_nontemporal_load(&zw[q[e] << sh]) & zmask;
    for (int32_t k = lane; k < W; k += kWave) bits[k] = 0u;
    wave_lds_order();
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e * kWave < n) atomicOr(&bits[t[e] >> 5], 1u << (t[e] & 31u));  // (clones mark the same topic)
    wave_lds_order();
    const int32_t R = (W + kWave - 1) / kWave, k0 = lane * R;
    uint32_t mine = 0;
    for (int32_t k = k0; k < k0 + R && k < W; ++k) mine += (uint32_t)__popc(bits[k]);
    const uint32_t inc = wave_inclusive_scan_u32(mine);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
    uint32_t run = inc - mine;
    for (int32_t k = k0; k < k0 + R && k < W; ++k) {
        below[k] = run;
        run += (uint32_t)__popc(bits[k]);
    }
    wave_lds_order();
    uint32_t at[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e * kWave >= n) continue;
        at[e] = below[t[e] >> 5] + (uint32_t)__popc(bits[t[e] >> 5] & ((1u << (t[e] & 31u)) - 1u));
        keys[at[e]] = t[e] << kImpliedTopicShift;  // the same value from every token of the topic
    }
    wave_lds_order();
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e * kWave + lane < n) atomicAdd(&keys[at[e]], 1u);
    wave_lds_order();
    const size_t o = off[w];
    for (uint32_t k = lane; k < total; k += kWave) key[o + k] = keys[k];
    if (lane == 0) n_out[w] = (int32_t)total;
}

// Dense rows from the lists, a wave per word, unless the rows are kept.
__global__ __launch_bounds__(256) void rows_from_lists_kernel(const int32_t* __restrict__ words, int32_t w0,
                                                              int32_t n_words, int32_t K,
                                                              const uint32_t* __restrict__ off,
                                                              const uint32_t* __restrict__ key,
                                                              const int32_t* __restrict__ n_list,
                                                              int32_t* __restrict__ nkw,
                                                              const int32_t* __restrict__ stale)
{
    if (*stale == 0) return;
    const int32_t i = (int32_t)blockIdx.x * 4 + (int32_t)(threadIdx.x >> 6);
    if (i >= n_words) return;
    const int32_t w = words ? words[i] : w0;
    const int lane = threadIdx.x & (kWave - 1);
    int32_t* const row = nkw + (size_t)w * (size_t)K;
    const uint32_t* __restrict__ mine = key + off[w];
    for (int32_t k = lane; k < K; k += kWave) row[k] = 0;
    // the counts come after the zeros, both of one wave (an agent's fence writes the L2 back: 60 000 rows of
    // 1000 counts 1.87 ms with one, 0.05 so)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    for (int32_t e = lane, n = n_list[w]; e < n; e += kWave)
        row[mine[e] >> kImpliedTopicShift] = (int32_t)(mine[e] & kImpliedCount);
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
    uint32_t* key;
    int32_t* n_list;
    uint64_t* __restrict__ corr;
    uint64_t* __restrict__ x;
    int4* __restrict__ misfits;
    int32_t* __restrict__ n_misfits;
    int32_t first;        // of these words among all, and the room of a list of misfits
    int32_t misfit_words;
    const int32_t* __restrict__ stale;
    int32_t cap;  // keys of a wave in LDS
};

// A wave per word: its topics from the list, or out of the dense row where that is kept, the sums of
// their weights, and the two running sums.  Out of the rows it is bound by reading them: 137 000 rows
// of 10 000 counts 1.22 ms, 4.5 TB/s (the tables of their bins took 10.6, 16 bytes written per bin);
// from lists 0.15 ms.
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
    const size_t off = a.off[w];
    const bool from_list = *a.stale != 0;
    uint32_t n = 0;
    if (from_list) {
        n = (uint32_t)a.n_list[w];
        for (uint32_t e = lane; e < n; e += kWave) keys[e] = a.key[off + e] & ~kImpliedLight;
    } else {
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
        if (lane == 0) a.n_list[w] = (int32_t)n;
    }
    wave_lds_order();
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
    const bool fits = Q0 < ((uint64_t)K << 31) && most + 1 < C;
    if (!fits) {  // its bins are built, and until then drawn from; counts are looked up in the list
        for (uint32_t e = lane; e < n; e += kWave) a.key[off + e] = keys[e];
        if (lane == 0) {
            a.head[w] = make_uint4(n | kImpliedDense, 0u, 0u, 0u);
            a.corr[off] = Q0;  // for the builder of its bins
            a.x[off] = Q;
            const int32_t list = (a.first + i) & (kMisfitLists - 1);
            a.misfits[list * a.misfit_words + atomicAdd(a.n_misfits + list * kMisfitStride, 1)] = make_int4(w, (int32_t)off, (int32_t)n, 0);
        }
        return;
    }
    uint64_t c_run = 0, x_run = 0;
    for (uint32_t e0 = 0; e0 < n; e0 += kWave) {
        const uint32_t e = e0 + lane;
        const uint32_t key = e < n ? keys[e] : 0u;
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
    if (lane == 0) a.head[w] = make_uint4(n, (uint32_t)C, (uint32_t)pad, 0u);
}

// Log-likelihood, word part, of all words of an all-dense store with implied tables: a wave per word,
// over its list, or its row where that is kept (fixed: the words whose row always is).
constexpr int32_t kRowPiece = 2048;

__global__ __launch_bounds__(1024) void loglik_implied_kernel(const int32_t* __restrict__ fixed, int32_t n_fixed,
                                                             const int32_t* __restrict__ words, int32_t n_words,
                                                             int32_t K, const uint32_t* __restrict__ off,
                                                             const uint32_t* __restrict__ key,
                                                             const int32_t* __restrict__ n_list,
                                                             const int32_t* __restrict__ nkw,
                                                             const int32_t* __restrict__ stale, double beta,
                                                             double lg_beta, const double* __restrict__ terms,
                                                             double* __restrict__ partial)
{
    __shared__ double wtot[16];
    __shared__ uint16_t counts[16][kImpliedTokens];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
    const bool lists = *stale != 0;
    double acc = 0.0;
    // a row's pieces of kRowPiece counts are dealt out like words
    const int32_t pieces = (K + kRowPiece - 1) / kRowPiece;
    const int64_t row_pieces = (int64_t)n_fixed * pieces, total = row_pieces + n_words;
    for (int64_t i = (int64_t)blockIdx.x * 16 + wv; i < total; i += (int64_t)gridDim.x * 16) {
        if (i < row_pieces) {
            const int32_t r = (int32_t)(i / pieces), p = (int32_t)(i - (int64_t)r * pieces);
            acc += row_terms<false>(nkw + (size_t)fixed[r] * (size_t)K, p * kRowPiece,
                             K - p * kRowPiece < kRowPiece ? K : (p + 1) * kRowPiece, beta, lg_beta, terms);
            continue;
        }
        const int32_t w = words[i - row_pieces];
        if (lists) {
            const uint32_t* __restrict__ mine = key + off[w];
            const int32_t n = n_list[w];
            for (int32_t e = lane; e < n; e += kWave) acc += terms[mine[e] & kImpliedCount];  // (at most kImpliedTokens)
        } else {
            // the list out of the row first: the same terms in the same order either way
            const int32_t* __restrict__ row = nkw + (size_t)w * (size_t)K;
            uint32_t n = 0;
            wave_lds_order();
            for (int32_t k0 = 0; k0 < K; k0 += 8 * kWave) {
                int32_t v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int32_t k = k0 + u * kWave + lane;
                    v[u] = k < K ? row[k] : 0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint64_t mask = __ballot(v[u] > 0);
                    if (v[u] > 0) counts[wv][n + rank_below(mask)] = (uint16_t)v[u];
                    n += (uint32_t)__popcll(mask);
                }
            }
            wave_lds_order();
            for (uint32_t e = lane; e < n; e += kWave) acc += terms[counts[wv][e]];
        }
    }
    const double s = block_sum_f64(acc, wtot);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

}  // namespace

// Classes by the tokens of a word, which bound its topics: the LDS of a wave's keys.
static constexpr int32_t kImpliedClassCap[lda_ctx::kImpliedClasses] = {256, kImpliedTokens};

template <class T>
static bool take(lda_ctx* c, T** p, size_t n)
{
    *p = static_cast<T*>(try_device_malloc(c, sizeof(T) * n));
    return *p != nullptr;
}

// Without the memory for them (20 bytes per token of their words) every word has its bins; so the caller
// allocates first what a sampler cannot do without.
int setup_implied(lda_ctx* c, const std::vector<int32_t>& woff, const std::vector<RebuildTile>& tiles)
{
    const int32_t V = c->V, K = c->K;
    const bool two_pass = c->opt.proposal_mode != 2 &&
                          (c->chunk_tokens + c->sweep_block - 1) / c->sweep_block <= 4;
    if (c->hybrid || c->opt.doc_refresh || c->opt.stream_block_tokens > 0 || !two_pass) return LDA_OK;
    const int32_t most = std::min(kImpliedTokens, K / kImpliedShare);
    // A word fits the form if its capacity, some (tokens + K beta) / K of a bin's share, exceeds every
    // mass of a topic without tokens.  With topics as even as a random assignment leaves them, four
    // standard deviations, words with fewer tokens than this do not, and get their bins from the rows as
    // other words do; sizes that drift apart are allowed for with a factor of 2.5.  (4.3 * 10^5 tokens, 22 500
    // words, K = 1734, half of the words of up to four tokens: five iterations 1.75 ms with bins, 2.14 with all
    // words tried.)
    const double topic = (double)c->N / (double)K, spread = 4.0 * std::sqrt(topic);
    const double least = 2.5 * (double)K * c->beta * spread / std::max(topic - spread + c->betabar, 1e-300);
    std::vector<int32_t> words[lda_ctx::kImpliedClasses], fixed;
    std::vector<uint32_t> off((size_t)V + 1);
    std::vector<uint8_t> form((size_t)V);
    uint64_t entries = 0;
    int64_t n = 0;
    for (int32_t w = 0; w < V; ++w) {
        const int32_t cw = woff[w + 1] - woff[w];
        off[w] = (uint32_t)entries;
        form[w] = cw == 0 ? 2 : (cw <= most && topic > spread && (double)cw >= least ? 1 : 0);
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
    c->h_table_form = std::move(form);
    std::vector<int4> pieces, others;
    list_implied_pieces(c, woff, pieces, others);
    std::vector<RebuildTile> row_tiles;
    for (const RebuildTile& t : tiles)
        if (c->h_table_form[t.w] == 0) row_tiles.push_back(t);
    c->n_wide_row_tiles = wide_tiles_first(K, row_tiles);
    c->n_row_tiles = (int32_t)row_tiles.size();
    c->n_fixed_words = (int32_t)fixed.size();
    c->n_im_pieces = (int32_t)pieces.size();
    c->n_other_pieces = (int32_t)others.size();
    for (int i = 0; i < lda_ctx::kImpliedClasses; ++i) c->n_im_class[i] = (int32_t)words[i].size();
    const bool room =
        take(c, &c->d_im_words, all.size()) && take(c, &c->d_im_n, (size_t)V) && take(c, &c->d_rows_stale, 1) &&
        take(c, &c->d_im_off, off.size()) && take(c, &c->d_im_head, (size_t)V) && take(c, &c->d_im_key, entries) &&
        take(c, &c->d_im_corr, entries) && take(c, &c->d_im_x, entries) && take(c, &c->d_im_qz, (size_t)K) &&
        take(c, &c->d_im_pz, (size_t)K + 1) && take(c, &c->d_im_sum, 3) && take(c, &c->d_fixed_words, fixed.size()) &&
        take(c, &c->d_misfits, (size_t)misfit_list_words((int32_t)n) * kMisfitLists) &&
        take(c, &c->d_n_misfits, kMisfitLists * kMisfitStride) && take(c, &c->d_im_pieces, pieces.size()) &&
        take(c, &c->d_other_pieces, others.size()) && take(c, &c->d_row_tiles, row_tiles.size());
    if (!room) {
        free_implied(c);
        return LDA_OK;
    }
    auto upload = [](auto* to, const auto& from) {
        return from.empty() ? hipSuccess : hipMemcpy(to, from.data(), sizeof(from[0]) * from.size(), hipMemcpyHostToDevice);
    };
    LDA_HIP(c, upload(c->d_im_words, all));
    LDA_HIP(c, upload(c->d_im_off, off));
    LDA_HIP(c, upload(c->d_fixed_words, fixed));
    LDA_HIP(c, upload(c->d_im_pieces, pieces));
    LDA_HIP(c, upload(c->d_other_pieces, others));
    LDA_HIP(c, upload(c->d_row_tiles, row_tiles));
    // words without tokens
    LDA_HIP(c, hipMemsetAsync(c->d_im_head, 0, sizeof(uint4) * (size_t)V, c->stream));
    LDA_HIP(c, hipMemsetAsync(c->d_im_n, 0, sizeof(int32_t) * (size_t)V, c->stream));
    LDA_HIP(c, hipMemsetAsync(c->d_rows_stale, 0, sizeof(int32_t), c->stream));
    // The recounts that make lists write no rows of words without tokens; the tables over all K bins are
    // built from those rows too.
    LDA_HIP(c, hipMemsetAsync(c->d_nkw, 0, sizeof(int32_t) * (size_t)V * (size_t)K, c->stream));
    c->n_implied = (int32_t)n;
    return LDA_OK;
}

void free_implied(lda_ctx* c)
{
    auto give = [c](auto*& p) {
        device_free(c, p);
        p = nullptr;
    };
    give(c->d_im_words); give(c->d_im_n); give(c->d_rows_stale); give(c->d_im_off); give(c->d_im_head);
    give(c->d_im_key); give(c->d_im_corr); give(c->d_im_x); give(c->d_im_qz); give(c->d_im_pz); give(c->d_im_sum);
    give(c->d_fixed_words); give(c->d_misfits); give(c->d_n_misfits); give(c->d_im_pieces); give(c->d_other_pieces);
    give(c->d_row_tiles);
    c->n_implied = 0;
    c->h_table_form.clear();
    c->implied_built = false;
}

// Where a sweep finds no room for its records: every word has its bins from now on, as in a sampler that
// never had room for the lists.  Refused while a graph may use them.
int give_up_implied(lda_ctx* c)
{
    if (c->implied_in_graph) return LDA_ERR_OOM;
    const int rc = have_all_dense_tables(c);  // and the rows
    if (rc != LDA_OK) return rc;
    LDA_HIP(c, hipStreamSynchronize(c->stream));
    free_implied(c);
    return LDA_OK;
}

// The implied tables, and in d_misfits the list of the words that have dense ones after all
int launch_implied_tables(lda_ctx* c)
{
    hipLaunchKernelGGL(implied_sums_kernel, dim3(1), dim3(kSumThreads), 0, c->stream, c->d_nk, c->K, c->beta,
                       c->betabar, c->d_im_qz, c->d_im_pz, c->d_im_sum, c->d_n_misfits);
    LDA_HIP(c, hipGetLastError());
    ImpliedArgs a{};
    a.K = c->K; a.nkw = c->d_nkw; a.nk = c->d_nk; a.beta = c->beta; a.betabar = c->betabar;
    a.qz = c->d_im_qz; a.sum = c->d_im_sum; a.off = c->d_im_off; a.head = c->d_im_head; a.key = c->d_im_key;
    a.corr = c->d_im_corr; a.x = c->d_im_x; a.misfits = c->d_misfits; a.n_misfits = c->d_n_misfits;
    a.words = c->d_im_words; a.n_list = c->d_im_n; a.stale = c->d_rows_stale;
    a.misfit_words = misfit_list_words(c->n_implied);
    for (int i = 0; i < lda_ctx::kImpliedClasses; ++i) {
        a.n_words = c->n_im_class[i];
        a.cap = kImpliedClassCap[i];
        if (a.n_words > 0)
            hipLaunchKernelGGL(implied_tables_kernel, dim3((a.n_words + 3) / 4), dim3(256),
                               sizeof(uint32_t) * 4 * (size_t)a.cap, c->stream, a);
        LDA_HIP(c, hipGetLastError());
        a.words += a.n_words;
        a.first += a.n_words;
    }
    return LDA_OK;
}

int launch_implied_lists(lda_ctx* c)
{
    const int32_t* words = c->d_im_words;
    for (int i = 0; i < lda_ctx::kImpliedClasses; ++i) {
        const int32_t n = c->n_im_class[i];
        const size_t lds = sizeof(uint32_t) * 4 * (size_t)(2 * ((c->K + 31) / 32) + kImpliedClassCap[i]);  // < 32 KB
        auto kern = i == 0 ? implied_lists_kernel<kImpliedClassCap[0] / kWave> : implied_lists_kernel<kImpliedClassCap[1] / kWave>;
        if (n > 0)
            hipLaunchKernelGGL(kern, dim3((n + 3) / 4), dim3(256), lds, c->stream, words, n, c->K, c->d_woff, c->d_zt,
                               c->zt_shift, c->zt_mask, c->d_xmap, c->d_im_off, c->d_im_key, c->d_im_n);
        LDA_HIP(c, hipGetLastError());
        words += n;
    }
    return LDA_OK;
}

int launch_rows_from_lists(lda_ctx* c, int32_t w)
{
    const int32_t n = w < 0 ? c->n_implied : 1;
    hipLaunchKernelGGL(rows_from_lists_kernel, dim3((n + 3) / 4), dim3(256), 0, c->stream,
                       w < 0 ? c->d_im_words : nullptr, w, n, c->K, c->d_im_off, c->d_im_key, c->d_im_n, c->d_nkw,
                       c->d_rows_stale);
    LDA_HIP(c, hipGetLastError());
    return LDA_OK;
}

int launch_loglik_implied(lda_ctx* c, double lg_beta, const double* terms, int blocks, double* partial)
{
    hipLaunchKernelGGL(loglik_implied_kernel, dim3(blocks), dim3(1024), 0, c->stream, c->d_fixed_words,
                       c->n_fixed_words, c->d_im_words, c->n_implied, c->K, c->d_im_off, c->d_im_key, c->d_im_n,
                       c->d_nkw, c->d_rows_stale, c->beta, lg_beta, terms, partial);
    LDA_HIP(c, hipGetLastError());
    return LDA_OK;
}

}  // namespace lda

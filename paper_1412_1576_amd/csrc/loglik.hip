// Log-likelihood log p(w, z | alpha, beta) of the collapsed LDA model, the
// convergence metric of LightLDA Sec. 7 (doc-likelihood + word-likelihood):
//   doc  = sum_d [ lgG(K a) - lgG(L_d + K a) + sum_{k: n_kd>0} (lgG(n_kd + a) - lgG(a)) ]
//   word = sum_k [ lgG(V b) - lgG(n_k + V b) ] + sum_{w,k: n_kw>0} (lgG(n_kw + b) - lgG(b))
// fp64 throughout; every block reduces in a fixed tree and writes one partial,
// the host adds the partials in index order with compensation.  Which slot of a document's
// hash table a topic lands in depends on the order in which the threads' inserts win, so the
// doc part is summed per token instead of per slot: the term of (document, topic) is added
// by the first token of the document that has the topic.  Every run adds the same terms in
// the same order and returns the same bits.
#include <algorithm>
#include <mutex>

#include "common.hpp"
#include "doc_tile.hpp"
#include "loglik_terms.hpp"

namespace lda {

namespace {

__global__ __launch_bounds__(256) void term_table_kernel(double a, double lg_a, double* __restrict__ table)
{
    const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < kTermTable) table[v] = lgamma((double)v + a) - lg_a;
}

static_assert(kMaxTileTokens < kTermTable, "a count of a document tile is in the table");

// doc part over LDS document tiles: one partial per tile.  (1.9 * 10^6 tokens in documents of 170, K = 500:
// 36 us with hash tables, 19 with counters.)
__global__ __launch_bounds__(1024) void loglik_doc_tiles_kernel(
    const int32_t* __restrict__ z, const int32_t* __restrict__ doff,
    const int32_t* __restrict__ chunk_doc, const uint8_t* __restrict__ tokdoc, int32_t cap_tokens,
    int32_t cap_docs, double alpha, double alphabar, double lg_alpha, double lg_alphabar,
    const double* __restrict__ terms, double* __restrict__ partial, int32_t words)
{
    extern __shared__ int32_t smem[];
    __shared__ double wtot[16];
    const int32_t c = blockIdx.x;
    const int32_t d0 = chunk_doc[c], d1 = chunk_doc[c + 1];
    double acc = 0.0;
    if (words > 0 && doff[d1] - doff[d0] <= cap_tokens) {
        // K counters of 16 bits per document (`words` ints) fit the tile: summed in their order
        const int32_t tok0 = doff[d0], n = doff[d1] - tok0, nd = d1 - d0;
        for (int32_t i = threadIdx.x; i < nd * words; i += blockDim.x) smem[i] = 0;
        __syncthreads();
        for (int32_t i = threadIdx.x; i < n; i += blockDim.x) {
            const int32_t k = z[tok0 + i];
            atomicAdd(&smem[(int32_t)tokdoc[tok0 + i] * words + (k >> 1)], 1 << (16 * (k & 1)));
        }
        __syncthreads();
        for (int32_t i = threadIdx.x; i < nd; i += blockDim.x)
            acc += lg_alphabar - lgamma((double)(doff[d0 + i + 1] - doff[d0 + i]) + alphabar);
        for (int32_t i = threadIdx.x; i < nd * words; i += blockDim.x) {
            const uint32_t v = (uint32_t)smem[i];
            if (v & 0xFFFFu) acc += terms[v & 0xFFFFu];  // (at most kMaxTileTokens)
            if (v >> 16) acc += terms[v >> 16];
        }
    } else if (doff[d1] - doff[d0] <= cap_tokens) {
        const DocTile T = load_doc_tile(smem, cap_tokens, z, doff, tokdoc, d0, d1);
        // first[s] = the lowest token of the tile whose topic sits in slot s
        int32_t* first = smem + doc_tile_lds_bytes(cap_tokens, cap_docs) / sizeof(int32_t);
        for (int32_t i = threadIdx.x; i < 2 * T.ntok; i += blockDim.x) first[i] = 0x7FFFFFFF;
        __syncthreads();
        auto slot_of = [&](int32_t i) {
            const int32_t dl = tokdoc ? (int32_t)tokdoc[T.tok0 + i] : find_doc(T.sdoff, T.nd, i);
            return 2 * T.sdoff[dl] + (int32_t)(T.zs[i] >> kTopicBits);
        };
        for (int32_t i = threadIdx.x; i < T.ntok; i += blockDim.x) atomicMin(&first[slot_of(i)], i);
        __syncthreads();
        for (int32_t i = threadIdx.x; i < T.nd; i += blockDim.x)
            acc += lg_alphabar - lgamma((double)(T.sdoff[i + 1] - T.sdoff[i]) + alphabar);
        for (int32_t i = threadIdx.x; i < T.ntok; i += blockDim.x) {
            const int32_t s = slot_of(i);
            if (first[s] == i) acc += terms[T.tab[s] >> kTopicBits];  // (at most kMaxTileTokens)
        }
    }
    const double s = block_sum_f64(acc, wtot);
    if (threadIdx.x == 0) partial[c] = s;
}

__global__ __launch_bounds__(1024) void loglik_long_docs_kernel(
    const int32_t* __restrict__ z, const int32_t* __restrict__ doff,
    const int32_t* __restrict__ long_doc, const int64_t* __restrict__ long_slot, int32_t* keys,
    int32_t* cnts, int32_t* first_all, double alpha, double alphabar, double lg_alpha,
    double lg_alphabar, const double* __restrict__ terms, double* __restrict__ partial)
{
    __shared__ double wtot[16];
    const int32_t d = long_doc[blockIdx.x];
    const int32_t tok0 = doff[d];
    const int32_t L = doff[d + 1] - tok0;
    const int64_t s0 = long_slot[blockIdx.x];
    const GlobalDocTable tab = load_long_doc(keys + s0, cnts + s0, z + tok0, L);
    // first[s] = the lowest token of the document whose topic sits in slot s
    int32_t* first = first_all + s0;
    for (uint32_t i = threadIdx.x; i < tab.slots; i += blockDim.x)
        __hip_atomic_store(&first[i], 0x7FFFFFFF, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    for (int32_t i = threadIdx.x; i < L; i += blockDim.x) atomicMin(&first[tab.slot_of(z[tok0 + i])], i);
    __syncthreads();
    double acc = 0.0;
    if (threadIdx.x == 0) acc += lg_alphabar - lgamma((double)L + alphabar);
    for (int32_t i = threadIdx.x; i < L; i += blockDim.x) {
        const uint32_t s = tab.slot_of(z[tok0 + i]);
        if (GlobalDocTable::ld(&first[s]) == i)
            acc += count_term(GlobalDocTable::ld(&tab.cnts[s]), alpha, lg_alpha, terms);
    }
    const double s = block_sum_f64(acc, wtot);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// the same with K counters in LDS (K <= kLongDocTopics), summed by topic
__global__ __launch_bounds__(1024) void loglik_long_counters_kernel(
    const int32_t* __restrict__ z, const int32_t* __restrict__ doff, const int32_t* __restrict__ long_doc,
    int32_t K, double alpha, double alphabar, double lg_alpha, double lg_alphabar,
    const double* __restrict__ terms, double* __restrict__ partial)
{
    extern __shared__ int32_t smem[];
    __shared__ double wtot[16];
    const int32_t d = long_doc[blockIdx.x];
    const int32_t tok0 = doff[d], L = doff[d + 1] - tok0;
    count_long_doc(smem, K, z + tok0, L);
    double acc = 0.0;
    if (threadIdx.x == 0) acc += lg_alphabar - lgamma((double)L + alphabar);
    for (int32_t k = threadIdx.x; k < K; k += blockDim.x) {
        const int32_t v = smem[k];
        if (v > 0) acc += count_term(v, alpha, lg_alpha, terms);
    }
    const double s = block_sum_f64(acc, wtot);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// word part: grid-stride over the dense table, one partial per block; a thread adds its terms in
// the order of their places, eight counts in flight.  Bound by reading the rows: 2.7 * 10^7 counts
// (108 MB) took 97 us with an lgamma per non-zero.  With the table, and one copy and one wait for
// all partial sums instead of four, a likelihood of 1.9 * 10^6 tokens at K = 500 costs 0.12 ms less.
__global__ __launch_bounds__(256) void loglik_word_kernel(const int32_t* __restrict__ nkw,
                                                          int64_t total, double beta,
                                                          double lg_beta,
                                                          const double* __restrict__ terms,
                                                          double* __restrict__ partial)
{
    __shared__ double wtot[4];
    double acc = 0.0;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 7 * step < total; i += 8 * step) {
        int32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = nkw[i + u * step];
        acc = add_terms<8>(acc, v, beta, lg_beta, terms);
    }
    for (; i < total; i += step) {
        const int32_t v = nkw[i];
        if (v > 0) acc += count_term(v, beta, lg_beta, terms);
    }
    const double s = block_sum_f64(acc, wtot);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void loglik_nk_kernel(const int32_t* __restrict__ nk, int32_t K,
                                                        double betabar, double lg_betabar,
                                                        double* __restrict__ partial)
{
    __shared__ double wtot[4];
    double acc = 0.0;
    for (int32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < K; k += gridDim.x * blockDim.x)
        acc += lg_betabar - lgamma((double)nk[k] + betabar);
    const double s = block_sum_f64(acc, wtot);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// word part of a store with lists: a wave per piece of a row or per kListGroup words, grid-stride; the words
// of `rows` over their dense rows, those of `lists` over their lists, which are shorter for words of few
// tokens even where there is a row too.  A group's list bounds are read together, and four lists at a time:
// a wave per word waited for three loads in a row for each of its words, 39 us in all.  (54 000 words of 35 tokens, K = 500: 66 us over all rows, 9 more over the lists without a
// row; so 19.)
constexpr int32_t kRowPiece = 4096;
constexpr int32_t kListGroup = 16;

__global__ __launch_bounds__(256) void loglik_lists_kernel(const int32_t* __restrict__ rows, int32_t n_rows,
                                                           const int32_t* __restrict__ nkw, int32_t K,
                                                           const int32_t* __restrict__ lists, int32_t n_lists,
                                                           const uint32_t* __restrict__ sp_off,
                                                           const int32_t* __restrict__ sp_count,
                                                           const int32_t* __restrict__ sp_nnz,
                                                           double beta, double lg_beta,
                                                           const double* __restrict__ terms,
                                                           double* __restrict__ partial)
{
    __shared__ double wtot[4];
    const int lane = threadIdx.x & (kWave - 1);
    double acc = 0.0;
    // a row's pieces of kRowPiece counts are dealt out like words
    const int32_t pieces = (K + kRowPiece - 1) / kRowPiece;
    const int64_t total = (int64_t)n_rows * pieces + (n_lists + kListGroup - 1) / kListGroup;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < total; i += (int64_t)gridDim.x * 4) {
        if (i < (int64_t)n_rows * pieces) {
            const int32_t r = (int32_t)(i / pieces), p = (int32_t)(i - (int64_t)r * pieces);
            acc += row_terms<true>(nkw + (size_t)rows[r] * (size_t)K, p * kRowPiece,
                             K - p * kRowPiece < kRowPiece ? K : (p + 1) * kRowPiece, beta, lg_beta, terms);
        } else {
            const int32_t j0 = (int32_t)(i - (int64_t)n_rows * pieces) * kListGroup;
            int32_t n_mine = 0, off_mine = 0;  // (list offsets are below 2^31)
            if (lane < kListGroup && j0 + lane < n_lists) {
                const int32_t w = lists[j0 + lane];
                n_mine = sp_nnz[w];
                off_mine = (int32_t)sp_off[w];
            }
            for (int j = 0; j < kListGroup; j += 4) {
                int32_t n[4], v[4];
                const int32_t* cnt[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    n[u] = __builtin_amdgcn_readlane(n_mine, j + u);
                    cnt[u] = sp_count + __builtin_amdgcn_readlane(off_mine, j + u);
                    v[u] = lane < n[u] ? cnt[u][lane] : 0;
                }
                acc = add_terms<4>(acc, v, beta, lg_beta, terms);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    for (int32_t e = lane + kWave; e < n[u]; e += kWave) acc += count_term(cnt[u][e], beta, lg_beta, terms);
            }
        }
    }
    const double s = block_sum_f64(acc, wtot);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// compensated (Neumaier) sum, terms added in the order given
struct CompensatedSum {
    double s = 0.0, comp = 0.0;
    void add(double x)
    {
        const double t = s + x;
        comp += (fabs(s) >= fabs(x)) ? (s - t) + x : (x - t) + s;
        s = t;
    }
    double value() const { return s + comp; }
};

// Scratch of lda_loglik_noalloc: the per-block partial sums of the kernels above.  One copy
// of the array per GPU, at an address that hipGetSymbolAddress reports for the current
// device; host code uses that address, never the array's name.
constexpr size_t kStaticPartials = (size_t)1 << 20;  // 8 MB
static __device__ __align__(256) double g_static_partials[kStaticPartials];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double* g_scratch_ptr[kMaxDevices] = {};

// Device address of g_static_partials on the current device (looked up once per device).
int static_partials(lda_ctx* c, double** out)
{
    int dev = -1;
    LDA_HIP(c, hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(c, LDA_ERR_UNSUPPORTED, "lda_loglik_noalloc: device index %d", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        LDA_HIP(c, hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_partials)));
        if (!p) return fail(c, LDA_ERR_HIP, "lda_loglik_noalloc: no address for the static scratch");
        g_scratch_ptr[dev] = static_cast<double*>(p);
    }
    *out = g_scratch_ptr[dev];
    return LDA_OK;
}

// Partial sums of several kernels side by side in one device buffer: one copy to the host and
// one wait for all of them, as far as the buffer holds them.
class Parts {
public:
    Parts(lda_ctx* c, double* d, size_t cap, double* h, size_t h_cap) : c_(c), d_(d), cap_(cap), h_(h), h_cap_(h_cap) {}
    // room for n partials (n <= cap) whose sum will be added to *into; NULL on an error (rc)
    double* take(size_t n, double* into, int* rc)
    {
        *rc = LDA_OK;
        if (used_ + n > cap_ && (*rc = finish()) != LDA_OK) return nullptr;
        part_[n_parts_++] = Part{used_, n, into};
        used_ += n;
        return d_ + used_ - n;
    }
    // waits for the stream and adds every part's sum, parts and terms in the order they were taken
    int finish()
    {
        size_t i = 0, at = 0;
        CompensatedSum acc;
        for (size_t i0 = 0; i0 < used_; i0 += h_cap_) {
            const size_t m = (used_ - i0 < h_cap_) ? used_ - i0 : h_cap_;
            LDA_HIP(c_, hipMemcpyAsync(h_, d_ + i0, sizeof(double) * m, hipMemcpyDeviceToHost, c_->stream));
            LDA_HIP(c_, hipStreamSynchronize(c_->stream));
            for (size_t j = 0; j < m; ++j) {
                acc.add(h_[j]);
                if (++at == part_[i].n) {
                    *part_[i].into += acc.value();
                    acc = CompensatedSum();
                    at = 0;
                    ++i;
                }
            }
        }
        used_ = 0;
        n_parts_ = 0;
        return LDA_OK;
    }

private:
    struct Part { size_t first, n; double* into; };
    lda_ctx* c_;
    double* d_;
    size_t cap_;
    double* h_;
    size_t h_cap_;
    size_t used_ = 0;
    int n_parts_ = 0;
    Part part_[8];
};

constexpr int kWordBlocks = 4096, kNkBlocks = 64;

// Workgroups of the word part, whose sums the host adds: at most kWordBlocks, one for every 8192 tokens
// (lists) or counts of rows.  By tokens alone, a corpus of few tokens and many rows has too few in flight:
// 10^6 tokens, 10^5 rows of 10 000 counts 1600 us, so 1270; 30 000 rows of 16 000 beside lists 1045, so 730.
int word_blocks(const lda_ctx* c)
{
    const int64_t rows = c->n_implied > 0 ? c->n_fixed_words : (c->hybrid ? c->n_row_words : c->V);
    const int64_t counts = rows * c->K / (c->n_implied > 0 ? 4 : 1);  // (that kernel's have four times the threads)
    return (int)std::min<int64_t>(kWordBlocks, 256 + std::max(c->N, counts) / 8192);
}

// The log-likelihood with the partial sums in d_partial (device memory of cap doubles, at least
// max(n_chunks, n_long, kWordBlocks)) and host staging in `h` (h_cap doubles).
int run_loglik(lda_ctx* c, double* d_partial, size_t cap, double* h, size_t h_cap, double* doc_part,
               double* word_part)
{
    const double lga = lgamma(c->alpha), lgab = lgamma(c->alphabar);
    const double lgb = lgamma(c->beta), lgbb = lgamma(c->betabar);
    double doc = 0.0, word = 0.0;
    double* p;
    int rc;
    Parts parts(c, d_partial, cap, h, h_cap);
    if (c->n_chunks > 0) {
        if (!(p = parts.take((size_t)c->n_chunks, &doc, &rc))) return rc;
        rc = c->streamed ? launch_loglik_doc_streamed(c, p) : launch_loglik_doc_tiles(c, p);
        if (rc != LDA_OK) return rc;
    }
    if (c->n_long > 0) {
        if (!(p = parts.take((size_t)c->n_long, &doc, &rc))) return rc;
        if (c->K <= kLongDocTopics) {
            const size_t lds = sizeof(int32_t) * (size_t)c->K;
            if (lds > 48 * 1024)
                LDA_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(loglik_long_counters_kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
            hipLaunchKernelGGL(loglik_long_counters_kernel, dim3(c->n_long), dim3(1024), lds, c->stream, c->d_z,
                               c->d_doff, c->d_long_doc, c->K, c->alpha, c->alphabar, lga, lgab, c->d_lg_terms, p);
        } else {
            hipLaunchKernelGGL(loglik_long_docs_kernel, dim3(c->n_long), dim3(1024), 0, c->stream,
                               c->d_z, c->d_doff, c->d_long_doc, c->d_long_slot, c->d_long_keys,
                               c->d_long_cnts, c->d_long_first, c->alpha, c->alphabar, lga, lgab, c->d_lg_terms, p);
        }
        LDA_HIP(c, hipGetLastError());
    }
    const double* beta_terms = c->d_lg_terms + kTermTable;
    const int blocks = word_blocks(c);
    if (!(p = parts.take((size_t)blocks, &word, &rc))) return rc;
    if (c->n_implied > 0) {
        if ((rc = launch_loglik_implied(c, lgb, beta_terms, blocks, p)) != LDA_OK) return rc;
    } else if (c->hybrid) {
        hipLaunchKernelGGL(loglik_lists_kernel, dim3(blocks), dim3(256), 0, c->stream, c->d_row_words,
                           c->n_row_words, c->d_nkw, c->K, c->d_sparse_words, c->n_sparse, c->d_sp_off,
                           c->d_sp_count, c->d_sp_nnz, c->beta, lgb, beta_terms, p);
        LDA_HIP(c, hipGetLastError());
    } else {
        hipLaunchKernelGGL(loglik_word_kernel, dim3(blocks), dim3(256), 0, c->stream, c->d_nkw,
                           (int64_t)c->V * c->K, c->beta, lgb, beta_terms, p);
        LDA_HIP(c, hipGetLastError());
    }
    if (!(p = parts.take(kNkBlocks, &word, &rc))) return rc;
    hipLaunchKernelGGL(loglik_nk_kernel, dim3(kNkBlocks), dim3(256), 0, c->stream, c->d_nk, c->K,
                       c->betabar, lgbb, p);
    LDA_HIP(c, hipGetLastError());
    if ((rc = parts.finish()) != LDA_OK) return rc;
    *doc_part = doc;
    *word_part = word;
    return LDA_OK;
}

}  // namespace

// largest number of partial sums one log-likelihood has
size_t loglik_partials(const lda_ctx* c)
{
    return (size_t)c->n_chunks + (size_t)c->n_long + kWordBlocks + kNkBlocks;
}

// the term tables of alpha and beta
int setup_loglik(lda_ctx* c)
{
    LDA_ALLOC(c, &c->d_lg_terms, 2 * kTermTable, "log-likelihood terms");
    const double a[2] = {c->alpha, c->beta};
    for (int i = 0; i < 2; ++i) {
        hipLaunchKernelGGL(term_table_kernel, dim3(kTermTable / 256), dim3(256), 0, c->stream, a[i],
                           lgamma(a[i]), c->d_lg_terms + i * kTermTable);
        LDA_HIP(c, hipGetLastError());
    }
    return LDA_OK;
}

// doc part of the tiles the context's token arrays are bound to: partial[tile]
int launch_loglik_doc_tiles(lda_ctx* c, double* d_partial)
{
    const double lga = lgamma(c->alpha), lgab = lgamma(c->alphabar);
    const size_t lds = doc_tile_lds_bytes(c->chunk_tokens, c->chunk_docs) +
                       sizeof(int32_t) * 2 * (size_t)c->chunk_tokens;
    if (lds > 48 * 1024)
        LDA_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(loglik_doc_tiles_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(loglik_doc_tiles_kernel, dim3(c->n_chunks), dim3(c->sweep_block), lds, c->stream,
                       c->d_z, c->d_doff, c->d_chunk_doc, c->d_tokdoc, c->chunk_tokens, c->chunk_docs,
                       c->alpha, c->alphabar, lga, lgab, c->d_lg_terms, d_partial,
                       c->chunk_direct && c->d_tokdoc ? (c->K + 1) / 2 : 0);
    LDA_HIP(c, hipGetLastError());
    return LDA_OK;
}

int launch_loglik(lda_ctx* c, double* doc_part, double* word_part)
{
    std::vector<double> h((size_t)c->n_partial);
    return run_loglik(c, c->d_partial, (size_t)c->n_partial, h.data(), h.size(), doc_part, word_part);
}

}  // namespace lda

using namespace lda;

extern "C" int lda_loglik_noalloc(lda_ctx* c, double* total, double* doc_part, double* word_part)
{
    if (!c) return LDA_ERR_ARG;
    if (!total) return fail(c, LDA_ERR_ARG, "lda_loglik_noalloc: total is NULL");
    if (c->state != COUNTS_VALID && c->state != ALIAS_VALID)
        return fail(c, LDA_ERR_STATE, "lda_loglik_noalloc: counts are stale (call lda_rebuild_counts)");
    const size_t need = (size_t)std::max(std::max(c->n_chunks, c->n_long), 4096);
    if (need > kStaticPartials)
        return fail(c, LDA_ERR_UNSUPPORTED,
                    "lda_loglik_noalloc: %zu partial sums (one per document tile) exceed the static "
                    "scratch of %zu; use lda_loglik", need, kStaticPartials);
    double* scratch = nullptr;
    int rc = static_partials(c, &scratch);
    if (rc != LDA_OK) return rc;
    double staging[2048];  // host side: on the stack
    double d = 0.0, w = 0.0;
    rc = run_loglik(c, scratch, kStaticPartials, staging, sizeof(staging) / sizeof(staging[0]), &d, &w);
    if (rc != LDA_OK) return rc;
    if (doc_part) *doc_part = d;
    if (word_part) *word_part = w;
    *total = d + w;
    return LDA_OK;
}

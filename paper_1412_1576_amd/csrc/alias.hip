// Word-proposal tables (LightLDA Sec. 4.2, Eq. 6, Fig. 2).
//
// Dense form: one table per word over all K topics, weights (n_kw + beta)/(n_k + betabar).
// Mixture form (the paper's sparsified table): per word a table over its non-zero
// topics only, weights n_kw/(n_k + betabar), plus one table shared by all words over
// beta/(n_k + betabar); the sweep picks the term by the two integer masses QS_w and QB.
// Tables whose lists fit LDS are built by a wave or a workgroup each (alias_regs.hpp), larger
// ones by many workgroups each (alias_split.hpp).
#include <algorithm>

#include "alias_build.hpp"
#include "alias_regs.hpp"
#include "alias_split.hpp"
#include "implied.hpp"

namespace lda {

namespace {

__device__ __forceinline__ uint64_t quantise40(double a)
{
    return (uint64_t)floor(a * 1099511627776.0);
}

// dense form: entry k is topic k.  A bin also carries the word-topic counts of its two outcomes,
// so the sweep's accept test needs no second gather.
struct DenseIo {
    static constexpr bool kListed = false, kMassesFirst = true;
    const int32_t* __restrict__ row;
    const int32_t* __restrict__ nk;
    double beta, betabar;
    uint4* __restrict__ out;
    struct Raw { int32_t count, nk; };
    struct Loaded { int32_t other; };
    __device__ __forceinline__ Raw load(int32_t k) const { return Raw{row[k], nk[k]}; }
    __device__ __forceinline__ void load2(Raw&) const {}
    __device__ __forceinline__ uint64_t q0(const Raw& r) const
    {
#pragma clang fp contract(off)
        return quantise40(((double)r.count + beta) / ((double)r.nk + betabar));
    }
    __device__ __forceinline__ Loaded load(int32_t, uint32_t al, const Raw&) const { return Loaded{row[al]}; }
    __device__ __forceinline__ void store(int32_t k, uint32_t split, uint32_t al, const Raw& r,
                                          const Loaded& v) const
    {
        out[k] = make_uint4(split, al, (uint32_t)r.count, (uint32_t)v.other);
    }
};

// The same table from the word's list (implied.hpp) and the masses of topics without tokens; the row
// only exists in LDS.
struct DenseListIo {
    static constexpr bool kListed = true, kMassesFirst = false;
    const uint32_t* __restrict__ key;
    int32_t n_key;
    const uint64_t *__restrict__ sum0, *__restrict__ sum;
    const uint32_t* __restrict__ qz;
    const int32_t* __restrict__ nk;
    double beta, betabar;
    uint4* __restrict__ out;
    mutable const int32_t* row;
    struct Raw { int32_t count; };
    struct Loaded { int32_t other; };
    __device__ __forceinline__ uint64_t Q0() const { return *sum0; }
    __device__ __forceinline__ uint64_t Q() const { return *sum; }
    __device__ __forceinline__ uint64_t weight(int32_t count, int32_t k) const
    {
#pragma clang fp contract(off)
        return quantise40(((double)count + beta) / ((double)nk[k] + betabar));
    }
    __device__ __forceinline__ uint64_t mass(int32_t k) const { return qz[k]; }
    __device__ __forceinline__ void patch(uint64_t* m, int32_t t, int32_t threads) const
    {
        for (int32_t i = t; i < n_key; i += threads) {
            const uint32_t v = key[i];
            const int32_t k = (int32_t)(v >> kImpliedTopicShift);
            m[k] = weight((int32_t)(v & kImpliedCount), k);
        }
    }
    __device__ __forceinline__ void clear(int32_t* r, int32_t n, int32_t t, int32_t threads) const
    {
        row = r;
        for (int32_t k = t; k < n; k += threads) r[k] = 0;
    }
    __device__ __forceinline__ void fill(int32_t* r, int32_t t, int32_t threads) const
    {
        for (int32_t i = t; i < n_key; i += threads) {
            const uint32_t v = key[i];
            r[v >> kImpliedTopicShift] = (int32_t)(v & kImpliedCount);
        }
    }
    __device__ __forceinline__ Raw load(int32_t k) const { return Raw{row[k]}; }
    __device__ __forceinline__ Loaded load(int32_t, uint32_t al, const Raw&) const { return Loaded{row[al]}; }
    __device__ __forceinline__ void store(int32_t k, uint32_t split, uint32_t al, const Raw& r,
                                          const Loaded& v) const
    {
        out[k] = make_uint4(split, al, (uint32_t)r.count, (uint32_t)v.other);
    }
};

// sparse term of the mixture: entry i is the word's i-th non-zero topic (ascending); its bin
// carries the topics and counts of both outcomes
struct MixIo {
    static constexpr bool kListed = false, kMassesFirst = false;
    const int32_t* __restrict__ topic;
    const int32_t* __restrict__ count;
    const int32_t* __restrict__ nk;
    double betabar;
    uint4* __restrict__ out;
    struct Raw { int32_t topic, count, nk; };
    struct Loaded { int32_t topic, count; };
    __device__ __forceinline__ Raw load(int32_t i) const { return Raw{topic[i], count[i], 0}; }
    __device__ __forceinline__ void load2(Raw& r) const { r.nk = nk[r.topic]; }
    __device__ __forceinline__ uint64_t q0(const Raw& r) const
    {
#pragma clang fp contract(off)
        return quantise40((double)r.count / ((double)r.nk + betabar));
    }
    __device__ __forceinline__ Loaded load(int32_t, uint32_t al, const Raw&) const
    {
        return Loaded{topic[al], count[al]};
    }
    __device__ __forceinline__ void store(int32_t i, uint32_t split, uint32_t, const Raw& r,
                                          const Loaded& v) const
    {
        out[i] = pack_mix_bin(split, r.topic, v.topic, r.count, v.count);
    }
};

// shared beta term of the mixture: entry k is topic k
struct BetaIo {
    static constexpr bool kListed = false, kMassesFirst = false;
    const int32_t* __restrict__ nk;
    double beta, betabar;
    uint2* __restrict__ out;
    struct Raw { int32_t nk; };
    struct Loaded {};
    __device__ __forceinline__ Raw load(int32_t k) const { return Raw{nk[k]}; }
    __device__ __forceinline__ void load2(Raw&) const {}
    __device__ __forceinline__ uint64_t q0(const Raw& r) const
    {
#pragma clang fp contract(off)
        return quantise40(beta / ((double)r.nk + betabar));
    }
    __device__ __forceinline__ Loaded load(int32_t, uint32_t, const Raw&) const { return Loaded{}; }
    __device__ __forceinline__ void store(int32_t k, uint32_t split, uint32_t al, const Raw&,
                                          const Loaded&) const
    {
        out[k] = make_uint2(split, al);
    }
};

struct DenseArgs {
    const int32_t* words;  // NULL: word = block index
    int32_t n_words;
    const int32_t* nkw;
    const int32_t* nk;
    int32_t K;
    double beta, betabar;
    uint4* alias;
    uint32_t* cap;   // nullable
    uint4* metaA;    // nullable; word w at [2w]
    // words whose tables are made from lists (n_words is the most there can be): the lengths of kMisfitLists
    // lists of them, the lists, and the room of each
    const int32_t* n_dev;
    const int4* misfits;
    int32_t misfit_words;
    const uint32_t* key;
    const uint64_t *sum0, *sum;  // sums of the weights, in the place of a list's running sums
    const uint32_t* qz;
    uint32_t lds_stride;  // bytes of list memory per wave of a workgroup whose waves build a table each
};

__device__ __forceinline__ void dense_done(const DenseArgs& a, int32_t w, uint32_t C)
{
    if (a.cap) a.cap[w] = C;
    if (a.metaA) a.metaA[2 * (size_t)w] = make_uint4((uint32_t)a.K, C, 0u, 0u);
}

// Tables in LDS: one workgroup per word, or (ONE) one wave per word.
template <int E, bool ONE, int MAXB>
__global__ __launch_bounds__(MAXB) void alias_dense_lds_kernel(DenseArgs a)
{
    extern __shared__ unsigned char smem_raw[];
    const int wv = ONE ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    const int32_t i = ONE ? (int32_t)(blockIdx.x * (blockDim.x >> 6)) + wv : (int32_t)blockIdx.x;
    if (ONE && i >= a.n_words) return;
    const int32_t w = a.words ? a.words[i] : i;
    const int32_t* row = a.nkw + (size_t)w * (size_t)a.K;
    const DenseIo io{row, a.nk, a.beta, a.betabar, a.alias + (size_t)w * (size_t)a.K};
    uint64_t Q0;
    uint32_t C;
    build_table_regs<E, ONE>(a.K, io, io, smem_raw + (size_t)wv * a.lds_stride, Q0, C);
    if ((threadIdx.x & (ONE ? kWave - 1 : 1023)) == 0) dense_done(a, w, C);
}

// The same for the words whose sums did not fit the implied form, from their lists.  Only the device
// knows how many there are, so the workgroups loop.
static_assert(kMisfitLists == kWave, "a lane per list");
template <int E, bool ONE, int MAXB>
__global__ __launch_bounds__(MAXB, MAXB == 256 ? 8 : 1) void alias_dense_list_kernel(DenseArgs a)
{
    extern __shared__ unsigned char smem_raw[];
    const int wv = ONE ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    const int32_t step = ONE ? (int32_t)(gridDim.x * (blockDim.x >> 6)) : (int32_t)gridDim.x;
    // the lists' words count through: those of list l end before `upto`
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t mine = a.n_dev[lane * kMisfitStride];
    const int32_t upto = (int32_t)wave_inclusive_scan_u32((uint32_t)mine);
    const int32_t n = __builtin_amdgcn_readlane(upto, kWave - 1);
    const int32_t base = lane * a.misfit_words - (upto - mine);  // of the list's words, less those before it
    auto misfit = [&](int32_t j) {
        const uint64_t after = __ballot(upto > j);  // (j < n: some list's)
        return a.misfits[j + __builtin_amdgcn_readlane(base, __ffsll((unsigned long long)after) - 1)];
    };
    int32_t i = ONE ? (int32_t)(blockIdx.x * (blockDim.x >> 6)) + wv : (int32_t)blockIdx.x;
    if (i >= n) return;
    int4 next = misfit(i);
    for (; i < n; i += step) {
        const int32_t w = next.x;  // (word, list offset, entries)
        const size_t off = (uint32_t)next.y;
        const int32_t n_key = next.z;
        next = misfit(i + step < n ? i + step : i);
        // a fresh K every time, or the compiler keeps what it derives from it in registers over the
        // loop (128 instead of 86 VGPRs at E = 12, and spills: twice the time)
        int32_t K = a.K;
        asm volatile("" : "+s"(K));
        const DenseListIo io{a.key + off, n_key, a.sum0 + off, a.sum + off, a.qz, a.nk, a.beta, a.betabar,
                             a.alias + (size_t)w * (size_t)K, nullptr};
        uint64_t Q0;
        uint32_t C;
        build_table_regs<E, ONE>(K, io, io, smem_raw + (size_t)wv * a.lds_stride, Q0, C);
        if ((threadIdx.x & (ONE ? kWave - 1 : 1023)) == 0) dense_done(a, w, C);
        if constexpr (ONE) wave_lds_order(); else __syncthreads();  // before the lists are written again
    }
}

// the same tables for the builder of alias_split.hpp
struct DenseTables {
    DenseArgs a;
    __device__ __forceinline__ int32_t word(int32_t i) const { return a.words ? a.words[i] : i; }
    __device__ __forceinline__ int32_t entries(int32_t) const { return a.K; }
    __device__ __forceinline__ DenseIo io(int32_t i) const
    {
        const size_t wk = (size_t)word(i) * (size_t)a.K;
        return DenseIo{a.nkw + wk, a.nk, a.beta, a.betabar, a.alias + wk};
    }
    __device__ __forceinline__ void done(int32_t i, int32_t, uint64_t, uint32_t C) const { dense_done(a, word(i), C); }
};

struct MixArgs {
    const int32_t* words;
    int32_t n_words;
    const uint32_t* sp_off;
    const int32_t* sp_topic;
    const int32_t* sp_count;
    const int32_t* sp_nnz;
    const int32_t* nk;
    double betabar;
    uint4* ma;
    uint4* metaA;
    uint32_t lds_stride;
};

template <int E, bool ONE, int MAXB>
__global__ __launch_bounds__(MAXB) void alias_mix_lds_kernel(MixArgs a)
{
    extern __shared__ unsigned char smem_raw[];
    const int wv = ONE ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    const int32_t i = ONE ? (int32_t)(blockIdx.x * (blockDim.x >> 6)) + wv : (int32_t)blockIdx.x;
    if (ONE && i >= a.n_words) return;
    const int32_t w = a.words[i];
    const int32_t n = a.sp_nnz[w];
    const bool first = (threadIdx.x & (ONE ? kWave - 1 : 1023)) == 0;
    if (n <= 0) {  // a word without tokens is never drawn from
        if (first) a.metaA[2 * (size_t)w] = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    const size_t off = a.sp_off[w];
    const MixIo io{a.sp_topic + off, a.sp_count + off, a.nk, a.betabar, a.ma + off};
    uint64_t QS;
    uint32_t C;
    build_table_regs<E, ONE>(n, io, io, smem_raw + (size_t)wv * a.lds_stride, QS, C);
    if (first)
        a.metaA[2 * (size_t)w] = make_uint4((uint32_t)n, C, (uint32_t)QS, (uint32_t)(QS >> 32));
}

struct MixTables {
    MixArgs a;
    __device__ __forceinline__ int32_t entries(int32_t i) const { return a.sp_nnz[a.words[i]]; }
    __device__ __forceinline__ MixIo io(int32_t i) const
    {
        const size_t off = a.sp_off[a.words[i]];
        return MixIo{a.sp_topic + off, a.sp_count + off, a.nk, a.betabar, a.ma + off};
    }
    __device__ __forceinline__ void done(int32_t i, int32_t n, uint64_t Q0, uint32_t C) const
    {
        a.metaA[2 * (size_t)a.words[i]] = make_uint4((uint32_t)n, C, (uint32_t)Q0, (uint32_t)(Q0 >> 32));
    }
};

template <int E, bool ONE, int MAXB>
__global__ __launch_bounds__(MAXB) void alias_beta_lds_kernel(const int32_t* nk, int32_t K, double beta,
                                                              double betabar, uint2* out, uint64_t* hdr)
{
    extern __shared__ unsigned char smem_raw[];
    const BetaIo io{nk, beta, betabar, out};
    uint64_t QB;
    uint32_t C;
    build_table_regs<E, ONE>(K, io, io, smem_raw, QB, C);
    if (threadIdx.x == 0) {
        hdr[0] = QB;
        hdr[1] = C;
    }
}

struct BetaTables {
    const int32_t* nk;
    int32_t K;
    double beta, betabar;
    uint2* out;
    uint64_t* hdr;
    __device__ __forceinline__ int32_t entries(int32_t) const { return K; }
    __device__ __forceinline__ BetaIo io(int32_t) const { return BetaIo{nk, beta, betabar, out}; }
    __device__ __forceinline__ void done(int32_t, int32_t, uint64_t Q0, uint32_t C) const
    {
        hdr[0] = Q0;
        hdr[1] = C;
    }
};

// Non-zero topics of a dense row, ascending, into the word's list (a mixture word
// that keeps a dense row).  One workgroup per word; every wave owns a contiguous run of
// topics, counts its non-zeros, and after one barrier places them (the second read of the
// run comes from L2).  Four loads per lane are in flight.
__global__ __launch_bounds__(1024) void compact_rows_kernel(const int32_t* __restrict__ words,
                                                            const int32_t* __restrict__ nkw,
                                                            int32_t K,
                                                            const uint32_t* __restrict__ sp_off,
                                                            int32_t* __restrict__ sp_topic,
                                                            int32_t* __restrict__ sp_count,
                                                            int32_t* __restrict__ sp_nnz)
{
    __shared__ uint32_t wcnt[16];
    const int32_t w = words[blockIdx.x];
    const int32_t* __restrict__ row = nkw + (size_t)w * (size_t)K;
    const size_t off = sp_off[w];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
    const int nw = blockDim.x >> 6;
    const int32_t chunk = (((K + nw - 1) / nw) + kWave - 1) & ~(kWave - 1);
    const int32_t kb0 = (wv * chunk < K) ? wv * chunk : K;
    const int32_t kb1 = (kb0 + chunk < K) ? kb0 + chunk : K;
    uint32_t cnt = 0;
    int32_t kb = kb0;
    for (; kb + 4 * kWave <= kb1; kb += 4 * kWave) {
        int32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = row[kb + u * kWave + lane];
#pragma unroll
        for (int u = 0; u < 4; ++u) cnt += (uint32_t)__popcll(__ballot(v[u] > 0));
    }
    for (; kb < kb1; kb += kWave) {
        const int32_t k = kb + lane;
        const int32_t v = (k < kb1) ? row[k] : 0;
        cnt += (uint32_t)__popcll(__ballot(v > 0));
    }
    if (lane == 0) wcnt[wv] = cnt;
    __syncthreads();
    uint32_t pos = 0, total = 0;
    for (int i = 0; i < nw; ++i) {
        if (i < wv) pos += wcnt[i];
        total += wcnt[i];
    }
    auto place = [&](int32_t k, int32_t v) {
        const uint64_t mask = __ballot(v > 0);
        if (v > 0) {
            const size_t p = off + pos + rank_below(mask);
            sp_topic[p] = k;
            sp_count[p] = v;
        }
        pos += (uint32_t)__popcll(mask);
    };
    kb = kb0;
    for (; kb + 4 * kWave <= kb1; kb += 4 * kWave) {
        int32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = row[kb + u * kWave + lane];
#pragma unroll
        for (int u = 0; u < 4; ++u) place(kb + u * kWave + lane, v[u]);
    }
    for (; kb < kb1; kb += kWave) {
        const int32_t k = kb + lane;
        place(k, (k < kb1) ? row[k] : 0);
    }
    if (threadIdx.x == 0) sp_nnz[w] = (int32_t)total;
}

template <class Kern>
int set_lds(lda_ctx* c, Kern kern, size_t lds)
{
    if (lds > 48 * 1024)
        LDA_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    return LDA_OK;
}

// How a table of at most n entries (n <= kRegsMaxEntries) is built: E entries per thread; up to
// 256 entries by one wave, four such tables per workgroup, larger ones by a whole workgroup.
struct TableShape {
    int e;        // entries per thread: 1, 4 (one wave); 4, 8, 12 (workgroup)
    bool one;
    int threads;  // per workgroup
};

TableShape table_shape(int32_t n)
{
    if (n <= kWave) return {1, true, 256};
    if (n <= 4 * kWave) return {4, true, 256};
    if (n <= 1024) return {4, false, (n + 4 * kWave - 1) / (4 * kWave) * kWave};
    if (n <= 8192) return {8, false, (n + 8 * kWave - 1) / (8 * kWave) * kWave};
    return {12, false, 1024};
}

// calls f(E, ONE, MAXB) with the template arguments of a shape
template <int V>
struct IntConst { static constexpr int value = V; };
template <class F>
int with_shape(const TableShape& s, F&& f)
{
    if (s.one) return s.e == 1 ? f(IntConst<1>{}, IntConst<1>{}, IntConst<256>{}) : f(IntConst<4>{}, IntConst<1>{}, IntConst<256>{});
    if (s.e == 4) return f(IntConst<4>{}, IntConst<0>{}, IntConst<256>{});
    if (s.e == 8) return f(IntConst<8>{}, IntConst<0>{}, IntConst<1024>{});
    return f(IntConst<12>{}, IntConst<0>{}, IntConst<1024>{});
}

int launch_dense_lds(lda_ctx* c, DenseArgs a)
{
    if (a.n_words <= 0) return LDA_OK;
    const TableShape s = table_shape(a.K);
    const int per = s.one ? s.threads / kWave : 1;  // tables per workgroup
    a.lds_stride = (uint32_t)alias_regs_lds_bytes((size_t)a.K);
    const size_t lds = (size_t)a.lds_stride * (size_t)per;
    return with_shape(s, [&](auto e, auto one, auto maxb) -> int {
        constexpr int E = decltype(e)::value, MAXB = decltype(maxb)::value;
        constexpr bool ONE = decltype(one)::value != 0;
        auto kern = a.n_dev ? alias_dense_list_kernel<E, ONE, MAXB> : alias_dense_lds_kernel<E, ONE, MAXB>;
        const int rc = set_lds(c, kern, lds);
        if (rc != LDA_OK) return rc;
        int32_t blocks = (a.n_words + per - 1) / per;
        if (a.n_dev) {  // as many as the chip holds
            const int32_t most = std::min<int32_t>(2048 / s.threads, (int32_t)(163840 / (lds + 1024)));
            blocks = std::min(blocks, 256 * std::max(1, most));
        }
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(s.threads), lds, c->stream, a);
        LDA_HIP(c, hipGetLastError());
        return LDA_OK;
    });
}

// the five launches of alias_split.hpp for every batch of the set
template <class Tables>
int launch_big_tables(lda_ctx* c, hipStream_t stream, const BigSet& set, const Tables& tab)
{
    BigWork W{};
    W.chunks = set.d_chunks; W.first = set.d_first; W.list = set.d_list; W.sums = set.d_sums;
    W.state = set.d_state; W.dx = set.dx; W.hidx = set.hidx;
    for (size_t b = 0; b + 1 < set.batch_chunk.size(); ++b) {
        W.c0 = set.batch_chunk[b];
        const dim3 grid(set.batch_chunk[b + 1] - W.c0), block(kBigThreads);
        hipLaunchKernelGGL(big_mass_kernel<Tables>, grid, block, 0, stream, tab, W);
        hipLaunchKernelGGL(big_shift_kernel<Tables>, grid, block, 0, stream, tab, W);
        hipLaunchKernelGGL(big_counts_kernel<Tables>, grid, block, 0, stream, tab, W);
        hipLaunchKernelGGL(big_lists_kernel<Tables>, grid, block, 0, stream, tab, W);
        hipLaunchKernelGGL(big_pairs_kernel<Tables>, grid, block, 0, stream, tab, W);
        LDA_HIP(c, hipGetLastError());
    }
    return LDA_OK;
}

// Chunks and batches of the tables with the given largest numbers of entries: a batch's lists
// fit `room` list entries (a single table always does).  Returns the list entries needed.
template <class Entries>
int setup_big_set(lda_ctx* c, BigSet* set, size_t n_tables, Entries entries, uint64_t room, uint64_t* need)
{
    *need = 0;
    if (n_tables == 0) return LDA_OK;
    std::vector<int2> chunks;
    std::vector<uint32_t> first;
    std::vector<uint64_t> list;
    uint64_t used = 0;
    set->batch_chunk.assign(1, 0u);
    for (size_t t = 0; t < n_tables; ++t) {
        const int32_t n = entries(t);
        if (used > 0 && used + (uint64_t)n + 1 > room) {
            set->batch_chunk.push_back((uint32_t)chunks.size());
            used = 0;
        }
        list.push_back(used);
        used += (uint64_t)n + 1;
        *need = std::max(*need, used);
        first.push_back((uint32_t)chunks.size());
        for (int32_t k = 0; k < n; k += kBigChunk) chunks.push_back(make_int2((int32_t)t, k));
    }
    set->batch_chunk.push_back((uint32_t)chunks.size());
    LDA_ALLOC(c, &set->d_chunks, chunks.size(), "table chunks");
    LDA_ALLOC(c, &set->d_first, first.size(), "table chunks");
    LDA_ALLOC(c, &set->d_list, list.size(), "table chunks");
    LDA_ALLOC(c, &set->d_sums, chunks.size(), "table chunks");
    LDA_ALLOC(c, &set->d_state, n_tables, "table chunks");
    LDA_HIP(c, hipMemcpy(set->d_chunks, chunks.data(), sizeof(int2) * chunks.size(), hipMemcpyHostToDevice));
    LDA_HIP(c, hipMemcpy(set->d_first, first.data(), sizeof(uint32_t) * first.size(), hipMemcpyHostToDevice));
    LDA_HIP(c, hipMemcpy(set->d_list, list.data(), sizeof(uint64_t) * list.size(), hipMemcpyHostToDevice));
    return LDA_OK;
}

void free_big_set(lda_ctx* c, BigSet& s)
{
    device_free(c, s.d_chunks);
    device_free(c, s.d_first);
    device_free(c, s.d_list);
    device_free(c, s.d_sums);
    device_free(c, s.d_state);
    s = BigSet{};
}

}  // namespace

// Work lists and list memory of the tables built by many workgroups each: the dense tables and
// the shared beta table when K exceeds one workgroup's LDS, and the mixture words of `big_mix`.
// Dense and mixture tables follow each other on one stream and share their list memory; the
// beta table is built beside them and has its own.
int setup_big_tables(lda_ctx* c, const std::vector<int32_t>& big_mix)
{
    const int32_t K = c->K;
    const bool big_k = K > kRegsMaxEntries;
    // Room of a batch: 340 tables of K entries (4 KB K bytes, 4.3 GB for the largest K) fill the chip
    // many times over -- at the smallest K it is 2000 chunks -- and keep the lists small beside
    // the tables.
    const uint64_t room = 340ull * (uint64_t)K;
    uint64_t need_dense = 0, need_mix = 0, need_beta = 0;
    int rc = setup_big_set(c, &c->big_dense, big_k ? (size_t)c->n_dense_alias : 0,
                           [&](size_t) { return K; }, room, &need_dense);
    if (rc != LDA_OK) return rc;
    rc = setup_big_set(c, &c->big_mix, big_mix.size(), [&](size_t i) {
        const int32_t w = big_mix[i];
        return (int32_t)(c->h_sp_off[w + 1] - c->h_sp_off[w]);
    }, room, &need_mix);
    if (rc != LDA_OK) return rc;
    rc = setup_big_set(c, &c->big_beta, big_k && c->n_mix > 0 ? 1 : 0, [&](size_t) { return K; }, room, &need_beta);
    if (rc != LDA_OK) return rc;
    const uint64_t main = std::max(need_dense, need_mix);
    if (main + need_beta == 0) return LDA_OK;
    LDA_ALLOC(c, &c->d_big_dx, main + need_beta, "table workspace");
    LDA_ALLOC(c, &c->d_big_hidx, main + need_beta, "table workspace");
    c->big_dense.dx = c->big_mix.dx = c->d_big_dx;
    c->big_dense.hidx = c->big_mix.hidx = c->d_big_hidx;
    c->big_beta.dx = c->d_big_dx + main;
    c->big_beta.hidx = c->d_big_hidx + main;
    return LDA_OK;
}

void free_big_tables(lda_ctx* c)
{
    free_big_set(c, c->big_dense);
    free_big_set(c, c->big_mix);
    free_big_set(c, c->big_beta);
    device_free(c, c->d_big_dx);
    device_free(c, c->d_big_hidx);
    c->d_big_dx = nullptr;
    c->d_big_hidx = nullptr;
}

int max_lds_table_entries() { return kRegsMaxEntries; }
int max_alias_topics() { return kRegsMaxEntries; }

// all-dense mode: every word, lists in LDS
int launch_alias_build(lda_ctx* c)
{
    const int32_t K = c->K;
    if (K > max_lds_table_entries())
        return fail(c, LDA_ERR_UNSUPPORTED, "dense alias build in LDS supports K <= %d",
                    max_lds_table_entries());
    DenseArgs a{};
    a.words = nullptr; a.n_words = c->V; a.nkw = c->d_nkw; a.nk = c->d_nk; a.K = K;
    a.beta = c->beta; a.betabar = c->betabar; a.alias = c->d_alias; a.cap = c->d_cap;
    a.metaA = nullptr;
    return launch_dense_lds(c, a);
}

int launch_dense_listed(lda_ctx* c)
{
    DenseArgs a{};
    a.words = c->d_fixed_words; a.n_words = c->n_fixed_words;
    a.nkw = c->d_nkw; a.nk = c->d_nk; a.K = c->K; a.beta = c->beta; a.betabar = c->betabar;
    a.alias = c->d_alias; a.cap = c->d_cap;
    const int rc = launch_dense_lds(c, a);
    if (rc != LDA_OK) return rc;
    a.misfits = c->d_misfits; a.misfit_words = misfit_list_words(c->n_implied); a.n_words = c->n_implied; a.n_dev = c->d_n_misfits; a.key = c->d_im_key;
    a.sum0 = c->d_im_corr; a.sum = c->d_im_x; a.qz = c->d_im_qz;
    return launch_dense_lds(c, a);
}

int launch_dense_table(lda_ctx* c, int32_t w)
{
    DenseArgs a{};
    const size_t wk = (size_t)w * (size_t)c->K;
    a.n_words = 1; a.nkw = c->d_nkw + wk; a.nk = c->d_nk; a.K = c->K; a.beta = c->beta; a.betabar = c->betabar;
    a.alias = c->d_alias + wk; a.cap = c->d_cap + w;
    return launch_dense_lds(c, a);
}

// lda_build_alias makes the form that the last sweeps drew from; the bins of all words are made late when
// a sweep of one kernel comes after two-pass ones.
int have_implied_tables(lda_ctx* c)
{
    if (c->implied_built) return LDA_OK;
    int rc = launch_implied_tables(c);
    if (rc == LDA_OK && !c->all_dense_built) rc = launch_dense_listed(c);
    c->implied_built = rc == LDA_OK;
    return rc;
}

int have_all_dense_tables(lda_ctx* c)
{
    if (c->all_dense_built) return LDA_OK;
    int rc = c->n_implied > 0 ? launch_rows_from_lists(c, -1) : LDA_OK;
    if (rc == LDA_OK) rc = launch_alias_build(c);
    c->all_dense_built = rc == LDA_OK;
    return rc;
}

namespace {

// Mixture tables of the words in `words` whose list capacity is at most cap_entries
// (cap_entries = 0: any size, many workgroups each).
int launch_alias_mix_class(lda_ctx* c, hipStream_t stream, const int32_t* words, int32_t n_words,
                           int32_t cap_entries)
{
    if (n_words <= 0) return LDA_OK;
    MixArgs a{};
    a.words = words; a.n_words = n_words; a.sp_off = c->d_sp_off; a.sp_topic = c->d_sp_topic;
    a.sp_count = c->d_sp_count; a.sp_nnz = c->d_sp_nnz; a.nk = c->d_nk; a.betabar = c->betabar;
    a.ma = c->d_ma; a.metaA = c->d_metaA;
    if (cap_entries > 0) {
        const TableShape s = table_shape(cap_entries);
        const int per = s.one ? s.threads / kWave : 1;
        a.lds_stride = (uint32_t)alias_regs_lds_bytes((size_t)cap_entries);
        const size_t lds = (size_t)a.lds_stride * (size_t)per;
        return with_shape(s, [&](auto e, auto one, auto maxb) -> int {
            auto kern = alias_mix_lds_kernel<decltype(e)::value, decltype(one)::value != 0, decltype(maxb)::value>;
            const int rc = set_lds(c, kern, lds);
            if (rc != LDA_OK) return rc;
            hipLaunchKernelGGL(kern, dim3((n_words + per - 1) / per), dim3(s.threads), lds, stream, a);
            LDA_HIP(c, hipGetLastError());
            return LDA_OK;
        });
    }
    return launch_big_tables(c, stream, c->big_mix, MixTables{a});
}

// the shared beta table and the mixture tables that are built in LDS, in this order on `stream`
int launch_small_mixture_tables(lda_ctx* c, hipStream_t stream)
{
    const int32_t K = c->K;
    const int lds_max = max_lds_table_entries();
    int rc;
    if (K <= lds_max) {
        TableShape sh = table_shape(K);
        if (sh.one) sh.threads = kWave;
        const size_t lds = alias_regs_lds_bytes((size_t)K);
        rc = with_shape(sh, [&](auto e, auto one, auto maxb) -> int {
            auto kern = alias_beta_lds_kernel<decltype(e)::value, decltype(one)::value != 0, decltype(maxb)::value>;
            const int r = set_lds(c, kern, lds);
            if (r != LDA_OK) return r;
            hipLaunchKernelGGL(kern, dim3(1), dim3(sh.threads), lds, stream, c->d_nk, K, c->beta, c->betabar,
                               c->d_beta_alias, c->d_beta_hdr);
            return LDA_OK;
        });
        if (rc != LDA_OK) return rc;
        LDA_HIP(c, hipGetLastError());
    } else {
        rc = launch_big_tables(c, stream, c->big_beta,
                               BetaTables{c->d_nk, K, c->beta, c->betabar, c->d_beta_alias, c->d_beta_hdr});
        if (rc != LDA_OK) return rc;
    }
    for (int cl = 0; cl < kMixClasses; ++cl) {
        const int32_t cap = kMixClassCap[cl];
        if (cap < 0) continue;  // the class of any size
        rc = launch_alias_mix_class(c, stream, c->d_mix_class[cl], c->n_mix_class[cl],
                                    cap ? cap : lds_max);
        if (rc != LDA_OK) return rc;
    }
    return LDA_OK;
}

}  // namespace

// Hybrid mode: the shared beta table, dense tables of the head words, mixture tables of the
// rest.  Two chains of kernels run side by side: on a second stream of the library's own the
// beta table and the many small tables built in LDS; on the caller's stream the dense tables
// and the large mixture tables.
// The second stream is forked from the caller's by an event and joined at the end.
int launch_alias_build_hybrid(lda_ctx* c)
{
    const int32_t K = c->K;
    const int lds_max = max_lds_table_entries();
    int rc;
    if (c->n_compact > 0) {  // lists the mixture tables below are built from
        hipLaunchKernelGGL(compact_rows_kernel, dim3(c->n_compact), dim3(K <= 4096 ? 256 : 1024), 0,
                           c->stream, c->d_compact_words, c->d_nkw, K, c->d_sp_off, c->d_sp_topic,
                           c->d_sp_count, c->d_sp_nnz);
        LDA_HIP(c, hipGetLastError());
    }
    if (c->n_mix > 0) {
        if ((rc = fork_side_stream(c)) != LDA_OK) return rc;
        rc = launch_small_mixture_tables(c, c->side_stream);
        const int rd = side_stream_done(c);
        if (rc != LDA_OK || rd != LDA_OK) {
            (void)join_side_stream(c);
            return rc != LDA_OK ? rc : rd;
        }
    }
    if (c->n_dense_alias > 0) {
        DenseArgs a{};
        a.words = c->d_dense_alias_words; a.n_words = c->n_dense_alias; a.nkw = c->d_nkw;
        a.nk = c->d_nk; a.K = K; a.beta = c->beta; a.betabar = c->betabar; a.alias = c->d_alias;
        a.cap = c->d_cap; a.metaA = c->d_metaA;
        if (K <= lds_max) {
            rc = launch_dense_lds(c, a);
        } else {
            rc = launch_big_tables(c, c->stream, c->big_dense, DenseTables{a});
        }
    } else {
        rc = LDA_OK;
    }
    if (rc == LDA_OK)
        rc = launch_alias_mix_class(c, c->stream, c->d_mix_class[kMixClasses - 1],
                                    c->n_mix_class[kMixClasses - 1], 0);
    const int rj = join_side_stream(c);
    return rc != LDA_OK ? rc : rj;
}

}  // namespace lda

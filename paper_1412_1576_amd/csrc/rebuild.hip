// Count rebuild (LightLDA Sec. 3: the sufficient statistics n_kw and n_k).
//
// n_kw: tokens are laid out word-major, so every word's tokens are one
// contiguous segment.  z is first scattered into that order (one random 4-byte
// write per token, cheaper than a 128-byte line per gathered token); a workgroup
// then histograms a tile of a segment in LDS and writes the dense row.  Words whose segment is longer than one tile are split
// over several workgroups whose partial histograms are merged into a
// pre-zeroed row with integer atomics (order-free, hence exact).
// n_k: an LDS-privatised histogram of z over all tokens (for very large K over a copy of z
// partitioned by topic range, sparse_rows.hip).
#include <algorithm>

#include "common.hpp"
#include "xcd.hpp"

namespace lda {

namespace {

// Kernels of a recount that lda_update_counts may or may not want take a device flag: with `go`
// set and *go zero they return at once.
__device__ __forceinline__ bool unwanted(const int32_t* go) { return go && *go == 0; }

// zw[p] = topic of the p-th token in word-major order: zw[wpos[g]] = z[g].
//
// A word's tokens are ordered by document, so while g advances the writes into
// one word's segment are sequential: a 128-byte line of zw is completed by 32
// writes that are close in g.  Workgroups are dealt round-robin to the 8 XCDs,
// each with its own L2; every XCD therefore takes one contiguous eighth of the
// token range and walks it in order, so that the partially written lines of the
// frequent words stay in that XCD's L2 until they are full instead of being
// written back piecemeal by eight caches.
constexpr int kScatterPerThread = 1;
constexpr int kScatterBlock = 1024;

__global__ __launch_bounds__(1024) void scatter_wm_kernel(const int32_t* __restrict__ z,
                                                         const int32_t* __restrict__ wpos,
                                                         int64_t N, int32_t* __restrict__ zw,
                                                         int32_t sh, const int32_t* __restrict__ go)
{
    if (unwanted(go)) return;
    const int64_t per_xcd = (N + kXcds - 1) / kXcds;
    const int xcd = blockIdx.x % kXcds;
    const int64_t j = blockIdx.x / kXcds;
    const int64_t lo = xcd * per_xcd;
    const int64_t hi = (lo + per_xcd < N) ? lo + per_xcd : N;
    const int64_t base = lo + j * (int64_t)(blockDim.x * kScatterPerThread);
#pragma unroll
    for (int u = 0; u < kScatterPerThread; ++u) {
        const int64_t g = base + u * (int64_t)blockDim.x + threadIdx.x;
        if (g < hi)
            zw[(size_t)__builtin_nontemporal_load(&wpos[g]) << sh] = __builtin_nontemporal_load(&z[g]);
    }
}

// blockIdx.x: tile; blockIdx.y: range of `span` topics (one range when the row fits LDS).
// ONE: four short tiles to a workgroup, each a wave's, which meets no barrier (one range).  With
// a workgroup to each of 53 975 words of 35 tokens the launches of the workgroups bounded the
// pass: 76 us.
constexpr int32_t kTileRun = 32;  // consecutive tiles of an XCD, at most
constexpr int32_t kWaveTileTokens = 512, kWaveTileTopics = 2048;

struct TilesArgs {
    const RebuildTile* __restrict__ tiles;
    int32_t n_tiles, run;
    uint32_t n_blocks;  // that have a tile (ONE: four)
    const int32_t* __restrict__ zw;
    int32_t sh;
    uint32_t zmask;
    int32_t K, span;
    int32_t* __restrict__ nkw;
    const uint32_t* __restrict__ sp_off;
    int32_t *__restrict__ sp_topic, *__restrict__ sp_count, *__restrict__ sp_nnz;
    const int32_t* __restrict__ xmap;
    const int32_t* __restrict__ rshift;
    const int32_t* __restrict__ go;
};

template <bool ONE>
__device__ __forceinline__ void nkw_tile(const TilesArgs& A, const RebuildTile t, int32_t* hist, uint32_t* wcnt)
{
    const int32_t* __restrict__ zw = A.zw;
    int32_t* __restrict__ nkw = A.nkw;
    const int32_t shift = A.xmap ? A.rshift[t.w] : 0;
    const int32_t* __restrict__ xmap = shift == kMapped ? A.xmap : nullptr;
    const int32_t K = A.K, span = A.span, sh = A.sh;
    const uint32_t zmask = A.zmask;
    auto sync = [&]() {
        if constexpr (ONE) wave_lds_order(); else __syncthreads();
    };
    const int32_t k0 = (int32_t)blockIdx.y * span;
    const int32_t nk_r = ((k0 + span < K) ? k0 + span : K) - k0;
    const int tid = ONE ? (int)threadIdx.x & 63 : (int)threadIdx.x, nt = ONE ? 64 : (int)blockDim.x;
    auto count = [&](int32_t rec) {
        const uint32_t r = ((uint32_t)rec & zmask) - (uint32_t)k0;
        if (r < (uint32_t)nk_r) atomicAdd(&hist[r], 1);
    };
    auto at = [&](int32_t p) -> size_t { return xmap ? (size_t)xmap[p] : (size_t)(p + shift); };
    int32_t p = t.p0 + tid;
    // The thread's first records are requested before the histogram is cleared: most tiles are
    // short (a word of a thousand tokens), and the clearing and its barrier then hide the two
    // dependent round trips instead of preceding them.  Threads past the end repeat the last.
    int32_t first[2] = {0, 0};
    if (t.p1 > t.p0) {  // (a word without tokens has an empty tile)
        size_t q[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) q[u] = at(p + u * nt < t.p1 ? p + u * nt : t.p1 - 1);
#pragma unroll
        for (int u = 0; u < 2; ++u) first[u] = __builtin_nontemporal_load(&zw[q[u] << sh]);
    }
    for (int32_t k = tid; k < nk_r; k += nt) hist[k] = 0;
    sync();
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (p + u * nt < t.p1) count(first[u]);
    p += 2 * nt;
    for (; p + 3 * nt < t.p1; p += 4 * nt) {  // four loads in flight per thread
        size_t q[4];
        int32_t rec[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = at(p + u * nt);
#pragma unroll
        for (int u = 0; u < 4; ++u) rec[u] = __builtin_nontemporal_load(&zw[q[u] << sh]);
#pragma unroll
        for (int u = 0; u < 4; ++u) count(rec[u]);
    }
    for (; p < t.p1; p += nt) count(zw[at(p) << sh]);
    sync();
    int32_t* __restrict__ row = nkw + (size_t)t.w * (size_t)K + (size_t)k0;
    if (t.multi == 1) {
        for (int32_t k = tid; k < nk_r; k += nt) {
            const int32_t v = hist[k];
            if (v) atomicAdd(&row[k], v);
        }
    } else if (t.multi >= 2) {
        // the whole row is here (one tile, one topic range): write it and the list of its
        // non-zero topics, ascending
        const size_t off = A.sp_off[t.w];
        const int lane = tid & 63, wv = tid >> 6, nw = nt >> 6;
        // every wave owns a contiguous run of topics: count its non-zeros, then place them
        const int32_t chunk = (((nk_r + nw - 1) / nw) + 63) & ~63;
        const int32_t kb0 = wv * chunk;
        const int32_t kb1 = (kb0 + chunk < nk_r) ? kb0 + chunk : nk_r;
        uint32_t cnt = 0;
        for (int32_t kb = kb0; kb < kb1; kb += 64) {
            const int32_t k = kb + lane;
            const int32_t v = (k < kb1) ? hist[k] : 0;
            if (k < kb1 && t.multi == 2) row[k] = v;  // 3: the row is not kept
            cnt += (uint32_t)__popcll(__ballot(v > 0));
        }
        uint32_t base = cnt, pos = 0;
        if constexpr (!ONE) {
            if (lane == 0) wcnt[wv] = cnt;
            __syncthreads();
            base = 0;
            for (int i = 0; i < nw; ++i) {
                if (i < wv) pos += wcnt[i];
                base += wcnt[i];
            }
        }
        for (int32_t kb = kb0; kb < kb1; kb += 64) {
            const int32_t k = kb + lane;
            const int32_t v = (k < kb1) ? hist[k] : 0;
            const uint64_t mask = __ballot(v > 0);
            if (v > 0) {
                const size_t p = off + pos + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
                A.sp_topic[p] = k;
                A.sp_count[p] = v;
            }
            pos += (uint32_t)__popcll(mask);
        }
        if (tid == 0) A.sp_nnz[t.w] = (int32_t)base;
    } else {
        for (int32_t k = tid; k < nk_r; k += nt) row[k] = hist[k];
    }
}

// With `go`, where more than twice kLoopBlocks workgroups may be launched for nothing, that many
// loop over the tiles (LOOP): a workgroup that finds it is not wanted still costs its launch, 1.2 ns of
// the whole chip's time.  lda_update_counts with nothing moved, 2 * 10^7 tokens, us, one workgroup
// per tile (four) / so / the +-1 form alone: 10^5 words, K = 2500 113 / 69 / 53; 4 * 10^5 words,
// K = 300 90 / 69 / 57.  A wanted recount of 5 * 10^6 tokens, 6 * 10^4 words, K = 2500, takes 210
// instead of 190, the others as long as before.  (The scatter of the assignment keeps a workgroup to
// 1024 tokens: four rounds each, or looping workgroups, widen the window of partial lines; 2 * 10^7
// tokens of 10^5 words 285 -> 410 to 490.)
constexpr unsigned kLoopBlocks = 4096;  // a multiple of the XCDs

template <bool ONE, bool LOOP>
__global__ __launch_bounds__(ONE ? 256 : 1024) void nkw_tiles_kernel(TilesArgs A)
{
    extern __shared__ int32_t hist_all[];
    __shared__ uint32_t wcnt[16];
    if (unwanted(A.go)) return;
    // runs of consecutive tiles (neighbouring words) share an XCD and with it the lines of
    // the records they read
    const int wave = ONE ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    int32_t* const hist = hist_all + wave * A.span;
    for (uint32_t b = blockIdx.x; b < A.n_blocks; b += gridDim.x) {
        const int32_t ti = ONE ? 4 * xcd_runs(A.run, b) + wave : xcd_runs(A.run, b);
        if (ti < A.n_tiles) nkw_tile<ONE>(A, A.tiles[ti], hist, wcnt);  // (ONE: uniform over the wave)
        if constexpr (!LOOP) return;
        if constexpr (ONE) wave_lds_order(); else __syncthreads();  // before the histogram is cleared
    }
}

// Rows of more topics than one LDS histogram, of mixture words of at most kListRowTokens tokens: a
// workgroup takes the topic ranges of its word one after the other, so that the list of non-zeros
// comes out of the histograms with the row and no second pass reads the row back.  The word's
// topics are read once and kept in registers.  A histogram takes at most half of the LDS: two
// workgroups share a CU, and one's barriers are hidden by the other's work.
//
// Rows and tables of an iteration, ranges and lists in two passes before / in one here, ms: 6000
// words of 4000 tokens, K = 10^5, 1.96 / 1.18; 600 of them at K = 10^6 1.90 / 0.87.  (Writing only
// the topics of the previous and the new list, for words with few tokens, gained nothing.)
// Longer words would be read again for every range, one range after the other, where
// nkw_tiles_kernel has a workgroup to each range: 40 words of 250 000 tokens, K = 10^6, 1.11
// there and 7.02 in this form; of 16 000 tokens 0.46 and 0.76, 600 of them 2.55 and 2.26.
constexpr int32_t kListRowSpan = 18432;
constexpr int kListRowKept = kListRowTokens / 1024;  // topics of a thread, kept in registers

__global__ __launch_bounds__(1024, 8) void nkw_list_rows_kernel(
    const RebuildTile* __restrict__ tiles, int32_t n_tiles, int32_t run, const int32_t* __restrict__ zw,
    int32_t sh, uint32_t zmask, int32_t K, int32_t span, int32_t* __restrict__ nkw,
    const uint32_t* __restrict__ sp_off, int32_t* __restrict__ sp_topic, int32_t* __restrict__ sp_count,
    int32_t* __restrict__ sp_nnz, const int32_t* __restrict__ xmap)
{
    extern __shared__ int32_t hist[];  // span counters, a multiple of 64
    __shared__ uint32_t wcnt[2][16];
    const int32_t ti = xcd_runs(run);
    if (ti >= n_tiles) return;
    const RebuildTile t = tiles[ti];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const size_t off = sp_off[t.w];
    int32_t* __restrict__ row = nkw + (size_t)t.w * (size_t)K;
    auto topic_at = [&](int32_t p) {
        const size_t q = xmap ? (size_t)xmap[p] : (size_t)p;
        return (uint32_t)__builtin_nontemporal_load(&zw[q << sh]) & zmask;
    };
    uint32_t mine[kListRowKept];
#pragma unroll
    for (int e = 0; e < kListRowKept; ++e) {
        const int32_t p = t.p0 + e * 1024 + tid;
        mine[e] = p < t.p1 ? topic_at(p) : 0xFFFFFFFFu;  // (beyond every range)
    }
    for (int32_t k = 4 * tid; k < span; k += 4096) *reinterpret_cast<int4*>(&hist[k]) = make_int4(0, 0, 0, 0);
    const bool aligned = (K & 3) == 0;
    // every wave owns a contiguous run of a range's topics, four to a lane
    const int32_t chunk = (((span + 15) / 16) + 255) & ~255;
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t total = 0;  // entries of the ranges done
    int parity = 0;
    for (int32_t k0 = 0; k0 < K; k0 += span, parity ^= 1) {
        const uint32_t nk_r = (uint32_t)((k0 + span < K) ? span : K - k0);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kListRowKept; ++e) {
            const uint32_t r = mine[e] - (uint32_t)k0;
            if (r < nk_r) atomicAdd(&hist[r], 1);
        }
        __syncthreads();
        const int32_t kb0 = wv * chunk, kb1 = (kb0 + chunk < span) ? kb0 + chunk : span;
        uint32_t cnt = 0;
        for (int32_t kb = kb0; kb < kb1; kb += 256) {
            const int32_t k = kb + 4 * lane;
            int4 v = make_int4(0, 0, 0, 0);
            if (k < kb1) v = *reinterpret_cast<const int4*>(&hist[k]);
            if (k < (int32_t)nk_r) {
                if (aligned) {
                    *reinterpret_cast<int4*>(&row[k0 + k]) = v;
                } else {
                    row[k0 + k] = v.x;
                    if (k + 1 < (int32_t)nk_r) row[k0 + k + 1] = v.y;
                    if (k + 2 < (int32_t)nk_r) row[k0 + k + 2] = v.z;
                    if (k + 3 < (int32_t)nk_r) row[k0 + k + 3] = v.w;
                }
            }
            cnt += (uint32_t)(__popcll(__ballot(v.x > 0)) + __popcll(__ballot(v.y > 0)) +
                              __popcll(__ballot(v.z > 0)) + __popcll(__ballot(v.w > 0)));
        }
        if (lane == 0) wcnt[parity][wv] = cnt;
        __syncthreads();
        size_t pos = off + total;
        for (int i = 0; i < 16; ++i) {
            const uint32_t n = wcnt[parity][i];
            if (i < wv) pos += n;
            total += n;
        }
        for (int32_t kb = kb0; kb < kb1; kb += 256) {  // places, and clears for the next range
            const int32_t k = kb + 4 * lane;
            int4 v = make_int4(0, 0, 0, 0);
            if (k < kb1) {
                v = *reinterpret_cast<const int4*>(&hist[k]);
                *reinterpret_cast<int4*>(&hist[k]) = make_int4(0, 0, 0, 0);
            }
            const uint64_t m0 = __ballot(v.x > 0), m1 = __ballot(v.y > 0),
                           m2 = __ballot(v.z > 0), m3 = __ballot(v.w > 0);
            if ((m0 | m1 | m2 | m3) == 0) continue;  // uniform over the wave
            size_t p = pos + (uint32_t)(__popcll(m0 & below) + __popcll(m1 & below) + __popcll(m2 & below) +
                                        __popcll(m3 & below));
            const int32_t c[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (c[u] <= 0) continue;
                sp_topic[p] = k0 + k + u;
                sp_count[p] = c[u];
                ++p;
            }
            pos += (uint32_t)(__popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3));
        }
    }
    if (tid == 0) sp_nnz[t.w] = (int32_t)total;
}

// What the counts below add to: the rows of the words of several tiles, a workgroup each, and
// after them n_k, kZeroNk topics to a workgroup.  One launch for both: in a corpus of 10^5 tokens
// a launch is 4 of the 56 us of an iteration.  (And says what this recount leaves of the rows of
// words with implied tables.)
constexpr int32_t kZeroNk = 4096;

__global__ __launch_bounds__(256) void zero_counts_kernel(const int32_t* __restrict__ words, int32_t n_words,
                                                          int32_t K, int32_t* __restrict__ nkw,
                                                          int32_t* __restrict__ nk,
                                                          const int32_t* __restrict__ go,
                                                          int32_t* __restrict__ rows_stale, int32_t stale)
{
    if (unwanted(go)) return;
    const int32_t i = (int32_t)blockIdx.x;
    if (rows_stale && i == 0 && threadIdx.x == 0) *rows_stale = stale;
    if (i < n_words) {
        int32_t* __restrict__ row = nkw + (size_t)words[i] * (size_t)K;
        for (int32_t k = threadIdx.x; k < K; k += blockDim.x) row[k] = 0;
    } else {
        const int32_t k0 = (i - n_words) * kZeroNk, k1 = (K - k0 > kZeroNk) ? k0 + kZeroNk : K;
        for (int32_t k = k0 + threadIdx.x; k < k1; k += blockDim.x) nk[k] = 0;
    }
}

constexpr int32_t kNkRangeTopics = 36864;  // 144 KB of LDS counters per workgroup

// n_k: each block histograms a contiguous slice of z in LDS, then adds its non-zero bins to
// the (pre-zeroed) global row.  For K beyond one LDS histogram blockIdx.y selects a range of
// `span` topics and every range reads all of z.
__global__ __launch_bounds__(1024) void nk_hist_ranges_kernel(const int32_t* __restrict__ z,
                                                              int64_t N, int32_t K, int32_t span,
                                                              int32_t* __restrict__ nk,
                                                              const int32_t* __restrict__ go)
{
    extern __shared__ int32_t hist[];
    if (unwanted(go)) return;
    const int32_t k0 = (int32_t)blockIdx.y * span;
    const int32_t k1 = (k0 + span < K) ? k0 + span : K;
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int32_t k = tid; k < k1 - k0; k += nt) hist[k] = 0;
    __syncthreads();
    // blocks own runs of whole int4s; two int4 loads per thread are in flight together (one
    // dword per thread and iteration left the kernel bound by load latency)
    const int64_t n4 = N / 4;
    const int64_t per = (n4 + gridDim.x - 1) / gridDim.x;
    const int64_t b = (int64_t)blockIdx.x * per;
    const int64_t e = (b + per < n4) ? b + per : n4;
    using v4i = int32_t __attribute__((ext_vector_type(4)));
    const v4i* __restrict__ z4 = reinterpret_cast<const v4i*>(z);
    auto count = [&](int32_t t) {
        if (t >= k0 && t < k1) atomicAdd(&hist[t - k0], 1);
    };
    int64_t i = b + tid;
    for (; i + nt < e; i += 2 * (int64_t)nt) {
        const v4i a = __builtin_nontemporal_load(&z4[i]);
        const v4i c = __builtin_nontemporal_load(&z4[i + nt]);
        count(a.x); count(a.y); count(a.z); count(a.w);
        count(c.x); count(c.y); count(c.z); count(c.w);
    }
    if (i < e) {
        const v4i a = __builtin_nontemporal_load(&z4[i]);
        count(a.x); count(a.y); count(a.z); count(a.w);
    }
    if (blockIdx.x == 0 && tid < (int)(N - 4 * n4)) count(z[4 * n4 + tid]);
    __syncthreads();
    for (int32_t k = tid; k < k1 - k0; k += nt) {
        const int32_t v = hist[k];
        if (v) atomicAdd(&nk[k0 + k], v);
    }
}

// The paper's incremental rule (Sec. 3): a token that moved from topic a to topic b takes one
// from n_kw[w][a], n_k[a] and gives one to n_kw[w][b], n_k[b].  Integer atomics, so the result
// equals the recount whatever the order.  The deltas of n_k are summed per workgroup in LDS
// first (the all-dense store has K <= max_alias_topics()).  Bound by the rate of the atomics on
// n_kw, 5 to 10 moved tokens per ns.  With `recount` set and *recount non-zero it returns at once
// (*copy = *recount for the kernels of the recount).
__global__ __launch_bounds__(1024) void update_counts_kernel(const int32_t* __restrict__ z,
                                                            const int32_t* __restrict__ zprev,
                                                            const int32_t* __restrict__ word,
                                                            int64_t N, int32_t K,
                                                            int32_t* __restrict__ nkw,
                                                            int32_t* __restrict__ nk,
                                                            const int32_t* __restrict__ recount,
                                                            int32_t* __restrict__ copy)
{
    extern __shared__ int32_t dk[];
    if (copy && blockIdx.x == 0 && threadIdx.x == 0) *copy = *recount;
    if (recount && *recount) return;
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int32_t k = tid; k < K; k += nt) dk[k] = 0;
    __syncthreads();
    const int64_t per = (N + gridDim.x - 1) / gridDim.x;
    const int64_t b = (int64_t)blockIdx.x * per;
    const int64_t e = (b + per < N) ? b + per : N;
    for (int64_t g = b + tid; g < e; g += nt) {
        const int32_t to = __builtin_nontemporal_load(&z[g]);
        const int32_t from = __builtin_nontemporal_load(&zprev[g]);
        if (to == from) continue;
        int32_t* __restrict__ row = nkw + (size_t)word[g] * (size_t)K;
        atomicSub(&row[from], 1);
        atomicAdd(&row[to], 1);
        atomicSub(&dk[from], 1);
        atomicAdd(&dk[to], 1);
    }
    __syncthreads();
    for (int32_t k = tid; k < K; k += nt) {
        const int32_t v = dk[k];
        if (v) atomicAdd(&nk[k], v);
    }
}

// Workgroups of a pass over all tokens with K counters of its own each: 65536 tokens per
// workgroup, fewer for a small corpus (down to one 16-byte load per thread) as long as they are
// four times the counters that every workgroup adds to the result.
int64_t hist_blocks(const lda_ctx* c)
{
    const int64_t least = std::max<int64_t>(4096, 4 * (int64_t)c->K);
    const int64_t per = std::min<int64_t>(65536, std::max(least, c->N / 256));
    return (c->N + per - 1) / per;
}

// *recount = 1 if more than `most` of the kMovedSample tokens spread evenly over z have moved, or there
// are rows that +-1 cannot be added to.
// Every sampled token is two cache lines of its own: one workgroup alone took 78 us for them,
// sixteen, a token to a thread, 7.4 us.  *sum collects the workgroups' counts with one count of
// arrivals above them, in one atomic; the last workgroup decides and leaves it zero.
constexpr int32_t kMovedSample = 16384;
constexpr int kArrivalShift = 20;

__global__ __launch_bounds__(1024) void sample_moved_kernel(const int32_t* __restrict__ z,
                                                           const int32_t* __restrict__ zprev, int64_t N,
                                                           int32_t most, int32_t* __restrict__ recount,
                                                           int32_t* __restrict__ sum,
                                                           const int32_t* __restrict__ rows_stale)
{
    __shared__ int32_t moved;
    if (threadIdx.x == 0) moved = 0;
    __syncthreads();
    const int64_t g = ((int64_t)((int)blockIdx.x * 1024 + (int)threadIdx.x) * N) / kMovedSample;
    const uint64_t m = __ballot(z[g] != zprev[g]);
    if ((threadIdx.x & 63) == 0) atomicAdd(&moved, (int32_t)__popcll(m));
    __syncthreads();
    if (threadIdx.x != 0) return;
    const int32_t before = atomicAdd(sum, (1 << kArrivalShift) + moved);
    if ((before >> kArrivalShift) != (int32_t)gridDim.x - 1) return;
    const bool many = (before & ((1 << kArrivalShift) - 1)) + moved > most;
    *recount = many || (rows_stale && *rows_stale) ? 1 : 0;
    *sum = 0;
}

}  // namespace

int max_rebuild_topics() { return 36 * 1024; }

// Tiles that a wave counts by itself: a single tile of its word with at most kWaveTileTokens
// tokens, in a row that 64 lanes clear and write in few steps.
static bool is_wave_tile(int32_t K, const RebuildTile& t)
{
    return t.multi != 1 && K <= kWaveTileTopics && t.p1 - t.p0 <= kWaveTileTokens;
}

int32_t wide_tiles_first(int32_t K, std::vector<RebuildTile>& tiles)
{
    const int32_t n = (int32_t)(std::stable_partition(tiles.begin(), tiles.end(), [K](const RebuildTile& t) {
        return !is_wave_tile(K, t);
    }) - tiles.begin());
    // one launch where both would not fill the chip (10^5 tokens of 1000 words: 6.6 us in one, 8 in two)
    return (int32_t)tiles.size() - n < kWaveTilesLeast ? (int32_t)tiles.size() : n;
}

namespace {

// word-major copy of z, then the dense rows by LDS histograms over topic ranges; n_k is zeroed for
// launch_nk_hist.  lists: the words of implied tables get their lists instead (never with `go`).
int launch_dense_rows(lda_ctx* c, const int32_t* go = nullptr, bool lists = false)
{
    const int32_t K = c->K;
    const RebuildTile* const tiles = lists ? c->d_row_tiles : c->d_tiles;
    const int32_t n_tiles = lists ? c->n_row_tiles : c->n_tiles;
    const int32_t n_wide_tiles = lists ? c->n_wide_row_tiles : c->n_wide_tiles;
    if (!c->zt_current) {  // the sweep's doc pass may have written the new assignment already
        const int rc = launch_scatter_word_major(c, c->d_z, c->d_wpos, c->N, go);
        if (rc != LDA_OK) return rc;
        c->zt_current = !go;  // (the host does not know whether a conditional scatter ran)
        c->td_valid = false;  // any stored doc proposals belong to another assignment
    }
    {
        const int32_t n_nk = K <= 8 * kNkRangeTopics ? (K + kZeroNk - 1) / kZeroNk : 0;
        const int32_t n_rows = c->n_tiles > 0 ? c->n_multi_words : 0;
        if (n_rows + n_nk > 0)
            hipLaunchKernelGGL(zero_counts_kernel, dim3(n_rows + n_nk), dim3(256), 0, c->stream,
                               c->d_multi_words, n_rows, K, c->d_nkw, c->d_nk, go, c->d_rows_stale, lists ? 1 : 0);
        LDA_HIP(c, hipGetLastError());
    }
    if (lists) {
        const int rc = launch_implied_lists(c);
        if (rc != LDA_OK) return rc;
    }
    if (c->n_list_tiles > 0) {
        const int32_t ranges = (K + kListRowSpan - 1) / kListRowSpan;
        const int32_t part = (((K + ranges - 1) / ranges) + 63) / 64 * 64;
        const size_t part_lds = sizeof(int32_t) * (size_t)part;
        LDA_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(nkw_list_rows_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)part_lds));
        const int32_t lrun = xcd_run_length(c->n_list_tiles, kTileRun);
        hipLaunchKernelGGL(nkw_list_rows_kernel, dim3(xcd_runs_grid(c->n_list_tiles, lrun)), dim3(1024),
                           part_lds, c->stream, c->d_list_tiles, c->n_list_tiles, lrun, c->d_zt, c->zt_shift,
                           c->zt_mask, K, part, c->d_nkw, c->d_sp_off, c->d_sp_topic, c->d_sp_count,
                           c->d_sp_nnz, c->d_xmap);
        LDA_HIP(c, hipGetLastError());
    }
    if (n_tiles == 0) return LDA_OK;
    const int32_t nr = (K + max_rebuild_topics() - 1) / max_rebuild_topics();
    const int32_t span = (((K + nr - 1) / nr) + 63) / 64 * 64;
    const size_t lds = sizeof(int32_t) * (size_t)span;
    if (lds > 48 * 1024)  // (looping workgroups: the all-dense store, K <= 12 288)
        LDA_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(nkw_tiles_kernel<false, false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    TilesArgs A{};
    A.zw = c->d_zt; A.sh = c->zt_shift; A.zmask = c->zt_mask; A.K = K; A.span = span; A.nkw = c->d_nkw;
    A.sp_off = c->d_sp_off; A.sp_topic = c->d_sp_topic; A.sp_count = c->d_sp_count; A.sp_nnz = c->d_sp_nnz;
    A.xmap = c->d_xmap; A.rshift = c->d_rshift; A.go = go;
    if (n_wide_tiles > 0) {
        A.tiles = tiles; A.n_tiles = n_wide_tiles;
        A.run = xcd_run_length(A.n_tiles, kTileRun);
        A.n_blocks = xcd_runs_grid(A.n_tiles, A.run);
        const bool loop = go && A.n_blocks > 2 * kLoopBlocks;
        const dim3 grid(loop ? kLoopBlocks : A.n_blocks, nr), block(span <= 512 ? 256 : (span <= 16384 ? 512 : 1024));
        if (loop) hipLaunchKernelGGL((nkw_tiles_kernel<false, true>), grid, block, lds, c->stream, A);
        else hipLaunchKernelGGL((nkw_tiles_kernel<false, false>), grid, block, lds, c->stream, A);
    }
    const int32_t n_short = n_tiles - n_wide_tiles;
    if (n_short > 0) {  // (K <= kWaveTileTopics: one range, less than 48 KB for four histograms)
        const int32_t blocks = (n_short + 3) / 4;
        A.tiles = tiles + n_wide_tiles; A.n_tiles = n_short;
        A.run = xcd_run_length(blocks, kTileRun / 4);
        A.n_blocks = xcd_runs_grid(blocks, A.run);
        const bool loop = go && A.n_blocks > 2 * kLoopBlocks;
        const dim3 grid(loop ? kLoopBlocks : A.n_blocks), block(256);
        if (loop) hipLaunchKernelGGL((nkw_tiles_kernel<true, true>), grid, block, 4 * lds, c->stream, A);
        else hipLaunchKernelGGL((nkw_tiles_kernel<true, false>), grid, block, 4 * lds, c->stream, A);
    }
    LDA_HIP(c, hipGetLastError());
    return LDA_OK;
}


// n_k, zero since launch_dense_rows, by LDS histograms (K <= 8 * kNkRangeTopics)
int launch_nk_hist(lda_ctx* c, const int32_t* go = nullptr)
{
    const int32_t K = c->K;
    const int32_t nr = (K + kNkRangeTopics - 1) / kNkRangeTopics;
    const int32_t span = (K + nr - 1) / nr;
    const int64_t blocks = std::min<int64_t>(hist_blocks(c), nr > 1 ? 512 : 2048);
    const size_t lds = sizeof(int32_t) * (size_t)span;
    if (lds > 48 * 1024)
        LDA_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(nk_hist_ranges_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(nk_hist_ranges_kernel, dim3((unsigned)blocks, (unsigned)nr), dim3(1024), lds,
                       c->stream, c->streamed ? c->d_zt : c->d_z, c->N, K, span, c->d_nk, go);
    LDA_HIP(c, hipGetLastError());
    return LDA_OK;
}

}  // namespace

int launch_scatter_word_major(lda_ctx* c, const int32_t* z, const int32_t* wpos, int64_t n, const int32_t* go)
{
    if (n <= 0) return LDA_OK;
    if (!c->d_zt)  // a sweep ran out of memory, and what it had given back was gone
        return fail(c, LDA_ERR_OOM, "no memory for the word-major copy of the assignment");
    const int64_t per_xcd = (n + kXcds - 1) / kXcds;
    const int64_t per_block = kScatterBlock * kScatterPerThread;
    const int64_t blocks = ((per_xcd + per_block - 1) / per_block) * kXcds;
    hipLaunchKernelGGL(scatter_wm_kernel, dim3((unsigned)blocks), dim3(kScatterBlock), 0, c->stream, z, wpos,
                       n, c->d_zt, c->zt_shift, go);
    LDA_HIP(c, hipGetLastError());
    return LDA_OK;
}

// Two forms of the same counts: the paper's +-1 per moved token, whose cost is that of its
// atomics, and the recount, which does not depend on how many tokens moved.  Where the recount
// can be the cheaper one, a sample of the tokens decides on the device, without the host waiting
// for it: the kernels of the form that is not wanted return at once.
//
// The line: a moved token costs at least 0.1 ns (0.08 ns with 7.4 * 10^8 tokens over 141 000 rows,
// 0.19 ns with 1.8 * 10^6 over 30 011), a recount some 20 us of launches, 2 ns per row and the
// traffic of rows and tokens at about 4 TB/s (2.8 ms for the former corpus at K = 10 000, 0.1 ms
// for the latter at K = 333).  First sweeps move nearly every token: 1.8 * 10^6 tokens in short
// documents, K = 333: 350 us by +-1, 190 us as decided here.
// Neither is known better beforehand: moved tokens that share counters cost up to 2.5 ns (K = 2), a
// recount where one topic holds most of a word's tokens 6.5 ps per token instead of 2, and after a
// sweep of one pass (the refreshed doc side, chains without records) it first copies the assignment
// into word-major order, 5 to 6.5 ps per token.  Both at their dearest for the form chosen: 2 * 10^7
// tokens, 5000 words, K = 2000, 5 % moved after a refreshed sweep, 111 us by +-1 and 229 by the recount.
// With the two in the model, a like corpus with 7 % moved among counters that are shared went from
// 241 to 558 us, so they are left out.
int launch_update_counts(lda_ctx* c)
{
    if (c->K > kNkRangeTopics)
        return fail(c, LDA_ERR_UNSUPPORTED, "lda_update_counts supports K <= %d", kNkRangeTopics);
    c->rows_wanted = 2;
    const double N = (double)c->N, V = (double)c->V, K = (double)c->K;
    const double recount_ns = 2.0e4 + 2.0 * V + V * K / 1000.0 + N / 500.0;
    const double break_even = recount_ns / (0.1 * N);  // share of moved tokens
    int32_t* recount = nullptr;
    if (break_even < 1.0) {
        recount = c->d_flag + 1;
        hipLaunchKernelGGL(sample_moved_kernel, dim3(kMovedSample / 1024), dim3(1024), 0, c->stream, c->d_z,
                           c->d_znew, c->N, (int32_t)(break_even * kMovedSample), recount, c->d_flag + 2,
                           c->d_rows_stale);
        LDA_HIP(c, hipGetLastError());
    }
    // without a sample, a recount only if rows are stale
    const int32_t* const decided = recount ? recount : c->d_rows_stale;
    int32_t* const copy = !recount && decided ? c->d_flag + 1 : nullptr;
    if (copy) recount = copy;
    const int64_t blocks = std::min<int64_t>(hist_blocks(c), 2048);
    const size_t lds = sizeof(int32_t) * (size_t)c->K;
    if (lds > 48 * 1024)
        LDA_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(update_counts_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(update_counts_kernel, dim3((unsigned)blocks), dim3(1024), lds, c->stream, c->d_z,
                       c->d_znew, c->d_word, c->N, c->K, c->d_nkw, c->d_nk, decided, copy);
    LDA_HIP(c, hipGetLastError());
    if (!recount) return LDA_OK;
    const int rc = launch_dense_rows(c, recount);
    return rc != LDA_OK ? rc : launch_nk_hist(c, recount);
}

int launch_rebuild(lda_ctx* c)
{
    const int32_t K = c->K;
    if (K > max_rebuild_topics())
        return fail(c, LDA_ERR_UNSUPPORTED, "count rebuild supports K <= %d", max_rebuild_topics());
    // Rows of words with implied tables are only made where something lately read them: the sweeps that
    // draw from bins, or lda_update_counts, which may be taking turns with this.
    const bool rows = c->n_implied == 0 || c->bins_left > 0 || c->rows_wanted > 0;
    if (c->rows_wanted > 0) --c->rows_wanted;
    int rc = launch_dense_rows(c, nullptr, !rows);
    if (rc != LDA_OK) return rc;
    return launch_nk_hist(c);
}

// Hybrid store (LightLDA Sec. 5): dense rows for the head words as above; for every other word
// a list of its non-zero (topic, count) pairs in ascending topic order plus an open-addressing
// hash row (load <= 1/2) for random lookups, both made word by word from the word's own
// segment of the word-major order (sparse_rows.hip).
int launch_rebuild_hybrid(lda_ctx* c)
{
    const int32_t K = c->K;
    // ---- word-major copy of z and the dense head rows ----
    {
        const int rc = launch_dense_rows(c);
        if (rc != LDA_OK) return rc;
    }
    // ---- sparse rows: lists, lengths and hash rows (sparse_rows.hip) ----
    {
        const int rc = launch_sparse_rows(c);
        if (rc != LDA_OK) return rc;
    }
    // ---- n_k ----
    if (K > 8 * kNkRangeTopics) return launch_nk_by_ranges(c);
    return launch_nk_hist(c);
}

}  // namespace lda

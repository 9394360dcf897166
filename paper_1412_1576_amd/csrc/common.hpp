// Shared declarations of the gfx950 LightLDA library: context, launch helpers,
// and the small device routines every kernel uses (Philox4x32-10, mulhi).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "../../include/lda_mi355x.h"

namespace lda {

constexpr int kWave = 64;
constexpr int32_t kMapped = INT32_MIN;  // d_rshift: the word's records are in buckets

enum State { COUNTS_VALID = 1, ALIAS_VALID = 2, SWEPT = 3 };

// One rebuild work item: a slice [p0, p1) of word w's word-major segment.
// Mixture tables are launched by size class so that a small table does not reserve a large
// table's LDS: list capacity of each class, 0 = the largest that fits LDS, -1 = any size.
constexpr int kMixClasses = 8;
constexpr int32_t kMixClassCap[kMixClasses] = {64, 256, 1024, 2048, 4096, 8192, 0, -1};

struct RebuildTile {
    int32_t w;
    int32_t p0;
    int32_t p1;
    int32_t multi;  // 1: the word has several tiles (row pre-zeroed, merged by atomics);
                    // 2: single tile of a mixture word, whose list of non-zeros is written too;
                    // 3: single tile of a list-only word (kKindListOnly): the list, not the row
};

// A tile of a partition pass (sparse_rows.hip): source positions [p0, p1) of segment seg (a
// long word, or the whole of z)
struct PartTile {
    int32_t seg;
    int32_t p0, p1;
};

// Alias tables built by many workgroups each (alias_split.hpp).  Per chunk of a table:
struct BigSums {
    uint64_t q0, q;        // sums of the quantised weights, of the shifted ones
    uint64_t df, ex;       // deficit of the lights, excess of the heavies
    uint32_t lights;
    uint32_t a_before;     // lights of the table's chunks before this one
};
// per table:
struct BigState {
    uint64_t Q0, C, pad;
    uint32_t sh;
    uint32_t A;            // lights
};
struct BigSet {
    int2* d_chunks = nullptr;
    uint32_t* d_first = nullptr;
    uint64_t* d_list = nullptr;
    BigSums* d_sums = nullptr;
    BigState* d_state = nullptr;
    uint64_t* dx = nullptr;    // not owned
    uint32_t* hidx = nullptr;
    std::vector<uint32_t> batch_chunk;  // first chunk of every batch, and the end
};

// Streamed data blocks (stream_blocks.hip): tiles [c0, c1) = tokens [g0, g1) of the corpus
struct StreamBlock {
    int32_t c0, c1;
    int64_t g0, g1;
};

// One of the two device buffers a block is loaded into
struct BlockBuffer {
    int32_t* word = nullptr;
    int32_t* z = nullptr;
    int32_t* znew = nullptr;
    int32_t* wpos = nullptr;
    uint8_t* tokdoc = nullptr;
    hipEvent_t loaded = nullptr, computed = nullptr, stored = nullptr;
};

}  // namespace lda

struct lda_ctx {
    // problem
    int64_t D = 0, N = 0;
    int32_t V = 0, K = 0;
    double alpha = 0, beta = 0, alphabar = 0, betabar = 0;
    uint64_t seed = 0;
    lda_options opt{};
    hipStream_t stream = nullptr;
    int state = 0;
    uint32_t sweep_index = 0;
    bool prev_valid = false;  // d_znew holds the assignment before the last sweep
    int32_t longest_doc = 0;  // tokens of the longest document
    int32_t most_word_tokens = 0;
    std::string err;

    // corpus, document-major (CSR order)
    int32_t* d_word = nullptr;  // [N] word id of token g
    int32_t* d_doff = nullptr;  // [D+1] token offset of document d
    int32_t* d_z = nullptr;     // [N] snapshot assignment
    int32_t* d_znew = nullptr;  // [N] next assignment
    // word-major view
    int32_t* d_gid = nullptr;   // [N] CSR position of the p-th token in word-major order
    int32_t* d_wpos = nullptr;  // [N] position of token g's records in zt / rec: its word-major
                                //     position (inverse of gid), mapped through d_xmap if set
    int32_t* d_xmap = nullptr;  // [N] word-major position -> record position (NULL: identity)
    int32_t* d_rshift = nullptr;  // [V] with d_xmap: record position - word-major position of a word's
                                  //     tokens where that is one number, else kMapped
    int32_t record_bucket_shift = -1;  // records of words with fewer than bucket_below tokens ordered by (CSR
                                       // position >> shift, word-major position), after those of the
                                       // others, which are in word-major order; -1: all are
    int32_t bucket_below = 0;
    // Word-major token records of 2^zt_shift ints.  Fields: the token's z, then the topic that
    // doc step i of the coming sweep proposes for it (when td_valid); one int per field, or,
    // with zt_pack16 (K <= 65536), two 16-bit fields per int.  The z field is the low
    // zt_mask bits of the record's first int.
    int32_t* d_zt = nullptr;
    size_t zt_ints = 0;         // allocated ints
    int32_t zt_shift = 0;
    bool zt_pack16 = false;
    uint32_t zt_mask = 0xFFFFFFFFu;
    bool zt_current = false;    // record [0] equals d_z
    bool td_valid = false;      // the stored doc proposals are those of sweep td_sweep, drawn
    uint32_t td_sweep = 0;      //   from d_z, for a chain of td_nw word and td_nd doc steps
    int32_t td_nw = 0, td_nd = 0;
    // Word-pass output, word-major, 2^rec_shift ints per token (sweep_split.hip)
    int32_t* d_rec = nullptr;
    size_t rec_ints = 0;
    size_t refused_ints = SIZE_MAX;  // of records of chains of 5 to 8 steps: not asked for again
    // Work lists of the word pass: items (w, p0, n, 0) whose rows are staged in LDS, and
    // pieces (w0, w1, p0, n) of several short words whose rows are gathered
    int4* d_row_items = nullptr;
    int4* d_mix_items = nullptr;  // items (w, p0, n, 0) of mixture words whose row is rebuilt in LDS
    int4* d_gather_pieces = nullptr;
    int32_t n_row_items = 0, n_mix_items = 0, n_gather_pieces = 0;
    // option time_sweep_passes: events before the word pass, between the passes and after
    // the doc pass's tile kernel
    hipEvent_t pass_ev[3] = {nullptr, nullptr, nullptr};
    bool pass_ev_recorded = false;
    int32_t* d_woff = nullptr;  // [V+1] segment offsets
    // model
    int32_t* d_nkw = nullptr;   // [V*K] word-topic counts (dense rows)
    int32_t* d_nk = nullptr;    // [K]
    uint4* d_alias = nullptr;   // [V*K] (split, alias, n_kw[bin], n_kw[alias]) per bin
    uint32_t* d_cap = nullptr;  // [V] bin capacity of the word's table
    // Implied tables (implied.hpp): of words with few tokens, instead of K bins each.  A table's
    // entries start at im_off[w]; h_table_form: 0 dense, 1 implied, 2 no tokens (no table is drawn from).
    static constexpr int kImpliedClasses = 2;
    int32_t n_implied = 0, n_im_class[kImpliedClasses] = {};
    std::vector<uint8_t> h_table_form;   // empty: every word has its dense table
    int32_t* d_im_words = nullptr;
    int32_t* d_im_n = nullptr;           // [V] entries of the word's list (d_im_key)
    uint32_t* d_im_off = nullptr;        // [V+1]
    uint4* d_im_head = nullptr;          // [V]
    uint32_t* d_im_key = nullptr;
    uint64_t *d_im_corr = nullptr, *d_im_x = nullptr;
    uint32_t* d_im_qz = nullptr;         // [K]
    uint64_t* d_im_pz = nullptr;         // [K+1]
    uint64_t* d_im_sum = nullptr;        // [3]
    int32_t* d_fixed_words = nullptr;    // words with a dense table always
    int32_t n_fixed_words = 0;
    int4* d_misfits = nullptr;           // (word, list offset, entries) of the words whose sums do not fit the
    int32_t* d_n_misfits = nullptr;      //   implied form, which have dense tables made from their lists; how many:
                                         //   several lists of them (implied.hpp)
    int4* d_im_pieces = nullptr;         // pieces of the word pass, as d_gather_pieces
    int32_t n_im_pieces = 0;
    int4* d_other_pieces = nullptr;      // d_gather_pieces without those words
    int32_t n_other_pieces = 0;
    int4* d_short_pieces = nullptr;      // and of words of the mixture form with few tokens
    int32_t n_short_pieces = 0;
    // Which forms hold the tables of the current counts.  One-pass sweeps draw from bins, two-pass ones from
    // either; after a one-pass sweep the next kBinsSweeps two-pass ones draw from bins as well, so that a
    // program that takes the two in turn has its tables made once (api.hip).
    static constexpr int32_t kBinsSweeps = 4;
    bool implied_built = false, all_dense_built = false;
    int32_t bins_left = 0;
    // A sweep was captured into a graph that draws from these: lda_build_alias makes them from then on, as
    // the host does not see the replays.
    bool implied_captured = false, bins_captured = false;
    bool implied_in_graph = false;  // a graph may use the arrays of the implied tables: never given back early
    // The counts of words with implied tables: in their lists alone after a recount, unless their rows
    // are wanted (by one-pass sweeps, or lda_update_counts lately).  What holds is kept on the device,
    // where captured work finds it too: *d_rows_stale = 1: the lists do, 0: the rows do.
    int32_t* d_rows_stale = nullptr;
    int32_t rows_wanted = 0;
    lda::RebuildTile* d_row_tiles = nullptr;  // d_tiles without the words of implied tables
    int32_t n_row_tiles = 0, n_wide_row_tiles = 0;
    // sweep tiling: chunk c covers documents [chunk_doc[c], chunk_doc[c+1])
    int32_t* d_chunk_doc = nullptr;
    int32_t* d_chunk_tok = nullptr;  // [n_chunks+1] first token of chunk c (= doff[chunk_doc[c]])
    uint8_t* d_tokdoc = nullptr;     // [N] index of the token's document inside its tile
    int32_t n_chunks = 0;
    int32_t chunk_tokens = 0, chunk_docs = 0, sweep_block = 0;
    // second tiling of the same documents with larger tiles, used by the doc pass of chains
    // of at most two steps (n_chunks2 == 0: not built).  A document is "long" under both
    // tilings when it exceeds chunk_tokens.
    int32_t* d_chunk_doc2 = nullptr;
    int32_t* d_chunk_tok2 = nullptr;
    uint8_t* d_tokdoc2 = nullptr;
    int32_t n_chunks2 = 0;
    int32_t chunk_tokens2 = 0, chunk_docs2 = 0, sweep_block2 = 0;
    bool chunk_direct = false, chunk_direct2 = false;  // K counters per document fit the tiles
    uint32_t* d_doc_limit = nullptr;  // [tokens of a tile's document] (doc_limits); NULL: there is none
    // documents too long for an LDS tile: hashed in a global workspace
    int32_t* d_long_doc = nullptr;     // [n_long] document ids
    int64_t* d_long_slot = nullptr;    // [n_long+1] first hash slot of each long document
    int32_t* d_long_keys = nullptr;    // [total slots]
    int32_t* d_long_cnts = nullptr;
    int32_t* d_long_first = nullptr;   // [total slots] log-likelihood beyond kLongDocTopics: first token of every topic
    int4* d_long_slices = nullptr;     // (first token, tokens, begin of the slice, its tokens): doc pass
    int4* d_long_parts = nullptr;      // the same for the doc proposals of the next sweep
    int32_t n_long_slices = 0, n_long_parts = 0;
    int32_t n_long = 0;
    int64_t long_slots = 0;
    int64_t long_tokens = 0;           // tokens of these documents
    std::vector<int32_t> h_long_doc;
    // rebuild tiling
    lda::RebuildTile* d_tiles = nullptr;
    int32_t n_tiles = 0;
    int32_t n_wide_tiles = 0;  // a workgroup's each; the short ones after them are a wave's
    lda::RebuildTile* d_list_tiles = nullptr;  // form 2, of rows of several topic ranges
    int32_t n_list_tiles = 0;
    int32_t rebuild_tile_tokens = 0;
    int32_t* d_multi_words = nullptr;  // words that own several tiles
    int32_t n_multi_words = 0;
    // hybrid store / mixture proposal (Sec. 4.2 and 5); all null in the all-dense mode
    bool hybrid = false;
    int32_t H = 0;                       // word ids [0, H) own a dense n_kw row
    int32_t* d_dense_alias_words = nullptr;  // words that draw from a dense K-bin table
    int32_t n_dense_alias = 0;
    int32_t n_mix = 0;                   // words that draw from the mixture
    int64_t mix_tokens = 0;              // and their tokens
    // the mixture words by list capacity (kMixClassCap; the tables of the last class are built by
    // many workgroups each)
    int32_t* d_mix_class[lda::kMixClasses] = {};
    int32_t n_mix_class[lda::kMixClasses] = {};
    int32_t* d_sparse_words = nullptr;   // words whose list the recount makes (the log-likelihood sums
                                         // over it): sparse rows, and most of the mixture's dense rows
    int32_t n_sparse = 0;
    int32_t* d_row_words = nullptr;      // the other words: the log-likelihood sums over their rows
    int32_t n_row_words = 0;
    int32_t n_list_only = 0;             // words marked kKindListOnly
    int32_t* d_list_rows = nullptr;      // those beyond kMixRowTopics topics: one-pass sweeps get their rows
    int32_t n_list_rows = 0;
    int32_t* d_compact_words = nullptr;  // mixture words with a dense row (list made by compaction)
    int32_t n_compact = 0;
    uint32_t* d_sp_off = nullptr;        // [V+1] first list entry of word w (capacity min(c_w, K))
    int32_t* d_sp_topic = nullptr;       // non-zero topics of the word, ascending
    int32_t* d_sp_count = nullptr;       // their counts
    int32_t* d_sp_nnz = nullptr;         // [V] entries in use
    uint32_t* d_hs_off = nullptr;        // [V+1] first hash slot of word w (power-of-two capacity)
    uint2* d_hs = nullptr;               // (topic, count) slots, topic = -1: empty
    uint4* d_ma = nullptr;               // mixture tables: one packed bin per list entry
    // one 32-byte record per word, [2w] = (entries n, capacity C, QS low, QS high) rewritten by
    // every table build, [2w+1] = (list offset, hash offset, log2 hash slots, kind) fixed
    uint4* d_metaA = nullptr;            // [2V]
    uint4* d_metaB = nullptr;            // = d_metaA + 1 (not owned)
    uint2* d_beta_alias = nullptr;       // [K] shared table of the beta term (split, alias)
    uint64_t* d_beta_hdr = nullptr;      // [2] QB, capacity
    // tables built by many workgroups each (alias_split.hpp): work lists, and the list memory
    lda::BigSet big_dense, big_mix, big_beta;
    uint64_t* d_big_dx = nullptr;
    uint32_t* d_big_hidx = nullptr;
    // the build of the beta table and of the small tables runs beside the other table kernels
    hipStream_t side_stream = nullptr;
    hipEvent_t side_fork = nullptr, side_join = nullptr;
    bool side_pending = false;           // side_join recorded, not yet waited for
    int64_t total_list = 0, total_hash = 0;
    std::vector<int32_t> h_wcount;       // corpus frequency of every word
    std::vector<uint8_t> h_wkind;        // bit 0: dense row, bit 1: dense proposal table,
                                         // bit 2 (kKindListOnly): the dense row is allotted but
                                         // not kept -- see kKindListOnly
    std::vector<uint32_t> h_sp_off, h_hs_off;
    // sparse-row rebuild (sparse_rows.hip): words sorted in LDS, in three size classes; longer
    // words partitioned by topic range in d_long_part (segment of long word i at d_long_base[i])
    int32_t* d_sort_words[3] = {};
    int32_t n_sort_words[3] = {};
    int32_t* d_long_words = nullptr;
    uint32_t* d_long_base = nullptr;
    lda::PartTile* d_long_tiles = nullptr;
    lda::PartTile* d_fill_tiles = nullptr;  // tiles over the places of the long words' lists
    int32_t n_long_words = 0, n_long_tiles = 0, n_fill_tiles = 0;
    uint32_t long_word_tokens = 0;
    uint32_t max_hash_row = 0;           // slots of the largest hash row that is filled by atomics
    bool clear_all_hash_rows = false;    // those rows own most of d_hs: clear it in one go
    int32_t* d_long_part = nullptr;
    uint32_t* d_long_dcount = nullptr;   // [n_long_words * ranges] tokens per range (zero between rebuilds)
    uint32_t* d_long_dstart = nullptr;   // [n_long_words * (ranges + 1)]
    uint32_t* d_long_cursor = nullptr;
    uint32_t* d_long_nnzd = nullptr;     // non-zero topics per range
    uint32_t* d_long_lofs = nullptr;     // their exclusive prefix: list position of a range
    // n_k for very large K: z partitioned by topic range
    int32_t* d_nk_part = nullptr;
    lda::PartTile* d_nk_tiles = nullptr;
    int32_t n_nk_tiles = 0;
    uint32_t* d_nk_ranges = nullptr;
    // streamed data blocks: the per-token arrays live in pinned host memory and pass through two
    // device buffers; d_word, d_z, d_znew, d_gid, d_wpos, d_tokdoc are then NULL between calls
    bool streamed = false;
    std::vector<lda::StreamBlock> blocks;
    int64_t max_block_tokens = 0;
    int32_t *h_word = nullptr, *h_z = nullptr, *h_znew = nullptr, *h_wpos = nullptr;
    uint8_t* h_tokdoc = nullptr;
    lda::BlockBuffer buf[2];
    hipStream_t load_stream = nullptr, store_stream = nullptr;
    hipEvent_t pass_begin = nullptr, pass_end = nullptr, stored_all = nullptr;
    bool stored_all_recorded = false;
    // scratch
    double* d_partial = nullptr;       // per-block partial sums (log-likelihood)
    int32_t n_partial = 0;
    double* d_lg_terms = nullptr;      // log-likelihood terms by count: of alpha, then of beta
    int32_t* d_row = nullptr;          // [max(K,1)] row staging for accessors
    int32_t* d_flag = nullptr;         // [4] validation; recount wanted; sum of a sample (zero between uses)
    std::vector<void*> kept;           // replaced while the stream was being captured; freed at the end
    // host copies of small layouts
    std::vector<int32_t> h_doff;
};

namespace lda {

int fail(lda_ctx* c, int code, const char* fmt, ...);

// Device memory of a context: the caller's allocator (lda_options) or hipMalloc / hipFree.
// device_malloc returns LDA_OK or records LDA_ERR_OOM; *p is NULL on failure.  try_device_malloc
// records nothing and returns NULL.
void* try_device_malloc(lda_ctx* c, size_t bytes);
int device_malloc(lda_ctx* c, void** p, size_t bytes, const char* what);
void device_free(lda_ctx* c, void* p);
// Gives back memory that work queued on the context's stream may still use: waits for the stream
// first (a caller's allocator may hand the block to other work at once), or, while the stream is
// being captured and cannot be waited for, keeps the block until lda_destroy.
void device_release(lda_ctx* c, void* p);
bool stream_is_captured(lda_ctx* c);

template <class T>
int device_malloc(lda_ctx* c, T** p, size_t count, const char* what)
{
    return device_malloc(c, reinterpret_cast<void**>(p), sizeof(T) * (count ? count : 1), what);
}

#define LDA_ALLOC(ctx, ptr, count, what)                                                  \
    do {                                                                                  \
        const int rc__ = lda::device_malloc((ctx), (ptr), (size_t)(count), (what));       \
        if (rc__ != LDA_OK) return rc__;                                                  \
    } while (0)

#define LDA_HIP(ctx, call)                                                              \
    do {                                                                                \
        hipError_t e__ = (call);                                                        \
        if (e__ != hipSuccess)                                                          \
            return lda::fail((ctx), e__ == hipErrorOutOfMemory ? LDA_ERR_OOM : LDA_ERR_HIP, \
                             "%s: %s (%s:%d)", #call, hipGetErrorString(e__), __FILE__, __LINE__); \
    } while (0)

// launchers implemented in the kernel files
int launch_layout(lda_ctx* c, const int32_t* h_word);      // word-major order, woff, z init
int launch_alias_build(lda_ctx* c);
int launch_alias_build_hybrid(lda_ctx* c);
int launch_dense_listed(lda_ctx* c);                       // dense tables of d_fixed_words and d_misfits
int launch_dense_table(lda_ctx* c, int32_t w);             // of one word (all-dense store)
// implied tables (implied.hpp)
int setup_implied(lda_ctx* c, const std::vector<int32_t>& woff, const std::vector<RebuildTile>& tiles);
void free_implied(lda_ctx* c);
int give_up_implied(lda_ctx* c);                           // for their memory; the tables of the current counts are bins then
void list_implied_pieces(const lda_ctx* c, const std::vector<int32_t>& woff, std::vector<int4>& implied,
                         std::vector<int4>& others);       // word pass: their pieces, and those of the other words
int launch_implied_tables(lda_ctx* c);
int launch_implied_lists(lda_ctx* c);                      // their lists from the word-major z
int launch_rows_from_lists(lda_ctx* c, int32_t w);         // rows of all such words (w < 0) or one, if stale
int launch_loglik_implied(lda_ctx* c, double lg_beta, const double* terms, int blocks, double* partial);
// the tables of either form, unless they are made (all-dense store)
int have_implied_tables(lda_ctx* c);
int have_all_dense_tables(lda_ctx* c);
int launch_rebuild_hybrid(lda_ctx* c);
int launch_sweep_hybrid(lda_ctx* c, int32_t mh_steps);
int launch_loglik_word_hybrid(lda_ctx* c, double* word_part);
// A second stream of the library's own (default priority) for kernels that can run beside
// the caller's stream: fork (the side stream waits for everything queued on the caller's
// stream so far), launch on c->side_stream, side_stream_done, and later join (the caller's
// stream waits for the side stream).  One fork may be pending at a time.
int fork_side_stream(lda_ctx* c);
int side_stream_done(lda_ctx* c);
int join_side_stream(lda_ctx* c);
int max_lds_table_entries();  // largest alias table built in LDS
int setup_big_tables(lda_ctx* c, const std::vector<int32_t>& big_mix);
void free_big_tables(lda_ctx* c);

// Up to this many topics the doc pass keeps a copy of n_k in every workgroup's LDS.
constexpr int32_t kNkLdsTopics = 16384;

// slot of topic t in a hash row of 2^lg slots (multiplicative hashing, top bits)
__host__ __device__ inline uint32_t row_hash_slot(int32_t t, uint32_t lg)
{
    return ((uint32_t)t * 0x9E3779B1u) >> (32u - lg);
}

// A bin of a mixture word's own table in 16 bytes: the split height and, for each
// of its two outcomes, the topic (20 bits) and the word's count of it (28 bits).
constexpr uint32_t kMixTopicBits = 20, kMixCountBits = 28;
__host__ __device__ inline uint4 pack_mix_bin(uint32_t split, int32_t t_own, int32_t t_other,
                                              int32_t n_own, int32_t n_other)
{
    return make_uint4(split, (uint32_t)t_own | ((uint32_t)n_own << kMixTopicBits),
                      (uint32_t)t_other | ((uint32_t)n_other << kMixTopicBits),
                      ((uint32_t)n_own >> 12) | (((uint32_t)n_other >> 12) << 16));
}
// A mixture word with a dense row, at least kMixRowMinTokens tokens, K <= kMixRowTopics and a
// segment that fits one rebuild tile is served everywhere from its list of non-zeros: the
// word pass rebuilds its row in LDS from the list, the table build reads the list, the
// log-likelihood sums over it.  So is, in a larger K, one of at most kShortTokens tokens, whose list the
// word pass keeps in LDS (12 600 rows of 10^5 topics were two thirds of those that a recount wrote, 1.2
// of 1.85 ms).  Rewriting its K-entry dense row at every count rebuild would
// be the largest write of the rebuild (c3: 5.4 of 6.4 GB) for nobody to read, so the row is
// left untouched (all zero since lda_init) and the word is marked with this bit; the rare
// lookup outside the word pass (fused sweep) searches the word's mixture table, whose bins
// are its non-zero topics in ascending order.  In the larger K, where such words are the rare ones
// and have most of the look-ups, a fused sweep puts the counts into the rows before it and
// zeros back after it (list_rows_kernel), and the words' records on the device are not marked.
constexpr uint32_t kKindListOnly = 4u;
constexpr int32_t kMixRowTopics = 16384;   // largest K whose n_kw row a mixture item keeps in LDS
constexpr int32_t kMixRowMinTokens = 128;
constexpr int32_t kShortTokens = 1024;     // tokens of a mixture word that the word pass serves from its list

__host__ __device__ inline void unpack_mix_bin(const uint4& e, bool own, int32_t& topic,
                                               int32_t& count)
{
    const uint32_t sel = own ? e.y : e.z;
    const uint32_t hi = own ? (e.w & 0xFFFFu) : (e.w >> 16);
    topic = (int32_t)(sel & ((1u << kMixTopicBits) - 1u));
    count = (int32_t)((sel >> kMixTopicBits) | (hi << 12));
}
int launch_sweep(lda_ctx* c, int32_t mh_steps);
// Sweep with the doc side refreshed after every token (sweep_refresh.hip)
int refresh_sweep_max_doc();
int launch_sweep_doc_refresh(lda_ctx* c, int32_t mh_steps, int32_t longest_doc);
// Two-pass sweep (word pass over word-major tokens, doc pass over document tiles)
bool split_sweep_supported(lda_ctx* c, int32_t mh_steps);
bool doc_limits(double alphabar, std::vector<uint32_t>& limit);
int setup_split_sweep(lda_ctx* c, const std::vector<int32_t>& woff);
int launch_sweep_split(lda_ctx* c, int32_t mh_steps, bool bins);  // bins: no word's table is implied
int launch_tokdoc(lda_ctx* c);                               // per-token document index in its tile
int launch_rebuild(lda_ctx* c);
int launch_update_counts(lda_ctx* c);  // n_kw, n_k by +-1 for the tokens the last sweep moved
int setup_sparse_rows(lda_ctx* c, const std::vector<int32_t>& woff);
int launch_sparse_rows(lda_ctx* c);   // lists, list lengths and hash rows of the sparse-row words
int launch_nk_by_ranges(lda_ctx* c);  // n_k when K is too large for a few LDS histograms over z
size_t loglik_partials(const lda_ctx* c);
int setup_loglik(lda_ctx* c);
int launch_loglik(lda_ctx* c, double* doc_part, double* word_part);
int launch_loglik_doc_tiles(lda_ctx* c, double* d_partial);  // partial[tile] of the bound tiles
// zw[wpos[i]] = z[i], i < n: topics into the word-major copy (go: only if *go is not zero)
int launch_scatter_word_major(lda_ctx* c, const int32_t* z, const int32_t* wpos, int64_t n,
                              const int32_t* go = nullptr);
// streamed data blocks (stream_blocks.hip)
int enter_streamed_mode(lda_ctx* c, const std::vector<int32_t>& chunk_doc);
void leave_streamed_mode(lda_ctx* c);
int launch_sweep_streamed(lda_ctx* c, int32_t mh_steps);
int launch_loglik_doc_streamed(lda_ctx* c, double* d_partial);
int streamed_get_z(lda_ctx* c, int32_t* z);
int streamed_set_z(lda_ctx* c, const int32_t* z);
int streamed_doc_z(lda_ctx* c, int64_t d, const int32_t** z_shifted);
int streamed_sync(lda_ctx* c);
int launch_ndk_row(lda_ctx* c, int64_t d);                  // dense n_dk row into c->d_row
int launch_check_range(lda_ctx* c, const int32_t* d_vals, int64_t n, int32_t lo, int32_t hi,
                       bool* ok);
int max_alias_topics();    // largest K the dense alias kernel handles
constexpr int32_t kWaveTilesLeast = 4096;
int32_t wide_tiles_first(int32_t K, std::vector<RebuildTile>& tiles);  // returns how many these are
int max_rebuild_topics();  // largest K the count-rebuild tiles handle
// Tokens of a word whose row of several topic ranges gives its list too (nkw_list_rows_kernel)
constexpr int32_t kListRowTokens = 8192;

// ------------------------------------------------------------------------------------
// device helpers
// ------------------------------------------------------------------------------------
// LDS written by some lanes of a wave is read by others after this
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ uint32_t mulhi32(uint32_t a, uint32_t b) { return __umulhi(a, b); }

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies,
// the key advanced by Weyl constants between rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        // full 64-bit products: one multiply instruction yields both halves
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
        // (0x96: the exclusive or of three, one instruction instead of two)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// (x + 1/2) / 2^32: uniform in (0,1), exact in fp64
__device__ __forceinline__ double unit_open(uint32_t x)
{
    return ((double)x + 0.5) * (1.0 / 4294967296.0);
}

}  // namespace lda

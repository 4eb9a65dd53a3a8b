// Internal declarations shared by the host runtime (api.cpp) and the HIP kernels.
// Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace oprag {

constexpr int kMaxK = 128;                 // largest k any list may ask for
constexpr int kMaxQPerLaunch = 4096;       // queries per dense launch (the host splits larger batches evenly)
constexpr int kChunkRowBits = 24;          // rows of a dense chunk: a queued hit keeps its offset in so many bits
constexpr int kHeldTiles = 80;             // kTileScores: most tiles of a chunk times queries (their scores fit LDS)
constexpr int kDtypeF32 = 0, kDtypeBF16 = 1, kDtypeF16 = 2;

// Modes of the tiled scoring kernel (kTileUnits: kTileMax with groups that span tiles; kTileSample: of
// rows spread over the index; kTileScores: every score, and the coarse maxima).
enum TileMode { kTileMax = 0, kTileFilt = 1, kTileDump = 2, kTileUnits = 3, kTileSample = 4, kTileScores = 5 };

struct DenseArgs {
  const void* X;                // slab rows [n_rows x d]
  long long n_rows;
  int d;
  const void* Q;                // queries of this launch [nq x d]
  int nq;
  int k;
  int n_qblocks;
  int n_chunks;
  long long tiles;              // chunk c takes row tiles [c tiles / n_chunks, (c + 1) tiles / n_chunks)
  // kTileSample, kTileFilt: tile j of the launch starts at row j tile_pitch (otherwise its tiles are the
  // index's).  kTileSample: a tile's rows are row_pitch apart.  kTileFilt with skip > 0: tile j starts at
  // row (j + j / skip + 1) tile_pitch, so every (skip + 1)-th is left out (skip_recip: 2^32 / skip,
  // rounded up).
  int tile_pitch = 0, row_pitch = 1, skip = 0;
  unsigned skip_recip = 0;
  unsigned long long* partial;  // workspace
  float* out_scores;            // [nq x k]
  long long* out_ids;           // [nq x k]
  // Filter: every row scoring >= th[q * th_stride] becomes a candidate key in cbuf[q][0 .. cap);
  // ccnt[q] counts them (and may exceed cap).  check_mask: tiles between looks at the workgroup's
  // queue of hits, less one (a power of two less one).
  const float* th = nullptr;
  int th_stride = 0;
  unsigned long long* cbuf = nullptr;
  int* ccnt = nullptr;
  long long cap = 0;
  int check_mask = 0;
  // When set, the launch does nothing unless *gate != 0 (a device-side overflow flag).
  const int* gate = nullptr;
  // Score dump: every score to dump[q * dump_ld + row]; with dump_mm set, also the minimum and
  // maximum of each (query, chunk) to dump_mm[(q * n_chunks + chunk) * 2 + {0, 1}].
  float* dump = nullptr;
  long long dump_ld = 0;
  float* dump_mm = nullptr;
  // Group maxima: the largest score of each group (a lane's rows of mx_gs consecutive 16-row subtiles;
  // kTileUnits: of all its subtiles in a unit of 1 << unit_sh consecutive tiles of a chunk) to
  // mx[q * mx_ld + group], and of each lane over its chunk to cmx[q * cmx_ld + ..] (NaN: no row;
  // either may be null).
  float* mx = nullptr;
  long long mx_ld = 0;
  int mx_gs = 1;
  int unit_sh = 0, upc = 0;     // upc units per chunk (the last of a chunk may be short or empty)
  float* cmx = nullptr;
  long long cmx_ld = 0;
};

// Maxima of one launch: groups of gs subtiles (a power of two), per_tile of a row tile (of a unit of
// tiles, DenseArgs), count in all; coarse ones in all (0: none are kept).  The groups' row stride ld,
// the coarse ones' cld.
struct MaxGroups {
  int gs = 1, per_tile = 0, count = 0, coarse = 0;
  int unit_sh = 0, upc = 0;
  long long ld = 0, cld = 0;
};

// The k best rows from a launch's maxima (gate as above).  Lane l of a tile (wave row and lane
// quarter, 1 << lanes_sh of them) has 1 << mt_sh subtiles in groups of 1 << gs_sh (1 << gl_sh of them);
// group ((tile << lanes_sh) + l << gl_sh) + i, coarse maximum (chunk << lanes_sh) + l, and chunk
// c has tiles [c tiles / n_chunks, (c + 1) tiles / n_chunks), at most `most`.  With unit_sh > 0 unit
// c upc + u, of the tiles 1 << unit_sh from the u-th such run of the chunk, takes a tile's place.
struct RescoreArgs {
  const void* X = nullptr;
  const void* Q = nullptr;
  long long n_rows = 0;
  int d = 0, k = 0;
  const float* fine = nullptr;   // null: the coarse maxima are the groups
  int two = 0;                   // the groups are searched through the coarse maxima
  long long fine_ld = 0;
  int n_fine = 0;
  const float* coarse = nullptr;
  long long coarse_ld = 0;
  int n_coarse = 0;
  int tile_rows = 0, n_chunks = 1, most = 0;
  int least = 0, spare = 0;      // tiles / n_chunks, tiles % n_chunks
  int gpt_sh = 0, lanes_sh = 0, gl_sh = 0, gs_sh = 0, mt_sh = 0;
  int unit_sh = 0, upc = 0;
  int scores = 0;                // fine holds every score ([nq x fine_ld] by row), of kTileScores
  float* out_scores = nullptr;
  long long* out_ids = nullptr;
  const int* gate = nullptr;
};

// Launchers of one storage type (dense_tile_*.hip).
template <int DT>
hipError_t tile_launch(int shape, int mode, long long grid, DenseArgs& arg, hipStream_t s, hipEvent_t ev0,
                       hipEvent_t ev1);
template <int DT>
hipError_t rescore_launch(const RescoreArgs& a, int nq, hipStream_t s);

// How a search of one launch runs (dense.hip): group maxima and rescoring, every score and a
// selection (kScores: through coarse maxima), or threshold levels.
struct DensePlan {
  enum Kind { kMaxima, kDump, kScores, kFilter };
  Kind kind = kMaxima;
  int n_cus = 0;                // compute units of the device the plan is for
  int shape = 0;                // tile shape over all rows
  long long ld = 0;             // kDump, kScores: row stride of the scores
  MaxGroups groups;             // kMaxima, and kFilter's first level
  // kFilter
  int shape0 = 0;               // tile shape of the first level
  int n_levels = 0;
  long long level_pitch[16] = {};    // rows from a tile of a level to the next
  int row_pitch0 = 1;                // and between the rows of the first level's tiles
  long long level_rows[16] = {};     // rows of the level and those before it
  long long cap = 0;            // candidate slots per query
  MaxGroups groups_all;         // exact fallback: coarse maxima over all rows,
  int cus_all = 0;              // in as many chunks as this many CUs would get
  int n_chunks = 0;             // plan_dense_dump: chunks of the launch
};

DensePlan plan_dense(int dtype, int d, long long n_rows, int nq, int k, int n_cus);
size_t dense_workspace_bytes(const DensePlan& p, int dtype, int d, int nq, long long n_rows, int k);
// Score dump: every score of nq queries against rows [0, a.n_rows) into a.dump.
DensePlan plan_dense_dump(int dtype, int d, long long n_rows, int nq, int n_cus);
// The most chunks such a plan has at any row count up to `capacity`.
int dense_dump_chunks(int dtype, int d, long long capacity, int nq, int n_cus);
hipError_t launch_dense_dump(const DensePlan& p, int dtype, const DenseArgs& a, hipStream_t s);
// Weighted fusion of dense scores D and lexical scores B ([nq x ld], lexical 0 past n_lex),
// min-max normalised per query over n chunks, then the exact top k (cbuf [nq x n], ccnt [nq]).
// The minima and maxima come from the dumps' partials mm_d [nq x pd x 2] and mm_l [nq x pl x 2].
hipError_t launch_weighted_fuse(int n_cus, const float* D, const float* B, long long ld, long long n, long long n_lex, int nq,
                                const float* mm_d, int pd, const float* mm_l, int pl, double wd, double wl, int k,
                                unsigned long long* cbuf, int* ccnt, float* out_scores, long long* out_ids,
                                hipStream_t s);
// Plans take the compute-unit count of the index's device (the grid aims at a multiple of it).
// Enough workspace for a search of up to nq queries at any row count up to `capacity`.
size_t dense_workspace_bound(int dtype, int d, long long capacity, int nq, int k, int n_cus);
// ev0 / ev1 (optional) are recorded on s right before and after the scoring kernel (threshold
// levels: the last level's).  Threshold levels also enqueue their exactness repair: launches
// gated on device-side overflow flags, so the search never waits for the host.
hipError_t launch_dense(const DensePlan& p, int dtype, const DenseArgs& a, hipStream_t s, hipEvent_t ev0 = nullptr,
                        hipEvent_t ev1 = nullptr);

// ---------------------------------------------------------------- sparse (BM25)
struct SparseIndex {
  int vocab = 0;
  long long n_docs = 0;
  long long nnz = 0;
  const long long* term_indptr = nullptr;   // caller-owned
  const int* post_chunk = nullptr;          // caller-owned
  const int* post_tf = nullptr;             // caller-owned
  float* idfk = nullptr;                    // library-owned [vocab]: idf(t) * (k1 + 1)
  float* wpost = nullptr;                   // library-owned [nnz]: tf / (tf + k1 (1 - b + b dl / avgdl))
  // library-owned chunk-major copy: chunk d's (term, weight) pairs at [fwd_ptr[d], fwd_ptr[d + 1])
  long long* fwd_ptr = nullptr;             // [n_docs + 1]
  int* fwd_term = nullptr;                  // [nnz]
  float* fwd_w = nullptr;                   // [nnz]
  // library-owned dense rows of the head terms (the most frequent ones): row hidx[t] of whead
  // holds term t's posting weight for every chunk, 0 where t is absent
  int n_head = 0;
  long long head_ld = 0;                    // row stride: n_docs rounded up to 4
  int* hidx = nullptr;                      // [vocab]: row of term t, -1 for the other terms
  float* whead = nullptr;                   // [n_head x head_ld]
  double avgdl = 0.0;
  float k1 = 0.f, b = 0.f;
};

constexpr int kSparseRange = 32768;        // chunks scored per workgroup (LDS accumulator, 128 KiB)
constexpr int kMaxHead = 992;              // head terms at most (the kernel lists a query's in LDS)
constexpr long long kHeadBytes = 64ll << 20;  // dense head rows at most

// Validates the CSR on the device; returns the number of violations found (synchronous).
hipError_t sparse_validate(int vocab, long long n_docs, long long nnz, const long long* indptr,
                           const int* chunk, const int* tf, const int* doc_len, unsigned int* d_flag,
                           hipStream_t s);
hipError_t sparse_prepare(SparseIndex& sp, const int* doc_len, unsigned long long* d_sum, hipStream_t s);
// Builds the chunk-major copy (fwd_ptr / fwd_term / fwd_w) from the postings and their
// weights; cnt is scratch of n_docs ints.
hipError_t sparse_forward(const SparseIndex& sp, int* cnt, hipStream_t s);
// Fills the dense head rows (whead, zeroed here) from the postings of the head terms
// head_terms[0 .. n_head) (device array, row h = term head_terms[h]).
hipError_t sparse_head_rows(const SparseIndex& sp, const int* head_terms, hipStream_t s);
size_t sparse_workspace_bytes(long long n_docs, int nq, int k);
hipError_t launch_sparse(const SparseIndex& sp, const int* qterm_indptr, const int* qterms, int nq, int k,
                         float* out_scores, long long* out_ids, void* ws, hipStream_t s);

// ---------------------------------------------------------------- fusion and upsert
// Dense-first hybrid: BM25 of the dense candidates cand [nq x n_cand] (dense order, -1 padded,
// 1 <= n_cand <= 128), reciprocal rank fusion with their dense order, top k.
// BM25 scores of every chunk [0, n_docs) for nq queries into dump [nq x ld], and the minimum
// and maximum over chunks [0, mm_rows) of each (query, range of kSparseRange chunks) into
// dump_mm [nq x ranges x 2] (+inf / -inf for a range with none of them).
// Weighted fusion inside the BM25 kernel when the corpus and the n scored chunks fit one
// range: the top k of w_d minmax(dense) + w_l minmax(BM25) over chunks [0, n).
hipError_t launch_sparse_weighted(const SparseIndex& sp, const int* qterm_indptr, const int* qterms, int nq, int k,
                                  const float* dense, long long ld, const float* dense_mm, int pd, long long n,
                                  double wd, double wl, float* out_scores, long long* out_ids, hipStream_t s);
// The hybrid's BM25 list and its reciprocal rank fusion with the dense list in one launch, when
// the corpus fits one range: the fused top k of each query.
hipError_t launch_sparse_rrf(const SparseIndex& sp, const int* qterm_indptr, const int* qterms, int nq, int k_sparse,
                             const long long* dense_ids, int k_dense, int rrf_k, int k, float* out_fused,
                             long long* out_ids, hipStream_t s);
hipError_t launch_sparse_dump(const SparseIndex& sp, const int* qterm_indptr, const int* qterms, int nq, float* dump,
                              long long ld, float* dump_mm, long long mm_rows, hipStream_t s);
hipError_t launch_dense_first(const SparseIndex& sp, const int* qterm_indptr, const int* qterms,
                              const long long* cand, int n_cand, long long nq, int rrf_k, int k, float* out_fused,
                              long long* out_ids, hipStream_t s);
hipError_t launch_rrf(const long long* dense_ids, int k_dense, const long long* sparse_ids, int k_sparse,
                      long long nq, int rrf_k, int k, float* out_fused, long long* out_ids, hipStream_t s);
// Mean pool over each chunk's first lengths[i] (clamped to [0, T]) tokens of hidden states
// [m x T x d] (bf16 or fp32), L2 normalisation, round to the slab dtype into rows
// [first_row, first_row + m).
hipError_t launch_pool_upsert(void* slab, int slab_dtype, int d, long long first_row, const void* hidden,
                              int hidden_dtype, const int* lengths, long long m, int T, hipStream_t s);
hipError_t launch_probe_read(const void* src, long long bytes, unsigned int* sink, int blocks, hipStream_t s);
hipError_t launch_upsert(void* slab, int slab_dtype, int d, long long first_row, const void* rows,
                         int rows_dtype, long long m, hipStream_t s);

}  // namespace oprag

// Dense scoring of bf16, fp16 and fp32 query batches as a tiled matrix product on the matrix cores
// (Section 4.4: vectorised scoring over the embedding matrix), with the selection's first step
// in the epilogue of every tile.
//
// One workgroup of eight waves scores tiles of BM rows x BN queries, 64 dimensions (one
// 128-byte line of each row and query) at a time.  Both operands go from memory straight to
// LDS (buffer_load ... lds, 16 bytes a lane), several 64-dimension stages ahead, and the
// loads run on across the tiles of a chunk.
//
// The waves form two groups of four, one wave of each group on every SIMD, half a phase apart:
// in every interval between two barriers one group issues 16 MFMAs from registers while the
// other reads its next operands from LDS and issues its share of the loads.  A wait only ever
// covers the stage the next phase reads (counted vmcnt), so the loads of the later stages stay
// in flight across all barriers.
//
// LDS holds 128-byte rows; 16-byte piece c of row r is stored at piece c ^ ((r / 2) % 8), so the
// 16 rows x 16 bytes of a fragment read touch every bank once.  The loads write LDS linearly,
// so the swizzle is applied to their source addresses.
//
// Epilogues, on the tile's scores in the accumulators:
//  - MAX: the largest score of every group of rows, for a search that finds the k best groups and
//    scores their rows again (rescore_kernel): no list is kept and nothing is exchanged between
//    waves, so the epilogue is a few dozen instructions;
//  - SCORES: every score and the largest of a lane's over its chunk, for small batches;
//  - FILT: the scores that reach their query's threshold become candidates;
//  - DUMP: every score;
#pragma once

#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>

#include "mfma.h"
#include "oprag_internal.h"
#include "select.h"

namespace oprag {
namespace {

using namespace dev;

constexpr int kTileThreads = 512;

// Wave grid WM x WN; a wave owns MP x MS 16-row subtiles and NP x NS 16-query subtiles, and a
// phase multiplies one row part (MS subtiles) with one query part (NS): MS x NS x 2 MFMAs.
// BR: query rows of a stage in LDS (at least the 64 that one load of every wave fills).
template <int BM, int BN>
struct TileShape;
template <>
struct TileShape<128, 16> {
  static constexpr int WM = 8, WN = 1, MP = 1, MS = 1, NP = 1, NS = 1, NBUF = 6, BR = 64;
};
template <>
struct TileShape<256, 256> {
  static constexpr int WM = 2, WN = 4, MP = 2, MS = 4, NP = 2, NS = 2, NBUF = 2, BR = 256;
};
template <>
struct TileShape<128, 256> {
  static constexpr int WM = 2, WN = 4, MP = 1, MS = 4, NP = 2, NS = 2, NBUF = 3, BR = 256;
};
template <>
struct TileShape<256, 128> {
  static constexpr int WM = 4, WN = 2, MP = 1, MS = 4, NP = 2, NS = 2, NBUF = 3, BR = 128;
};
template <>
struct TileShape<128, 128> {
  static constexpr int WM = 2, WN = 4, MP = 1, MS = 4, NP = 1, NS = 2, NBUF = 4, BR = 128;
};
template <>
struct TileShape<128, 64> {
  static constexpr int WM = 4, WN = 2, MP = 1, MS = 2, NP = 1, NS = 2, NBUF = 6, BR = 64;
};

typedef unsigned int rsrc_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rsrc_t tile_rsrc(const void* base, long long bytes) {
  const unsigned long long b = (unsigned long long)base;
  rsrc_t r;
  r[0] = (unsigned)b;
  r[1] = (unsigned)(b >> 32) & 0xffffu;
  r[2] = (unsigned)(bytes < 0 ? 0 : (bytes > 0xffffffffll ? 0xffffffffll : bytes));
  r[3] = 0x00020000u;
  return r;
}

// 64 lanes x 16 bytes from a buffer resource to LDS [lds, lds + 1024), lane after lane; past the
// resource's end nothing is read.  (Written out because the compiler would drain every load
// before any LDS read; the load has no destination register.  m0 is no clobber: the compiler reserves it,
// writes it before each use of its own, and refuses to preserve it.)
__device__ __forceinline__ void lds_load16(rsrc_t r, int voff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(r)
               : "memory");
}
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }
template <int N>
__device__ __forceinline__ void vm_wait() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Filter mode: hits wait in one LDS queue of the workgroup, (score bits << 32) | (row of the
// chunk's, counted over its tiles, << 8) | query slot, and are moved to the queries' buffers when it fills.  The planner
// gives no chunk more than 2^kChunkRowBits rows.
template <int BM, int BN>
struct TileQueue {
  using S = TileShape<BM, BN>;
  static constexpr int kLds = S::NBUF * (BM + S::BR) * 128;
  static constexpr int kFree = 163840 - kLds - BN * 12 - 64;
  static constexpr int CAP = kFree >= 24576 ? 3072 : 1536;  // entries
  static_assert(CAP * 8 <= kFree, "the queue fits beside the stages");
  static_assert(BN <= 256 && kChunkRowBits + 8 <= 32, "row offset and query slot share 32 bits");
};

// SCORES: the first row of a chunk.
__device__ __forceinline__ long long scores_chunk_row(long long chunk, long long n_rows, int n_chunks) {
  return chunk * ((n_rows + 15) / 16) / n_chunks * 16;
}

template <int DT, int BM, int BN, int MODE>
__global__ __launch_bounds__(kTileThreads) void dense_tile_kernel(DenseArgs a) {
  if (a.gate != nullptr && *a.gate == 0) return;  // a repair launch with nothing to repair
  using M = Mfma<DT>;
  using V = typename M::V;
  using S = TileShape<BM, BN>;
  constexpr bool UNITS = MODE == kTileUnits, SAMPLE = MODE == kTileSample;
  constexpr bool MAX = MODE == kTileMax || UNITS || SAMPLE;
  constexpr int MP = S::MP, MS = S::MS, NP = S::NP, NS = S::NS;
  constexpr int NBUF = MODE == kTileScores ? S::NBUF - 1 : S::NBUF;  // (the scores take the place of a stage)
  constexpr int MT = MP * MS, NT = NP * NS;          // subtiles per wave
  constexpr int AI = BM / MP / 64;            // load instructions per wave and part: rows,
  constexpr int BI = S::BR / NP / 64;                // queries
  constexpr int RB = BM * 128;                       // queries of a stage start here
  constexpr int RAP = (BM / MP) * 128, RBP = (S::BR / NP) * 128;  // bytes of a part
  constexpr int BUF = (BM + S::BR) * 128;
  constexpr int LA = NP == 2 ? 2 : NBUF - 2;         // stages loaded ahead (MP 2: one to two)
  static_assert(S::WM * S::WN == 8 && S::WM * MT * 16 == BM && S::WN * NT * 16 == BN, "wave grid");
  static_assert(MP == 1 || (NP == 2 && NBUF == 2), "schedules");
  static_assert(AI >= 1 && BI >= 1 && BUF <= 65536, "parts and immediates");
  using Q = TileQueue<BM, BN>;
  constexpr int SMEM = MODE == kTileFilt     ? Q::kLds + Q::CAP * 8 + BN * 12 + 64
                       : MODE == kTileScores ? NBUF * BUF + kHeldTiles * BM * 4
                                             : Q::kLds;
  static_assert(SMEM <= 163840, "LDS");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];
  u64* queue = reinterpret_cast<u64*>(smem + Q::kLds);
  int* qhist = reinterpret_cast<int*>(smem + Q::kLds + (MODE == kTileFilt ? Q::CAP * 8 : 0));  // [BN]
  int* qbase = qhist + BN;                                                                     // [BN]
  float* qth = reinterpret_cast<float*>(qbase + BN);                                           // [BN]
  int* qcnt = qbase + 2 * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / S::WN, wn = w % S::WN;
  const bool late = w >= 4;  // the group that runs one interval behind
  const long long L = logical_block();
  const int qb = (int)(L % a.n_qblocks);
  const long long chunk = L / a.n_qblocks;
  const int q0 = qb * BN;
  const int rowb = a.d * (DT == kDtypeF32 ? 4 : 2);  // bytes of a row
  const int nkt = max(2, (rowb + 127) / 128);        // 128-byte stages per tile
  // The chunk has tiles j0 .. j0 + n_tiles - 1 of the launch's (DenseArgs).
  constexpr bool SKIPS = MODE == kTileFilt;
  constexpr bool SCORES = MODE == kTileScores;
  int j0 = (int)(chunk * a.tiles / a.n_chunks);
  int n_tiles = a.n_rows > 0 ? (int)((chunk + 1) * a.tiles / a.n_chunks) - j0 : 0;
  const int tile_pitch = SKIPS || SAMPLE ? a.tile_pitch : BM, row_pitch = SAMPLE ? a.row_pitch : 1;
  auto tile_row = [&](unsigned j) __attribute__((always_inline)) {  // the first row of tile j
    if constexpr (SKIPS) j += __umulhi(j, a.skip_recip) + (a.skip > 0 ? 1u : 0u);
    return (unsigned)tile_pitch * j;
  };
  long long row_begin = tile_row(j0);
  long long row_end = min((long long)tile_row(j0 + max(n_tiles, 1) - 1) + BM * row_pitch, a.n_rows);
  if constexpr (SCORES) {  // chunks of as equal numbers of rows as 16-row steps allow
    j0 = 0;
    row_begin = scores_chunk_row(chunk, a.n_rows, a.n_chunks);
    row_end = min(scores_chunk_row(chunk + 1, a.n_rows, a.n_chunks), a.n_rows);
    n_tiles = (int)((row_end - row_begin + BM - 1) / BM);
  }
  // Row of the index, from the tile's first, at position r of the tile.  SAMPLE: similar rows, which are
  // often neighbours, go to groups of their own (a lane's four positions are a quarter of the tile apart, those
  // of its next subtile an eighth).  The bits of r count separately.
  auto row_at = [&](int r) __attribute__((always_inline)) {
    if constexpr (SAMPLE)
      return ((r & 3) * (BM / 4) + (r >> 4 & 1) * (BM / 8) + (r >> 5) * 4 + (r >> 2 & 3)) * row_pitch;
    return r;
  };

  const int qn0 = wn * NT * 16 + (lane & 15);  // this lane's queries
  float dmn[NT], dmx[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    dmn[j] = __builtin_inff();
    dmx[j] = -__builtin_inff();
  }
  // Filter mode: the queries' thresholds, in LDS (in registers they spill once they change: 1 % of the
  // time).  +inf, so no hits: past the batch, and once a query's buffer has overflowed.  It is
  // searched again then, and more hits would only cost time: 1,024 queries, 16 of them zeros, over
  // 1 M x 768 bf16, 14.5 ms with all hits taken and 5.6 without.
  if constexpr (MODE == kTileFilt) {  // seen after the barriers below
    if (tid == 0) *qcnt = 0;
    if (tid < BN) {
      const int q = q0 + tid;
      qth[tid] = q < a.nq && a.ccnt[q] <= a.cap ? a.th[(long long)q * a.th_stride] : __builtin_inff();
    }
  }

  if (n_tiles > 0) {
    const rsrc_t rx = tile_rsrc(static_cast<const unsigned char*>(a.X) + row_begin * rowb, (row_end - row_begin) * rowb);
    const rsrc_t rq = tile_rsrc(static_cast<const unsigned char*>(a.Q) + (long long)q0 * rowb,
                              (long long)min(a.nq - q0, BN) * rowb);
    const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
    // A load moves eight 128-byte rows; its lane l reads piece (l % 8) ^ swizzle of row l / 8.
    // Load j of wave w fills LDS rows 64 j + 8 w .. + 7 of its part.
    const int lofs = (lane >> 3) * rowb + (((lane & 7) ^ (4 * (w & 1) + (lane >> 4))) * 16);
    const int xofs = lofs + (row_at(lane >> 3) - (lane >> 3)) * rowb;  // of the index's rows
    const unsigned ldsw = lds0 + w * 1024;
    // fp32 rows may end inside a stage: past the row a lane's offset is out of range (reads 0)
    const int cpiece = ((lane & 7) ^ (4 * (w & 1) + (lane >> 4))) * 16;
    auto at = [&](int lane_ofs, int off, int k) __attribute__((always_inline)) {
      if constexpr (DT == kDtypeF32) return k + cpiece < rowb ? lane_ofs + off : -1;
      return lane_ofs + off;
    };
    int arow[AI], brow[BI];  // byte offset of the first of those rows (part 0) in the tile / block
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      const int r = j * 64 + w * 8;
      arow[j] = row_at((r / (MS * 16)) * (MT * 16) + r % (MS * 16)) * rowb;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      const int r = j * 64 + w * 8;
      brow[j] = ((r / (NS * 16)) * (NT * 16) + r % (NS * 16)) * rowb;
    }
    const int apart = row_at(MS * 16) * rowb, bpart = NS * 16 * rowb;
    const int kend = nkt * 128;
    // Byte offset of the chunk's tile i.  (Past the chunk it may wrap, of a single tile's chunk and a very
    // long pitch: such loads land inside the chunk again and are never used.)
    auto tile_ofs = [&](int i) __attribute__((always_inline)) {
      return (tile_row((unsigned)(j0 + i)) - tile_row((unsigned)j0)) * (unsigned)rowb;
    };
    // Cursors (byte offsets of the next stage to load): x for the parts loaded LA stages ahead,
    // y (MP 2) for the second parts, one stage ahead.  Past the chunk nothing is read.  Each goes on to its
    // next tile (at xn, yn) once while a tile is multiplied.
    int xk = 0, yk = 0;
    unsigned xt = 0u, yt = 0u, xn = 0u, yn = 0u;
#define OPRAG_ADV(K, T, N)       \
  {                              \
    K += 128;                    \
    T = K == kend ? N : T;       \
    K = K == kend ? 0 : K;       \
  }
#define OPRAG_LDA(P, K, T, BO)                                                     \
  _Pragma("unroll") for (int j = 0; j < AI; ++j)                                   \
      lds_load16(rx, at(xofs, (T) + (K) + (P) * apart + arow[j], K), ldsw + (BO) + (P) * RAP + j * 8192);
#define OPRAG_LDB(P, K, BO)                                                        \
  _Pragma("unroll") for (int j = 0; j < BI; ++j)                                   \
      lds_load16(rq, at(lofs, (K) + (P) * bpart + brow[j], K), ldsw + (BO) + RB + (P) * RBP + j * 8192);

    // fragment addresses: row (lane % 16) of the wave's first subtile, pieces 4 s + lane / 16
    const int sw = (lane >> 1) & 7;
    const int c0 = ((lane >> 4) ^ sw) * 16, c1 = ((4 + (lane >> 4)) ^ sw) * 16;
    const int fa = (wm * MS * 16 + (lane & 15)) * 128, fb = RB + (wn * NS * 16 + (lane & 15)) * 128;

    f32x4 acc[MT][NT];
    V af[MS][2], bf[NP][NS][2];

    int nxt = 0, cur1 = 0;  // MP 1: LDS offsets of the stage loaded now and of the one multiplied
    // The first stages' loads (from the cursors on); the first stage's first phase is waited for, and
    // the late group falls one interval behind.
    auto start = [&]() __attribute__((always_inline)) {
      nxt = LA % NBUF * BUF;
      cur1 = 0;
      xn = yn = tile_ofs(1);
      if constexpr (MP == 2) {
        OPRAG_LDA(0, xk, xt, 0)
        OPRAG_LDB(0, xk, 0)
        OPRAG_ADV(xk, xt, xn)
        OPRAG_LDB(1, yk, 0)
        OPRAG_LDA(1, yk, yt, 0)
        OPRAG_ADV(yk, yt, yn)
        OPRAG_LDA(0, xk, xt, BUF)
        OPRAG_LDB(0, xk, BUF)
        OPRAG_ADV(xk, xt, xn)
        vm_wait<2 * AI + 2 * BI>();
      } else {
#pragma unroll
        for (int u = 0; u < LA; ++u) {
          OPRAG_LDA(0, xk, xt, u * BUF)
          OPRAG_LDB(0, xk, u * BUF)
          if constexpr (NP == 2) OPRAG_LDB(1, xk, u * BUF)
          OPRAG_ADV(xk, xt, xn)
          if (xk == 0) xn = tile_ofs((u + 1) / nkt + 1);
        }
        if constexpr (NP == 2)
          vm_wait<AI + 3 * BI>();
        else
          vm_wait<(LA - 1) * (AI + BI)>();
      }
      wg_barrier();
      if (late) wg_barrier();
    };
    // Both groups in step again, every load landed (before the LDS is given up or reused).
    auto finish = [&]() __attribute__((always_inline)) {
      if (!late) wg_barrier();
      vm_wait<0>();
      wg_barrier();
    };

#define OPRAG_RDA(P)                                                                                     \
  _Pragma("unroll") for (int i = 0; i < MS; ++i) {                                                       \
    af[i][0] = *reinterpret_cast<const V*>(smem + cur + (P) * RAP + fa + c0 + i * 2048);                 \
    af[i][1] = *reinterpret_cast<const V*>(smem + cur + (P) * RAP + fa + c1 + i * 2048);                 \
  }
#define OPRAG_RDB(P)                                                                                     \
  _Pragma("unroll") for (int j = 0; j < NS; ++j) {                                                       \
    bf[P][j][0] = *reinterpret_cast<const V*>(smem + cur + (P) * RBP + fb + c0 + j * 2048);              \
    bf[P][j][1] = *reinterpret_cast<const V*>(smem + cur + (P) * RBP + fb + c1 + j * 2048);              \
  }
#define OPRAG_MUL(PA, PB, VM)                                                                            \
  vm_wait<VM>();                                                                                         \
  wg_barrier();                                                                                          \
  __builtin_amdgcn_sched_barrier(0);                                                                     \
  __builtin_amdgcn_s_setprio(1);                                                                         \
  _Pragma("unroll") for (int s = 0; s < 2; ++s) _Pragma("unroll") for (int i = 0; i < MS; ++i)           \
      _Pragma("unroll") for (int j = 0; j < NS; ++j) acc[(PA) * MS + i][(PB) * NS + j] =                 \
          M::run(af[i][s], bf[PB][j][s], acc[(PA) * MS + i][(PB) * NS + j]);                             \
  __builtin_amdgcn_s_setprio(0);                                                                         \
  __builtin_amdgcn_sched_barrier(0);                                                                     \
  wg_barrier();                                                                                          \
  __builtin_amdgcn_sched_barrier(0);

    // The epilogue of a (row part, query part) of the finished tile: acc[i][j][r] is row
    // tile0 + 16 (MT wm + i) + 4 (lane / 16) + r against query slot qn0 + 16 j (tile0 = row_begin + trow).
    int trow = 0;                                     // the tile's first row, from row_begin
    const int rows = (int)(row_end - row_begin);
    [[maybe_unused]] const long long unit0 = chunk * a.upc;  // UNITS: the chunk's first
    bool full = false;                                // every row of the tile exists (uniform)
    [[maybe_unused]] f32x4 mq, mw[8];                 // MAX, MT 1: the lane's maxima of 4 tiles, of 32
    [[maybe_unused]] float th[NT];                    // FILT: the thresholds, for the tile
    int lim = 0, t = 0;                               // row 16 i + r of the lane exists iff < lim
    const int row0 = wm * MT * 16 + (lane >> 4) * 4;  // tile offset of the lane's (i, r) = (0, 0)
    auto epilogue = [&](auto pa, auto pb) __attribute__((always_inline)) {
      constexpr int PA = decltype(pa)::value, PB = decltype(pb)::value;
#pragma unroll
      for (int jj = 0; jj < NS; ++jj) {
        const int j = PB * NS + jj, q = q0 + qn0 + j * 16;
        if constexpr (MAX) {
          // m[i]: the largest score of subtile i's rows, NaN where none exists
          float m[MS];
#pragma unroll
          for (int i = 0; i < MS; ++i) {
            const f32x4 x = acc[PA * MS + i][j];
            if (full) {
              m[i] = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(x[0], x[1]), x[2]), x[3]);
            } else {
              m[i] = __builtin_nanf("");
#pragma unroll
              for (int r = 0; r < 4; ++r) m[i] = (PA * MS + i) * 16 + r < lim ? __builtin_fmaxf(m[i], x[r]) : m[i];
            }
          }
          // the lane's running maximum over the chunk
          float x = PA == 0 && t == 0 ? __builtin_nanf("") : dmx[j];
#pragma unroll
          for (int i = 0; i < MS; ++i) x = __builtin_fmaxf(x, m[i]);
          dmx[j] = x;
          if constexpr (MT == 1) {
            // One group per lane and tile (or unit of tiles).  A store makes the counted waits after it wait
            // for its reply (2.7 us a time: 16 queries over 1 M x 1,024 rows, 374 us with a store in every
            // fourth tile, 355 now), so the maxima of 32 units are kept and leave together, the four
            // lanes of a query exchanging them for 16 bytes of one unit each.
            static_assert(NT == 1);
            const int s = UNITS ? t >> a.unit_sh : t;  // the tile or unit, in the chunk and in all
            const long long unit = UNITS ? unit0 + s : j0 + t;
            float g = m[0];                            // the group so far
            bool whole = true;                         // (workgroup-uniform) the unit ends here
            if constexpr (UNITS) {
              const int um = (1 << a.unit_sh) - 1;
              if ((t & um) != 0) g = __builtin_fmaxf(dmn[0], g);
              dmn[0] = g;
              whole = t == n_tiles - 1 || (t & um) == um;
            }
            if (n_tiles == 1) {  // workgroup-uniform: nothing to wait for later, and little code to fetch
              if (a.mx != nullptr && q < a.nq)
                a.mx[(long long)q * a.mx_ld + unit * (S::WM * 4) + wm * 4 + (lane >> 4)] = g;
            } else if (whole) {
              const int e = s & 3, tq = (s >> 2) & 7;
              mq[0] = e == 0 ? g : mq[0];
              mq[1] = e == 1 ? g : mq[1];
              mq[2] = e == 2 ? g : mq[2];
              mq[3] = e == 3 ? g : mq[3];
              const bool end = t == n_tiles - 1;
              if (a.mx != nullptr && (e == 3 || end)) {
#pragma unroll
                for (int u = 0; u < 8; ++u)
                  if (tq == u) mw[u] = mq;
                if (end || (tq == 7 && e == 3)) {
                  const int h = lane >> 4;
                  float* dst = a.mx + (long long)q * a.mx_ld + (unit - (s & 31)) * (S::WM * 4) + wm * 4;
#pragma unroll
                  for (int u = 0; u < 8; ++u) {
                    if (4 * u > (s & 31)) break;
                    float y[4];  // from lane h ^ o of the query, for unit 4 u + h
#pragma unroll
                    for (int o = 0; o < 4; ++o) {
                      const int c = h ^ o;
                      const float x = c & 2 ? (c & 1 ? mw[u][3] : mw[u][2]) : (c & 1 ? mw[u][1] : mw[u][0]);
                      y[o] = o == 0 ? x : __shfl_xor(x, 16 * o);
                    }
                    f32x4 v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                      const int c = h ^ r;
                      v[r] = c & 2 ? (c & 1 ? y[3] : y[2]) : (c & 1 ? y[1] : y[0]);
                    }
                    if (q < a.nq && 4 * u + h <= (s & 31))
                      *reinterpret_cast<f32x4*>(dst + (long long)(4 * u + h) * (S::WM * 4)) = v;
                  }
                }
              }
            }
          } else if constexpr (UNITS) {
            static_assert(MT == 2 && MP == 1);
            const int um = (1 << a.unit_sh) - 1;
            const float y = __builtin_fmaxf(m[0], m[1]);
            dmn[j] = (t & um) == 0 ? y : __builtin_fmaxf(dmn[j], y);
            if ((t == n_tiles - 1 || (t & um) == um) && q < a.nq)
              a.mx[(long long)q * a.mx_ld + (unit0 + (t >> a.unit_sh)) * (S::WM * 4) + wm * 4 + (lane >> 4)] = dmn[j];
          } else if (a.mx != nullptr && q < a.nq) {
            // the lane's groups of a query are consecutive: MT / gs of them, MS / gs in this part
            // (gs 8: one for both parts)
            const int gs = a.mx_gs, gl = MT / gs;  // launch-uniform
            float* dst = a.mx + (long long)q * a.mx_ld + (long long)(j0 + t) * (S::WM * 4 * gl) + (wm * 4 + (lane >> 4)) * gl +
                         (gs <= MS ? PA * (MS / gs) : 0);
            if (gs == 1) {
              if constexpr (MS == 4)
                *reinterpret_cast<float4*>(dst) = make_float4(m[0], m[1], m[2], m[3]);
              else if constexpr (MS == 2)
                *reinterpret_cast<float2*>(dst) = make_float2(m[0], m[1]);
            } else if (gs == 2) {
              if constexpr (MS == 4)
                *reinterpret_cast<float2*>(dst) = make_float2(__builtin_fmaxf(m[0], m[1]), __builtin_fmaxf(m[2], m[3]));
              else if constexpr (MS == 2)
                dst[0] = __builtin_fmaxf(m[0], m[1]);
            } else if constexpr (MS == 4) {
              const float y = __builtin_fmaxf(__builtin_fmaxf(m[0], m[1]), __builtin_fmaxf(m[2], m[3]));
              if (gs == 4) {
                dst[0] = y;
              } else if constexpr (MP == 2) {  // gs 8
                if (PA == 1) dst[0] = __builtin_fmaxf(dmn[j], y);
                dmn[j] = y;
              }
            }
          }
          if (a.cmx != nullptr && PA == MP - 1 && t == n_tiles - 1 && q < a.nq)
            a.cmx[(long long)q * a.cmx_ld + chunk * (S::WM * 4) + (wm * 4 + (lane >> 4))] = x;
        } else if constexpr (SCORES) {
          // The scores wait in LDS (each lane's for itself) until the chunk's end: a store has the counted waits
          // after it wait for its reply.  (In registers the unrolled code cost 1.5 us with 16 tiles, 4 with 32.)
          static_assert(MT == 1 && NT == 1);
          f32x4 x = acc[0][0];
          if (!full) {
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = r < lim ? x[r] : __builtin_nanf("");
          }
          dmx[0] = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(t == 0 ? __builtin_nanf("") : dmx[0], x[0]),
                                                   __builtin_fmaxf(x[1], x[2])), x[3]);
          if (q < a.nq) {
            f32x4* held = reinterpret_cast<f32x4*>(smem + NBUF * BUF) + ((lane & 15) * BM + row0) / 4;
            const int step = a.nq * BM / 4;
            held[t * step] = x;
            if (t == n_tiles - 1) {  // workgroup-uniform
              float* dst = a.dump + (long long)q * a.dump_ld + row_begin + row0;
#pragma unroll 2
              for (int u = 0; u < n_tiles; ++u)
                if (u * BM + row0 < rows) *reinterpret_cast<f32x4*>(dst + u * BM) = held[u * step];
              a.cmx[(long long)q * a.cmx_ld + chunk * (S::WM * 4) + (wm * 4 + (lane >> 4))] = dmx[0];
            }
          }
        } else if constexpr (MODE == kTileDump) {
          if (q < a.nq) {
            float* dst = a.dump + (long long)q * a.dump_ld + row_begin + trow + row0;
#pragma unroll
            for (int i = PA * MS; i < (PA + 1) * MS; ++i) {
              if (full || i * 16 + 3 < lim) {
                *reinterpret_cast<f32x4*>(dst + i * 16) = acc[i][j];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  dmn[j] = fminf(dmn[j], acc[i][j][r]);
                  dmx[j] = fmaxf(dmx[j], acc[i][j][r]);
                }
              } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                  if (i * 16 + r < lim) {
                    dst[i * 16 + r] = acc[i][j][r];
                    dmn[j] = fminf(dmn[j], acc[i][j][r]);
                    dmx[j] = fmaxf(dmx[j], acc[i][j][r]);
                  }
              }
            }
          }
        } else if constexpr (MODE == kTileFilt) {
          // Hits are rare: the maximum of the lane's scores against the threshold first.  (The code
          // for hits is kept small: unrolled over the scores, it misses the instruction cache on
          // every hit, which took half of the kernel's time over 8.4 M rows.)
          float m = acc[PA * MS][j][0];
#pragma unroll
          for (int i = 0; i < MS; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) m = __builtin_fmaxf(m, acc[PA * MS + i][j][r]);
          if (__ballot(m >= th[j]) == 0ull) continue;
          unsigned hm = 0u;  // the lane's hits, bit 4 i + r
#pragma unroll
          for (int i = 0; i < MS; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) hm |= (acc[PA * MS + i][j][r] >= th[j] ? 1u : 0u) << (i * 4 + r);
          if (!full) {
#pragma unroll
            for (int i = 0; i < MS; ++i)
#pragma unroll
              for (int r = 0; r < 4; ++r) hm &= (PA * MS + i) * 16 + r < lim ? ~0u : ~(1u << (i * 4 + r));
          }
          int pos = hm ? atomicAdd(qcnt, __popc(hm)) : 0;
          while (hm) {
            const int b = __builtin_ctz(hm);
            hm &= hm - 1u;
            float y[MS];
#pragma unroll
            for (int i = 0; i < MS; ++i) {
              const f32x4 v = acc[PA * MS + i][j];
              y[i] = b & 2 ? (b & 1 ? v[3] : v[2]) : (b & 1 ? v[1] : v[0]);
            }
            float x = y[0];
            if constexpr (MS >= 2) x = b & 4 ? y[1] : y[0];
            if constexpr (MS == 4) x = b & 8 ? (b & 4 ? y[3] : y[2]) : x;
            const unsigned row = (unsigned)(row0 + PA * MS * 16 + (b >> 2) * 16 + (b & 3));  // in the tile
            if (pos < Q::CAP) {
              queue[pos] = ((u64)__float_as_uint(x) << 32) | (u64)(((unsigned)(t * BM) + row) << 8 | (unsigned)(qn0 + j * 16));
            } else {  // the queue is full until the next flush: straight to the query's buffer
              const long long g = atomicAdd(a.ccnt + q, 1);
              if (g < a.cap)
                a.cbuf[(long long)q * a.cap + g] = composite(x, (uint32_t)row_begin + (uint32_t)trow + row);
              else
                qth[qn0 + j * 16] = __builtin_inff();
            }
            ++pos;
          }
        }
      }
    };
    constexpr std::integral_constant<int, 0> I0{};
    constexpr std::integral_constant<int, 1> I1{};
    // One stage.  Each phase: read its operands, issue loads, wait for what the next phase
    // reads, barrier, MFMAs, barrier.  A part is loaded over again two or more phases after its
    // last reads, when both groups are done with it.  PAR: the stage's buffer (MP 2).
    auto stage = [&](auto PAR) __attribute__((always_inline)) {
      if constexpr (MP == 2) {
        constexpr int cur = decltype(PAR)::value * BUF, oth = BUF - cur;
        OPRAG_RDB(0)
        OPRAG_RDA(0)
        OPRAG_LDB(1, yk, oth)
        OPRAG_MUL(0, 0, (2 * AI + 2 * BI))
        OPRAG_RDB(1)
        OPRAG_LDA(1, yk, yt, oth)
        OPRAG_ADV(yk, yt, yn)
        OPRAG_MUL(0, 1, (2 * AI + 2 * BI))
        OPRAG_RDA(1)
        OPRAG_LDA(0, xk, xt, cur)
        OPRAG_MUL(1, 1, (2 * AI + 2 * BI))
        OPRAG_LDB(0, xk, cur)
        OPRAG_ADV(xk, xt, xn)
        OPRAG_MUL(1, 0, (2 * AI + 2 * BI))
      } else {
        const int cur = cur1;
        OPRAG_RDB(0)
        OPRAG_RDA(0)
        OPRAG_LDA(0, xk, xt, nxt)
        OPRAG_LDB(0, xk, nxt)
        if constexpr (NP == 2) {
          OPRAG_MUL(0, 0, (2 * AI + 3 * BI))
          OPRAG_RDB(1)
          OPRAG_LDB(1, xk, nxt)
          OPRAG_ADV(xk, xt, xn)
          OPRAG_MUL(0, 1, (AI + 3 * BI))
        } else {
          OPRAG_ADV(xk, xt, xn)
          OPRAG_MUL(0, 0, ((LA - 1) * (AI + BI)))
        }
        cur1 = cur == (NBUF - 1) * BUF ? 0 : cur + BUF;
        nxt = nxt == (NBUF - 1) * BUF ? 0 : nxt + BUF;
      }
    };
    start();
    const int ahead = LA / nkt;  // the tile that x has reached when the first one is multiplied
    for (; t < n_tiles; ++t) {
      xn = tile_ofs(t + ahead + 1);
      if constexpr (MP == 2) yn = tile_ofs(t + 1);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (MP == 2) {  // nkt is even
        for (int k = 0; k < nkt; k += 2) {
          stage(I0);
          stage(I1);
        }
      } else {
        for (int k = 0; k < nkt; ++k) stage(I0);
      }
      trow = (int)(tile_row((unsigned)(j0 + t)) - tile_row((unsigned)j0));
      full = trow + BM <= rows;
      lim = min(BM, rows - trow) - row0;
      if constexpr (MODE == kTileFilt) {
#pragma unroll
        for (int j = 0; j < NT; ++j) th[j] = qth[qn0 + j * 16];
      }
      epilogue(I0, I0);
      if constexpr (NP == 2) epilogue(I0, I1);
      if constexpr (MP == 2) {
        epilogue(I1, I1);
        epilogue(I1, I0);
      }

      if constexpr (MODE == kTileFilt) {
        const bool last = t == n_tiles - 1;
        if (last || (t & a.check_mask) == a.check_mask) {  // workgroup-uniform
          if (!late) wg_barrier();  // both groups in step
          lds_barrier();
          const int n = min(*qcnt, Q::CAP);
          if (n > 0 && (last || n >= Q::CAP / 2)) {
            // count per query (an entry's rank among its query's), reserve, write
            if (tid < BN) qhist[tid] = 0;
            lds_barrier();
            constexpr int PT = (Q::CAP + kTileThreads - 1) / kTileThreads;
            int rank[PT];
#pragma unroll
            for (int u = 0; u < PT; ++u) {
              const int e = tid + u * kTileThreads;
              rank[u] = e < n ? atomicAdd(&qhist[(unsigned)queue[e] & 255u], 1) : 0;
            }
            lds_barrier();
            if (tid < BN) {
              const int c = qhist[tid];
              const int b = c > 0 ? atomicAdd(a.ccnt + q0 + tid, c) : 0;
              qbase[tid] = b;
              if ((long long)b + c > a.cap) qth[tid] = __builtin_inff();
            }
            lds_barrier();
#pragma unroll
            for (int u = 0; u < PT; ++u) {
              const int e = tid + u * kTileThreads;
              if (e < n) {
                const u64 x = queue[e];
                const int slot = (int)((unsigned)x & 255u);
                const long long g = (long long)qbase[slot] + rank[u];
                if (g < a.cap)
                  a.cbuf[(long long)(q0 + slot) * a.cap + g] =
                      composite(__uint_as_float((unsigned)(x >> 32)),
                                tile_row(j0 + ((unsigned)x >> 8) / BM) + ((unsigned)x >> 8) % BM);
              }
            }
            lds_barrier();
            if (tid == 0) *qcnt = 0;
            lds_barrier();
          }
          if (late) wg_barrier();  // half a phase apart again
        }
      }
    }
    finish();
    if constexpr (UNITS) {
      // a chunk with a unit less than upc: no rows there
      if (((n_tiles - 1) >> a.unit_sh) + 1 < a.upc) {  // workgroup-uniform
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const int q = q0 + qn0 + j * 16;
          if (q < a.nq)
            a.mx[(long long)q * a.mx_ld + (unit0 + a.upc - 1) * (S::WM * 4) + wm * 4 + (lane >> 4)] = __builtin_nanf("");
        }
      }
    }
#undef OPRAG_MUL
#undef OPRAG_RDA
#undef OPRAG_RDB
#undef OPRAG_LDA
#undef OPRAG_LDB
#undef OPRAG_ADV
  }
  if constexpr (MODE == kTileDump) {
    if (a.dump_mm != nullptr) {  // launch-uniform
      // the four lanes of a query, then the waves that share it, through LDS
      float* red = reinterpret_cast<float*>(smem);  // [WM][BN][2]
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        dmn[j] = fminf(dmn[j], __shfl_xor(dmn[j], 16));
        dmx[j] = fmaxf(dmx[j], __shfl_xor(dmx[j], 16));
        dmn[j] = fminf(dmn[j], __shfl_xor(dmn[j], 32));
        dmx[j] = fmaxf(dmx[j], __shfl_xor(dmx[j], 32));
        if (lane < 16) {
          red[(wm * BN + qn0 + j * 16) * 2] = dmn[j];
          red[(wm * BN + qn0 + j * 16) * 2 + 1] = dmx[j];
        }
      }
      __syncthreads();
      if (tid < BN && q0 + tid < a.nq) {
        float mn = __builtin_inff(), mx = -__builtin_inff();
#pragma unroll
        for (int u = 0; u < S::WM; ++u) {
          mn = fminf(mn, red[(u * BN + tid) * 2]);
          mx = fmaxf(mx, red[(u * BN + tid) * 2 + 1]);
        }
        float* o = a.dump_mm + ((long long)(q0 + tid) * a.n_chunks + chunk) * 2;
        o[0] = mn;
        o[1] = mx;
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// The k best rows of each query from the maxima of MAX mode (or the scores of SCORES), one workgroup per query.  Up to 8,192
// groups are searched directly; of more, every lane's maximum over its chunk (the coarse maxima, at
// most some 8,192 a query) bounds the k-th score from below and says where the groups that reach
// that bound lie, and only those lanes' groups are read.  With the groups ordered by (maximum desc,
// index asc), let c be the k-th: a row of the top k lies in a group with a larger maximum than c's,
// or in a group with c's maximum whose rows come no later than c's tile (k groups up to there each
// hold a row at least as good).  These groups' rows, k of them and the ties in c's tile, are scored
// again with the same matrix instructions in the same order as in the tile kernel, so the scores
// have the same bits, and ranked exactly.  Without groups (fine == nullptr) the coarse maxima are the
// groups, over all of a lane's rows.  With every score at hand (SCORES) the coarse maxima's lanes that reach
// the bound are read back, four rows a word, and the scores that reach it are ranked: 4 us less than with rows
// scored again.
//
// A launch of a few workgroups is bound by latency.  One query over 32,768 rows of 1,024 bf16 (a size that has
// come to select from every score instead) takes 7.0 us from start to end: 1.4 the maxima (the first reads), 0.7 tau, 1.1 the groups' order, 2.6 the
// rows, 0.8 their ranks.  It took 10.7 unrolled over the keys (28 KB of code fetched cold), so the code
// is kept short: the maxima are held as one per 16-byte word, and a word that holds a hit is read
// again; and 8.0 with tau counted by v_readlane and a test before each step's matrix instruction.
// Scattered rows are the dearest reads (about 40 ns each beyond the first few tens, over a long
// index), so groups are small.
// ------------------------------------------------------------------------------------
constexpr int kReThreads = 256;
constexpr int kReWords = 8;                              // 16-byte words per thread and step
constexpr int kReCand = 64;                              // groups ranked by a wave
constexpr int kReList = 256;                             // groups scored: k + the groups of one tile
constexpr int kReRows = 1024;                            // rows ranked together

template <int DT, int KIND>
__global__ __launch_bounds__(kReThreads, 4) void rescore_kernel(RescoreArgs a) {
  constexpr bool UNITS = KIND == kTileUnits, SCORES = KIND == kTileScores;
  if (a.gate != nullptr && *a.gate == 0) return;
  using M = Mfma<DT>;
  using V = typename M::V;
  constexpr int NT = kReThreads, NW = NT / 64;
  __shared__ u64 cand[kReRows];          // groups, later a batch's rows
  extern __shared__ __attribute__((aligned(16))) unsigned char qrow[];  // the query
  __shared__ __attribute__((aligned(16))) float gmax[NW][64], gsum[NW][64];
  __shared__ int clist[kReCand];
  __shared__ int list[kReList];
  __shared__ u64 best[2][kMaxK];
  __shared__ u64 red[NW];
  __shared__ int s_n, s_nh, s_nl, s_k[2];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const long long q = blockIdx.x;
  const bool two = SCORES || a.two != 0;  // launch-uniform: groups searched through the coarse maxima
  const bool by_chunk = !SCORES && a.fine == nullptr;  // the coarse maxima are the groups
  const int k = a.k;
  const int rowb = a.d * (DT == kDtypeF32 ? 4 : 2);
  const int np = rowb / 16;  // 16-byte pieces of a row
  const float nan = __builtin_nanf("");
  // 16-byte word i of a row of n maxima (16-byte aligned), NaN past it
  auto word_of = [&](const float* row, int n, int i) __attribute__((always_inline)) {
    float4 x = 4 * i < n ? reinterpret_cast<const float4*>(row)[i] : make_float4(nan, nan, nan, nan);
    if (4 * i + 4 > n) {
      x.y = 4 * i + 1 < n ? x.y : nan;
      x.z = 4 * i + 2 < n ? x.z : nan;
      x.w = 4 * i + 3 < n ? x.w : nan;
    }
    return x;
  };
  const float* groups = by_chunk ? a.coarse + q * a.coarse_ld : a.fine + q * a.fine_ld;
  const int n_groups = by_chunk ? a.n_coarse : a.n_fine;
  const float* coarse = two ? a.coarse + q * a.coarse_ld : groups;  // searched first
  const int n_coarse = two ? a.n_coarse : n_groups;
  float wm[kReWords];                                  // the words' maxima (of the last step)
  float m4[4] = {kNegInf, kNegInf, kNegInf, kNegInf};  // the thread's, by element
  auto load = [&](int i0) __attribute__((always_inline)) {
    float4 x[kReWords];
#pragma unroll
    for (int u = 0; u < kReWords; ++u) x[u] = word_of(coarse, n_coarse, i0 + NT * u);
#pragma unroll
    for (int u = 0; u < kReWords; ++u) {
      m4[0] = __builtin_fmaxf(m4[0], x[u].x);
      m4[1] = __builtin_fmaxf(m4[1], x[u].y);
      m4[2] = __builtin_fmaxf(m4[2], x[u].z);
      m4[3] = __builtin_fmaxf(m4[3], x[u].w);
      wm[u] = __builtin_fmaxf(__builtin_fmaxf(x[u].x, x[u].y), __builtin_fmaxf(x[u].z, x[u].w));
    }
  };
  // 1. the query to LDS, the coarse maxima
  if (t == 0) {
    s_n = 0;
    s_nh = 0;
    s_nl = 0;
    s_k[0] = s_k[1] = 0;
  }
  if constexpr (!SCORES) {
    const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const unsigned char*>(a.Q) + q * rowb);
    for (int i = t; i < np; i += NT) reinterpret_cast<u32x4*>(qrow)[i] = src[i];
  }
  const int steps = max(1, (n_coarse + 4 * NT * kReWords - 1) / (4 * NT * kReWords));
  for (int s = 0; s < steps; ++s) load(t + s * NT * kReWords);
  // 2. k <= 16: tau, the k-th largest of 64 maxima over disjoint sets of the coarse ones (element e of
  // the words i with i % 16 = j: set 4 j + e, so the first 64 fall in sets of their own): at least k
  // lanes, and so k groups, reach it (-inf: every group).
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    m4[e] = __builtin_fmaxf(m4[e], __shfl_xor(m4[e], 16));
    m4[e] = __builtin_fmaxf(m4[e], __shfl_xor(m4[e], 32));
  }
  if (lane < 16) *reinterpret_cast<float4*>(&gmax[w][4 * lane]) = make_float4(m4[0], m4[1], m4[2], m4[3]);
  __syncthreads();
  float tau = kNegInf;
  if (k <= 16) {  // every wave finds it for itself
    float me = gmax[0][lane];
#pragma unroll
    for (int u = 1; u < NW; ++u) me = __builtin_fmaxf(me, gmax[u][lane]);
    int ge = 0;
    gsum[w][lane] = me;  // (from LDS: by v_readlane the counts took 1.4 us)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll 8
    for (int u = 0; u < 16; ++u) {
      const float4 x = *reinterpret_cast<const float4*>(&gsum[w][4 * u]);
      ge += (x.x >= me ? 1 : 0) + (x.y >= me ? 1 : 0) + (x.z >= me ? 1 : 0) + (x.w >= me ? 1 : 0);
    }
    tau = wave_max(ge >= k ? me : kNegInf);
  }
  // 3. the lanes that reach tau, and their groups that do, as composites of maxima and indices
  auto offer = [&](float v, int g) __attribute__((always_inline)) {
    if (v >= tau) {
      const int p = atomicAdd(&s_n, 1);
      if (p < kReCand) cand[p] = composite(v, (uint32_t)g);
    }
  };
  for (int s = 0; s < steps; ++s) {
    const int i0 = t + s * NT * kReWords;
    if (steps > 1) load(i0);
    unsigned hm = 0u;
#pragma unroll
    for (int u = 0; u < kReWords; ++u) hm |= (wm[u] >= tau ? 1u : 0u) << u;
    for (; hm != 0u; hm &= hm - 1u) {
      const int i = i0 + NT * __builtin_ctz(hm);
      const float4 x = word_of(coarse, n_coarse, i);
      const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (!two) {
          offer(v[e], 4 * i + e);
        } else if (v[e] >= tau) {
          const int p = atomicAdd(&s_nh, 1);
          if (p < kReCand) clist[p] = 4 * i + e;
        }
      }
    }
  }
  __syncthreads();
  const int tb_sh = a.gpt_sh;   // groups of a tile (or unit of tiles, or, coarse, of a chunk): 1 << gpt_sh
  const int lanes_sh = a.lanes_sh, gl_sh = a.gl_sh;
  // chunk * tiles / n_chunks, in 32 bits
  auto first_tile = [&](int chunk) { return chunk * a.least + (int)((unsigned)(chunk * a.spare) / (unsigned)a.n_chunks); };
  if (two) {
    const int nh = s_nh, per = (UNITS ? a.upc : a.most) << gl_sh;  // groups of a lane over its chunk
    if constexpr (SCORES) {
      if (nh <= kReCand)
        for (int p = t; p < nh * per; p += NT) {
          const int c = clist[p / per], u = p % per, chunk = c >> lanes_sh, l = c & ((1 << lanes_sh) - 1);
          const long long row = scores_chunk_row(chunk, a.n_rows, a.n_chunks) + u * a.tile_rows + (l >> 2) * 16 + (l & 3) * 4;
          if (row < min(scores_chunk_row(chunk + 1, a.n_rows, a.n_chunks), a.n_rows)) {
            const float4 x = *reinterpret_cast<const float4*>(groups + row);  // (NaN past the last row)
            const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) offer(v[e], (int)row + e);
          }
        }
    } else if (nh <= kReCand)
      for (int p = t; p < nh * per; p += NT) {
        const int c = clist[p / per], u = p % per, chunk = c >> lanes_sh, l = c & ((1 << lanes_sh) - 1);
        const int unit0 = UNITS ? chunk * a.upc : first_tile(chunk);  // tiles or units
        const int end = UNITS ? unit0 + a.upc : first_tile(chunk + 1);
        const int unit = unit0 + (u >> gl_sh);
        if (unit < end) {
          const int g = (unit << tb_sh) + (l << gl_sh) + (u & ((1 << gl_sh) - 1));
          offer(groups[g], g);
        }
      }
    __syncthreads();
  }
  const bool few = s_n <= kReCand && s_nh <= kReCand;  // workgroup-uniform
  auto wanted = [&](u64 c, u64 star) {
    return c >= star || (comp_key(c) == comp_key(star) && (comp_row(c) >> tb_sh) <= (comp_row(star) >> tb_sh));
  };
  // 4. the k-th group, and the groups to score
  int nl = 0;
  if (few) {  // every wave for itself: lane l holds candidate l
    const int nc = s_n, need = min(k, nc);
    const u64 me = lane < nc ? cand[lane] : 0ull;
    int r = 0;
#pragma unroll 4
    for (int o = 0; o < nc; ++o) r += cand[o] > me ? 1 : 0;
    if constexpr (SCORES) {
      if (w == 0 && lane < nc && r < k) {
        a.out_ids[q * k + r] = (long long)comp_row(me);
        a.out_scores[q * k + r] = comp_score(me);
      }
      for (int r2 = need + t; r2 < k; r2 += NT) {
        a.out_ids[q * k + r2] = -1ll;
        a.out_scores[q * k + r2] = kNegInf;
      }
      return;
    }
    const u64 is = __ballot(lane < nc && r == need - 1);
    if (is != 0ull) {
      const u64 star = readlane64(me, __builtin_ctzll(is));
      const bool take = lane < nc && wanted(me, star);
      const u64 bal = __ballot(take);
      nl = __popcll(bal);
      // (each wave writes the same entries)
      if (take) list[__popcll(bal & ((1ull << lane) - 1ull))] = (int)comp_row(me);
    }
  } else {
    // many groups at tau (ties), or k > 16: the k-th group by k rounds of maxima over all groups
    const float* all = groups;
    const int n = n_groups, n4 = (n + 3) / 4;
    u64 last = ~0ull;
    for (int r = 0; r < k; ++r) {
      u64 x = 0ull;
#pragma unroll 2
      for (int i = t; i < n4; i += NT) {
        const float4 y = word_of(all, n, i);
        const float v[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const u64 c = v[e] >= tau ? composite(v[e], (uint32_t)(4 * i + e)) : 0ull;
          if (c < last) x = umax64(x, c);
        }
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) x = umax64(x, shfl_xor64(x, o));
      if (lane == 0) red[w] = x;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < NW; ++u) x = umax64(x, red[u]);
      if constexpr (SCORES) {
        if (t == 0) {
          a.out_ids[q * k + r] = x != 0ull ? (long long)comp_row(x) : -1ll;
          a.out_scores[q * k + r] = x != 0ull ? comp_score(x) : kNegInf;
        }
      }
      if (x != 0ull) last = x;  // fewer than k groups: the last one
      __syncthreads();
    }
    if constexpr (SCORES) return;
    const u64 star = last;
    for (int i = t; i < n4; i += NT) {
      const float4 y = word_of(all, n, i);
      const float v[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (v[e] >= tau && wanted(composite(v[e], (uint32_t)(4 * i + e)), star)) {
          const int p = atomicAdd(&s_nl, 1);
          if (p < kReList) list[p] = 4 * i + e;
        }
    }
    __syncthreads();
    nl = min(s_nl, kReList);
  }
  __syncthreads();  // every wave has read the candidates
  // 5. score the rows of the listed groups, 16 rows per wave and step, and keep the k best
  const int g_rows = by_chunk ? (4 << a.mt_sh) * a.most : 4 << (UNITS ? a.gs_sh + a.unit_sh : a.gs_sh);  // rows of a group
  const int total = nl * g_rows;  // (of distinct rows)
  const int nks = (rowb + 127) / 128 * 2;      // 64-byte steps
  const unsigned char* X = static_cast<const unsigned char*>(a.X);
  // row f of the list: row u = f % g_rows of group list[f / g_rows] (n_rows: none)
  auto row_of = [&](int f) -> long long {
    const int e = (int)((unsigned)f / (unsigned)g_rows), g = list[e], u = f - e * g_rows;
    int l, sub = u >> 2, tile;  // lane of the tile (wave and quarter), subtile
    if (!by_chunk) {
      const int rem = g & ((1 << tb_sh) - 1);
      l = rem >> gl_sh;
      sub += (rem & ((1 << gl_sh) - 1)) << a.gs_sh;
      tile = g >> tb_sh;
      if constexpr (UNITS) {
        const int chunk = tile / a.upc;
        tile = first_tile(chunk) + ((tile - chunk * a.upc) << a.unit_sh) + (sub >> a.mt_sh);
        sub &= (1 << a.mt_sh) - 1;
        if (tile >= first_tile(chunk + 1)) return a.n_rows;
      }
    } else {
      const int chunk = g >> lanes_sh;
      l = g & ((1 << lanes_sh) - 1);
      tile = first_tile(chunk) + (sub >> a.mt_sh);
      sub &= (1 << a.mt_sh) - 1;
      if (tile >= first_tile(chunk + 1)) return a.n_rows;
    }
    return (long long)tile * a.tile_rows + (l >> 2) * (16 << a.mt_sh) + sub * 16 + (l & 3) * 4 + (u & 3);
  };
  int kept = 0, cur = 0;  // rows kept so far, in best[cur] (by rank)
  for (int base = 0; base < total; base += kReRows) {
    const int nb = min(kReRows, total - base);
    for (int u0 = w * 16; u0 < nb; u0 += 16 * NW) {
      const int f = u0 + (lane & 15);
      long long row = f < nb ? row_of(base + f) : 0;
      const bool ok = f < nb && row < a.n_rows;
      if (!ok) row = 0;
      const unsigned char* xr = X + row * rowb + (lane >> 4) * 16;
      const unsigned char* qr = qrow + (lane >> 4) * 16;
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
      // rows 8 steps ahead of their use, two sets of registers in turn (past the last step: it again)
      constexpr int PF = 8;
      V xv[2][PF];
      auto piece = [&](const unsigned char* p, int st) __attribute__((always_inline)) {
        if constexpr (DT == kDtypeF32) {  // a row may end inside a 128-byte stage: zeros past it
          const u32x4 zero = {0u, 0u, 0u, 0u};
          return __builtin_bit_cast(V, st * 4 + (lane >> 4) < np ? *reinterpret_cast<const u32x4*>(p + st * 64) : zero);
        } else {
          return *reinterpret_cast<const V*>(p + st * 64);
        }
      };
      auto fetch = [&](V (&v)[PF], int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < PF; ++u) v[u] = piece(xr, min(s0 + u, nks - 1));
      };
      // (a test per step would wait for each step's 16 bytes of the query in turn)
      auto multiply = [&](const V (&v)[PF], int s0) __attribute__((always_inline)) {
        if (s0 + PF <= nks) {  // wave-uniform
          V qv[PF];
#pragma unroll
          for (int u = 0; u < PF; ++u) qv[u] = piece(qr, s0 + u);
#pragma unroll
          for (int u = 0; u < PF; ++u) acc = M::run(v[u], qv[u], acc);
        } else {
#pragma unroll
          for (int u = 0; u < PF; u += 2)  // nks is even
            if (s0 + u < nks) {
              acc = M::run(v[u], piece(qr, s0 + u), acc);
              acc = M::run(v[u + 1], piece(qr, s0 + u + 1), acc);
            }
        }
      };
      fetch(xv[0], 0);
      for (int s0 = 0; s0 < nks; s0 += 2 * PF) {
        fetch(xv[1], s0 + PF);
        multiply(xv[0], s0);
        if (s0 + 2 * PF < nks) fetch(xv[0], s0 + 2 * PF);
        multiply(xv[1], s0 + PF);
      }
      // every column holds the query; row 4 (lane / 16) + c of the 16 is element c
      const int c = lane & 15;
      const float x = c == 0 ? acc[0] : (c == 1 ? acc[1] : (c == 2 ? acc[2] : acc[3]));
      const int src = (lane >> 4) * 4 + (c & 3);
      const long long rr = __shfl(row, src);
      const bool okr = __shfl((int)ok, src) != 0;
      if (c < 4 && u0 + src < nb) cand[u0 + src] = okr && x == x ? composite(x, (uint32_t)rr) : 0ull;
    }
    __syncthreads();
    // ranks among the batch and the rows kept before; ranks below k are kept (composites of
    // distinct rows are distinct; 0 marks no row and is never kept)
    const int all = nb + kept;
    auto entry = [&](int i) { return i < nb ? cand[i] : best[cur][i - nb]; };
    int lg = 0;
    while (lg < 4 && (all << (lg + 1)) <= NT) ++lg;
    const int Lc = 1 << lg, p = t & (Lc - 1);
    const bool final = base + kReRows >= total;
    int mine = 0;
    for (int j0 = 0; j0 < all; j0 += NT >> lg) {
      const int jc = j0 + (t >> lg);
      int r = 0;
      u64 me = 0ull;
      if (jc < all) {
        me = entry(jc);
#pragma unroll 4
        for (int o = p; o < all; o += Lc) r += entry(o) > me ? 1 : 0;
      }
      // sums over Lc consecutive lanes
      if (lg >= 1) r += dpp<0xB1>(r);
      if (lg >= 2) r += dpp<0x4E>(r);
      if (lg >= 3) r += dpp<0x141>(r);
      if (lg >= 4) r += dpp<0x140>(r);
      if (jc < all && p == 0 && me != 0ull && r < k) {
        if (final) {
          a.out_ids[q * k + r] = (long long)comp_row(me);
          a.out_scores[q * k + r] = comp_score(me);
        } else {
          best[cur ^ 1][r] = me;
        }
        ++mine;
      }
    }
    if (mine) atomicAdd(&s_k[cur], mine);
    __syncthreads();
    kept = s_k[cur];
    cur ^= 1;
    if (t == 0) s_k[cur] = 0;  // next added to after the barrier that follows the next batch's scores
  }
  for (int r = kept + t; r < k; r += NT) {
    a.out_ids[q * k + r] = -1ll;
    a.out_scores[q * k + r] = kNegInf;
  }
}

}  // namespace

// Launches of one storage type (the file that includes this header instantiates them).
template <int DT>
hipError_t tile_launch(int shape, int mode, long long grid, DenseArgs& arg, hipStream_t s, hipEvent_t ev0,
                       hipEvent_t ev1) {
  void (*fn)(DenseArgs) = nullptr;
#define OPRAG_TILE(I, BM, BN)                                                  \
  if (shape == I)                                                              \
    fn = mode == kTileMax    ? dense_tile_kernel<DT, BM, BN, kTileMax>         \
         : mode == kTileFilt ? dense_tile_kernel<DT, BM, BN, kTileFilt>        \
         : mode == kTileDump ? dense_tile_kernel<DT, BM, BN, kTileDump>        \
         : mode == kTileSample ? dense_tile_kernel<DT, BM, BN, kTileSample>    \
                             : nullptr;
  OPRAG_TILE(0, 128, 16)
  OPRAG_TILE(1, 128, 64)
  OPRAG_TILE(2, 128, 128)
  if constexpr (DT != kDtypeF32) {
    OPRAG_TILE(3, 256, 128)
    OPRAG_TILE(4, 128, 256)
    OPRAG_TILE(5, 256, 256)
  }
  if (mode == kTileScores) fn = shape == 0 ? dense_tile_kernel<DT, 128, 16, kTileScores> : nullptr;
  if (mode == kTileUnits)
    fn = shape == 0   ? dense_tile_kernel<DT, 128, 16, kTileUnits>
         : shape == 1 ? dense_tile_kernel<DT, 128, 64, kTileUnits>
                      : nullptr;
#undef OPRAG_TILE
  if (fn == nullptr) return hipErrorInvalidValue;
  void* params[] = {&arg};
  // With timing events the launch carries them in its dispatch packet: they are stamped when
  // the kernel itself starts and ends.
  return ev0 ? hipExtLaunchKernel(reinterpret_cast<const void*>(fn), dim3((unsigned)grid), dim3(kTileThreads), params, 0,
                                  s, ev0, ev1, 0)
             : hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3((unsigned)grid), dim3(kTileThreads), params, 0, s);
}

template <int DT>
hipError_t rescore_launch(const RescoreArgs& a, int nq, hipStream_t s) {
  const size_t lds = (size_t)a.d * (DT == kDtypeF32 ? 4 : 2);
  if (a.scores)
    hipLaunchKernelGGL((rescore_kernel<DT, kTileScores>), dim3((unsigned)nq), dim3(kReThreads), 0, s, a);
  else if (a.unit_sh > 0)
    hipLaunchKernelGGL((rescore_kernel<DT, kTileUnits>), dim3((unsigned)nq), dim3(kReThreads), lds, s, a);
  else
    hipLaunchKernelGGL((rescore_kernel<DT, kTileMax>), dim3((unsigned)nq), dim3(kReThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace oprag

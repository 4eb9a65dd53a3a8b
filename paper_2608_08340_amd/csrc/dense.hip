// Dense exact top-k: R_k = Op_retrieve(q, I) (Section 3.2, "Retrieval"): inner-product
// scores of every query against every indexed unit vector, by matrix products over the
// embedding matrix, then partial top-k selection (Section 4.4).
//
// Every search scores with the tiled matrix-core kernel of dense_tile.h and differs in what
// the tiles hand on:
//  - up to 32,768 rows, and for k <= 16 few scores in all: every score; one workgroup per query selects
//    from its score row;
//  - up to 16 queries, k <= 16, over somewhat longer indexes: every score and their maxima over what a
//    lane has of a chunk, through which one workgroup per query finds the best;
//  - k <= 16 otherwise: the largest score of every group of 4 to 64 (for long indexes more) rows; the k
//    best groups of a query are found and their rows scored again (rescore_kernel);
//  - otherwise (k > 16, or more than 64 queries over a long index): threshold levels over growing
//    shares of the rows.  The first level's group maxima give each query a lower bound of its k-th
//    score; the next level collects only the rows that reach it, whose k-th score is the next
//    threshold; the last level completes the index.  Every level's rows are spread over the index:
//    rows come in the order in which documents were ingested, and with levels over prefixes a topic of
//    more adjacent rows than a buffer holds overflowed it (1 M x 768 bf16, 1,024 queries, k = 10: rows
//    in topics of 4,096, 6.5 ms by prefixes and 1.27 spread out; in random order 1.30 and 1.31).
#include <algorithm>
#include <type_traits>

#include "mfma.h"
#include "oprag_internal.h"
#include "select.h"

namespace oprag {

namespace {

using namespace dev;

// ------------------------------------------------------------------------------------
// Exact top-k (sorted) of a query's candidate keys, or (SCORES) of a row of n_scores fp32 scores,
// the position being the row id (NaN scores are never selected).  One workgroup
// of NT threads per query: 1,024 when one round of workgroups covers the batch (the query's
// latency counts), 256 for larger batches (more queries per CU at once).  Keys are unique
// composites (row ids are), so exactly min(k, n) keys qualify.  Buffers of up to 4,096 keys
// are read once (all loads in flight) and kept in registers.  The 256 groups of NT / 256
// adjacent threads take their largest key, and tau = the need-th largest of these maxima
// bounds the need-th best key from below (every maximum is a key of its own); the keys >= tau
// are ranked exactly.  Too many of them, or larger buffers, take a most-significant-digit
// radix select (8-bit digits, stopping as soon as a whole bucket is needed).
// ------------------------------------------------------------------------------------
template <int NT, bool SCORES>
__global__ __launch_bounds__(NT) void select_topk_kernel(const void* __restrict__ src_all, int n_scores,
                                                         int* __restrict__ ccnt, long long cap, int k,
                                                         float* out_scores, long long* out_ids, int* overflow,
                                                         const int* gate, int threshold_only) {
  constexpr int kCand = 1024;  // candidates the threshold path ranks directly
  constexpr int kRegKeys = SCORES ? 1 : 4096 / NT;
  constexpr int GS = NT / 256;        // threads per group
  constexpr int GB = 256 / GS;        // group maxima each thread of a group counts over
  constexpr int GST = GB + 2;         // block stride: the GS blocks start in different banks
  static_assert(NT == 256 || NT == 1024, "workgroup size");
  __shared__ u64 cand[kCand];
  __shared__ __attribute__((aligned(16))) u64 gmax[GS * GST];
  __shared__ u64 s_tau;
  __shared__ int s_nc;
  __shared__ unsigned int hist[256];
  __shared__ int wtot[NT / 64];
  __shared__ u64 sel[kMaxK];
  __shared__ u64 s_prefix, s_mask;
  __shared__ int s_need, s_done, s_ns;
  if (gate != nullptr && *gate == 0) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int q = blockIdx.x;
  const int cnt = SCORES ? n_scores : ccnt[q];
  if (!SCORES && t == 0 && cnt > cap && overflow != nullptr) atomicAdd(overflow, 1);
  const int n = (int)min((long long)cnt, cap);  // SCORES: cap is the row stride, n_scores <= 32 NT
  auto key_at = [&](int i) -> u64 {
    if constexpr (SCORES) {
      const float v = static_cast<const float*>(src_all)[(long long)q * cap + i];
      return v == v ? composite(v, (uint32_t)i) : 0ull;
    } else {
      return static_cast<const u64*>(src_all)[(long long)q * cap + i];
    }
  };
  if (t == 0) {
    s_prefix = 0ull;
    s_mask = 0ull;
    s_need = min(k, n);
    s_done = s_need == 0;
    s_ns = 0;
    s_tau = 0ull;
    s_nc = 0;
  }
  __syncthreads();
  if (t == 0 && !(threshold_only && !SCORES) && ccnt != nullptr) ccnt[q] = 0;  // every thread has read it: the next pass starts from zero
  const int need = min(k, n);
  // A level with fewer than k keys so far (the rows behind the last threshold may be in later levels): that
  // threshold stays.
  if (!SCORES && threshold_only && need < k) return;  // workgroup-uniform
  const bool in_reg = !SCORES && n <= kRegKeys * NT;  // workgroup-uniform
  // Register keys: thread t holds keys ib + NT u, where ib puts the first 256 keys in 256
  // different groups, so at least min(n, 256) >= need groups are nonempty.  Of scores only the maximum
  // of each 16-byte word is kept (word ib + NT u), and a word that holds a hit is read again: the
  // kernel is bound by latency, and short code counts.
  const int ib = t / GS + 256 * (t % GS);
  u64 kv[kRegKeys];
  float wm[8];
  const float nan = __builtin_nanf("");
  auto word = [&](int i) __attribute__((always_inline)) {  // scores 4 i .. 4 i + 3, NaN past the row
    const float4* src = reinterpret_cast<const float4*>(static_cast<const float*>(src_all) + (long long)q * cap);
    float4 x = 4 * i < n ? src[i] : make_float4(nan, nan, nan, nan);
    if (4 * i + 4 > n) {
      x.y = 4 * i + 1 < n ? x.y : nan;
      x.z = 4 * i + 2 < n ? x.z : nan;
      x.w = 4 * i + 3 < n ? x.w : nan;
    }
    return x;
  };
  if constexpr (SCORES) {
    float4 x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = word(ib + u * NT);
#pragma unroll
    for (int u = 0; u < 8; ++u) wm[u] = fmaxf(fmaxf(x[u].x, x[u].y), fmaxf(x[u].z, x[u].w));
  } else if (in_reg) {
#pragma unroll
    for (int u = 0; u < kRegKeys; ++u) kv[u] = ib + u * NT < n ? key_at(ib + u * NT) : 0ull;
  }
  // keys of this thread beyond the registers, eight loads in flight per step
  auto scan_global = [&](auto&& f) __attribute__((always_inline)) {
    for (int i0 = t; i0 < n; i0 += 8 * NT) {
      u64 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = i0 + u * NT < n ? key_at(i0 + u * NT) : 0ull;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i0 + u * NT < n) f(v[u]);
    }
  };
  if (need > 0) {
    // tau (as a key; 0: every key): the need-th largest of the 256 groups' maxima
    u64 tau = 0ull;
    float ftau = kNegInf;
    const int grp = t / GS, sub = t % GS;
    if constexpr (SCORES) {
      float m = kNegInf;
#pragma unroll
      for (int u = 0; u < 8; ++u) m = fmaxf(m, wm[u]);
      if constexpr (GS == 4) {
        m = fmaxf(m, __int_as_float(dpp<0xB1>(__float_as_int(m))));
        m = fmaxf(m, __int_as_float(dpp<0x4E>(__float_as_int(m))));
      }
      // blocks of the maxima, four floats of padding apart, so that the threads of a group read
      // from different banks
      float* fm = reinterpret_cast<float*>(gmax);
      if (t == 0) s_tau = ~0ull;
      if (sub == 0) fm[(grp / GB) * (GB + 4) + grp % GB] = m;
      __syncthreads();
      int gt = 0;
      const float4* blk = reinterpret_cast<const float4*>(fm + sub * (GB + 4));
#pragma unroll 4
      for (int u = 0; u < GB / 4; ++u) {
        const float4 x = blk[u];
        gt += (x.x > m ? 1 : 0) + (x.y > m ? 1 : 0) + (x.z > m ? 1 : 0) + (x.w > m ? 1 : 0);
      }
      if constexpr (GS == 4) {
        gt += dpp<0xB1>(gt);
        gt += dpp<0x4E>(gt);
      }
      // the need-th largest maximum is the least with fewer than need above it
      if (sub == 0 && gt < need) atomicMin(&s_tau, (u64)score_key(m));
      __syncthreads();
      ftau = key_score((uint32_t)s_tau);
    } else {
      u64 m = 0ull;
      if (in_reg) {
#pragma unroll
        for (int u = 0; u < kRegKeys; ++u) m = umax64(m, kv[u]);
      } else {
        scan_global([&](u64 x) { m = umax64(m, x); });
      }
#pragma unroll
      for (int o = 1; o < GS; o <<= 1) m = umax64(m, shfl_xor64(m, o));
      if (sub == 0) gmax[(grp / GB) * GST + grp % GB] = m;
      __syncthreads();
      // each of the group's threads counts the larger maxima in its share of the list
      int gt = 0;
      const u64* blk = gmax + sub * GST;
#pragma unroll 16
      for (int u = 0; u < GB; ++u) gt += blk[u] > m ? 1 : 0;
#pragma unroll
      for (int o = 1; o < GS; o <<= 1) gt += __shfl_xor(gt, o);
      // nonzero maxima are unique, and at least need groups hold keys
      if (sub == 0 && m != 0ull && gt == need - 1) s_tau = m;
      __syncthreads();
      tau = s_tau;
    }
    if (threshold_only) {
      // An earlier level only hands its k-th score on as the next threshold, and tau is a
      // valid one: at least k keys reach it.
      const float f = SCORES ? ftau : (tau != 0ull ? comp_score(tau) : kNegInf);
      if (t == 0) out_scores[(long long)q * k + (k - 1)] = need == k ? f : kNegInf;
      return;
    }
    // the keys >= tau, in any order (they are ranked exactly): most waves skip most of their keys
    auto take = [&](u64 x) __attribute__((always_inline)) {
      if (x >= tau && x != 0ull) {
        const int pos = atomicAdd(&s_nc, 1);
        if (pos < kCand) cand[pos] = x;
      }
    };
    if constexpr (SCORES) {
      unsigned hm = 0u;
#pragma unroll
      for (int u = 0; u < 8; ++u) hm |= (wm[u] >= ftau ? 1u : 0u) << u;
      for (; hm != 0u; hm &= hm - 1u) {
        const int i = ib + NT * __builtin_ctz(hm);
        const float4 x = word(i);
        const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v[e] >= ftau) {
            const int pos = atomicAdd(&s_nc, 1);
            if (pos < kCand) cand[pos] = composite(v[e], (uint32_t)(4 * i + e));
          }
      }
    } else if (in_reg) {
#pragma unroll
      for (int u = 0; u < kRegKeys; ++u)
        if (__ballot(kv[u] >= tau) != 0ull && ib + u * NT < n) take(kv[u]);
    } else {
      scan_global(take);
    }
    __syncthreads();
    const int nc = s_nc;
    if (nc <= kCand) {  // workgroup-uniform
      // rank = number of larger keys; L adjacent lanes share a candidate, each comparing
      // every L-th entry
      int lg = 0;
      while (lg < 4 && (nc << (lg + 1)) <= NT) ++lg;
      const int L = 1 << lg, p = t & (L - 1);
      for (int j0 = 0; j0 < nc; j0 += NT >> lg) {
        const int jc = j0 + (t >> lg);
        int r = 0;
        u64 me = 0ull;
        if (jc < nc) {
          me = cand[jc];
          for (int o = p; o < nc; o += 8 * L) {
            u64 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = cand[min(o + u * L, nc - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) r += (o + u * L < nc && v[u] > me) ? 1 : 0;
          }
        }
        for (int s = 1; s < L; s <<= 1) r += __shfl_xor(r, s);
        if (jc < nc && p == 0 && r < need) {
          out_ids[(long long)q * k + r] = (long long)comp_row(me);
          out_scores[(long long)q * k + r] = comp_score(me);
        }
      }
      for (int r2 = min(need, nc) + t; r2 < k; r2 += NT) {
        out_ids[(long long)q * k + r2] = -1ll;
        out_scores[(long long)q * k + r2] = kNegInf;
      }
      return;
    }
  }
  for (int shift = 56; shift >= 0; shift -= 8) {
    if (s_done) break;  // block-uniform
    const u64 prefix = s_prefix, mask = s_mask;
    const int need_d = s_need;
    if (t < 256) hist[t] = 0u;
    __syncthreads();
    auto count = [&](u64 key) __attribute__((always_inline)) {
      if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
    };
    if (in_reg) {
#pragma unroll
      for (int u = 0; u < kRegKeys; ++u)
        if (ib + u * NT < n) count(kv[u]);
    } else {
      scan_global(count);
    }
    __syncthreads();
    // threads 0 .. 255 (waves 0 .. 3): thread t holds digit 255 - t; an inclusive scan over t
    // counts the keys whose digit is >= 255 - t within the prefix bucket
    int hd = 0, x = 0;
    if (t < 256) {
      hd = (int)hist[255 - t];
      x = hd;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
      }
      if (lane == 63) wtot[w] = x;
    }
    __syncthreads();
    if (t < 256) {
      int before = 0;
      for (int i = 0; i < w; ++i) before += wtot[i];
      const int incl = before + x;          // keys with digit >= 255 - t
      const int above = incl - hd;          // keys with digit > 255 - t
      if (above < need_d && incl >= need_d) {  // exactly one thread: the digit of the k-th key
        const int dgt = 255 - t;
        s_prefix = prefix | ((u64)dgt << shift);
        s_mask = mask | (255ull << shift);
        s_need = need_d - above;
        s_done = (hd == need_d - above) ? 1 : 0;  // the whole bucket is needed: stop here
      }
    }
    __syncthreads();
  }
  const u64 prefix = s_prefix, mask = s_mask;
  auto gather = [&](u64 key) __attribute__((always_inline)) {
    if ((key & mask) >= prefix) {
      const int slot = atomicAdd(&s_ns, 1);
      if (slot < kMaxK) sel[slot] = key;
    }
  };
  if (in_reg) {
#pragma unroll
    for (int u = 0; u < kRegKeys; ++u)
      if (ib + u * NT < n) gather(kv[u]);
  } else {
    scan_global(gather);
  }
  __syncthreads();
  const int ns = min(s_ns, k);  // == min(k, n)
  if (t < ns) {
    const u64 key = sel[t];
    int rank = 0;
    for (int j = 0; j < ns; ++j) rank += sel[j] > key ? 1 : 0;
    out_ids[(long long)q * k + rank] = (long long)comp_row(key);
    out_scores[(long long)q * k + rank] = comp_score(key);
  }
  for (int r = ns + t; r < k; r += NT) {
    out_ids[(long long)q * k + r] = -1ll;
    out_scores[(long long)q * k + r] = kNegInf;
  }
}

// Weighted fusion (Section 4.4): per query, the dense and lexical scores of every chunk,
// min-max normalised over all chunks (a constant row normalises to 0), weighted and summed in
// fp64 and rounded to fp32.  Lexical scores past n_lex chunks are 0.  One workgroup of 1,024
// threads per query; eight chunks per thread and step, their loads issued before use.
//   pass 1: the minima and maxima of both rows, from the dumps' per-chunk / per-range
//           partials (and 0 for the lexical row when chunks past n_lex exist);
//   pass 2: every chunk's fused composite; tau = the need-th largest of the maxima of the 128
//           eight-thread groups (need = min(k, n) <= 128) bounds the need-th best composite
//           from below;
//   pass 3: the same composites again, and those >= tau go to cbuf[q] (in any order) with
//           their count in ccnt[q], for the exact selection.
// Pass 2 keeps the score keys of the first kFuseLds chunks in LDS for pass 3 and the rest are
// computed again; every operation is rounded explicitly, so both ways give the same composites.
constexpr int kFuseThreads = 1024, kFuseGroups = kFuseThreads / 8, kFuseLds = 32768;
static_assert(kFuseLds % (8 * kFuseThreads) == 0, "whole steps come from LDS");
static_assert(kMaxK <= kFuseGroups, "tau needs k group maxima");
__device__ __forceinline__ u64 fused_composite(double sd, double sl, double mnd, double mnl, float x, float y,
                                               long long i) {
  return composite(fused_value(sd, sl, mnd, mnl, x, y), (uint32_t)i);
}
__global__ __launch_bounds__(kFuseThreads) void weighted_fuse_kernel(const float* __restrict__ D,
                                                                 const float* __restrict__ B, long long ld,
                                                                 long long n, long long n_lex,
                                                                 const float* __restrict__ mm_d, int pd,
                                                                 const float* __restrict__ mm_l, int pl, double wd,
                                                                 double wl, int k, unsigned long long* cbuf, int* ccnt) {
  __shared__ float red[4][kFuseThreads / 64];
  __shared__ uint32_t skey[kFuseLds];
  __shared__ u64 gmax[kFuseGroups];
  __shared__ u64 s_tau;
  __shared__ int s_cnt;
  const long long q = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const float* d = D + q * ld;
  const float* b = B + q * ld;
  float mnd = __builtin_inff(), mxd = -__builtin_inff(), mnl = __builtin_inff(), mxl = -__builtin_inff();
  for (int i = t; i < pd; i += kFuseThreads) {
    mnd = fminf(mnd, mm_d[(q * pd + i) * 2]);
    mxd = fmaxf(mxd, mm_d[(q * pd + i) * 2 + 1]);
  }
  for (int i = t; i < pl; i += kFuseThreads) {
    mnl = fminf(mnl, mm_l[(q * pl + i) * 2]);
    mxl = fmaxf(mxl, mm_l[(q * pl + i) * 2 + 1]);
  }
  if (n_lex < n) {  // chunks past the sparse corpus score 0 lexically
    mnl = fminf(mnl, 0.f);
    mxl = fmaxf(mxl, 0.f);
  }
  for (int o = 32; o > 0; o >>= 1) {
    mnd = fminf(mnd, __shfl_xor(mnd, o));
    mxd = fmaxf(mxd, __shfl_xor(mxd, o));
    mnl = fminf(mnl, __shfl_xor(mnl, o));
    mxl = fmaxf(mxl, __shfl_xor(mxl, o));
  }
  if (lane == 0) {
    red[0][w] = mnd;
    red[1][w] = mxd;
    red[2][w] = mnl;
    red[3][w] = mxl;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kFuseThreads / 64; ++u) {
    mnd = fminf(mnd, red[0][u]);
    mxd = fmaxf(mxd, red[1][u]);
    mnl = fminf(mnl, red[2][u]);
    mxl = fmaxf(mxl, red[3][u]);
  }
  const double sd = mxd > mnd ? wd / ((double)mxd - (double)mnd) : 0.0;
  const double sl = mxl > mnl ? wl / ((double)mxl - (double)mnl) : 0.0;
  const double mnd64 = mnd, mnl64 = mnl;
  // pass 2: this thread's largest composite, then its group's
  u64 m = 0ull;
  for (long long i0 = t; i0 < n; i0 += 8 * kFuseThreads) {
    float x[8], y[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const long long i = i0 + (long long)u * kFuseThreads;
      x[u] = i < n ? d[i] : 0.f;
      y[u] = i < n_lex ? b[i] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const long long i = i0 + (long long)u * kFuseThreads;
      if (i < n) {
        const u64 c = fused_composite(sd, sl, mnd64, mnl64, x[u], y[u], i);
        m = umax64(m, c);
        if (i < kFuseLds) skey[i] = comp_key(c);
      }
    }
  }
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) m = umax64(m, __shfl_xor(m, o));
  if ((t & 7) == 0) gmax[t >> 3] = m;
  if (t == 0) {
    s_tau = 0ull;
    s_cnt = 0;
  }
  __syncthreads();
  // Nonzero group maxima are distinct composites; when fewer than need of them exist, tau
  // stays 0 and every chunk is a candidate.
  const int need = (int)min((long long)k, n);
  if (t < kFuseGroups && need > 0) {
    const u64 g = gmax[t];
    int gt = 0;
#pragma unroll 8
    for (int u = 0; u < kFuseGroups; ++u) gt += gmax[u] > g ? 1 : 0;
    if (g != 0ull && gt == need - 1) s_tau = g;
  }
  __syncthreads();
  const u64 tau = s_tau;
  // pass 3: compact the composites >= tau, one LDS reservation per wave and step
  unsigned long long* dst = cbuf + q * n;
  for (long long i0 = t; i0 < n; i0 += 8 * kFuseThreads) {
    float x[8], y[8];
    const bool from_lds = i0 + 7ll * kFuseThreads < kFuseLds;  // uniform: whole steps
    if (!from_lds) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const long long i = i0 + (long long)u * kFuseThreads;
        x[u] = i < n ? d[i] : 0.f;
        y[u] = i < n_lex ? b[i] : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const long long i = i0 + (long long)u * kFuseThreads;
      u64 c = 0ull;
      if (i < n)
        c = from_lds ? ((u64)skey[i] << 32) | (u64)(uint32_t)(~(uint32_t)i)
                     : fused_composite(sd, sl, mnd64, mnl64, x[u], y[u], i);
      const bool take = i < n && c >= tau;
      const u64 bal = __ballot(take);
      if (bal != 0ull) {
        int base = 0;
        if (lane == __ffsll((long long)bal) - 1) base = atomicAdd(&s_cnt, __popcll(bal));
        base = __shfl(base, __ffsll((long long)bal) - 1);
        if (take) dst[base + __popcll(bal & ((1ull << lane) - 1ull))] = c;
      }
    }
  }
  __syncthreads();
  if (t == 0) ccnt[q] = s_cnt;
}

// Clears the filtered-mode counters (a kernel, not a memset: safe inside captured graphs).
__global__ void clear_ints_kernel(int* p, long long n, const int* gate) {
  if (gate != nullptr && *gate == 0) return;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    p[i] = 0;
}

// ------------------------------------------------------------------------------------
// Planning.
// ------------------------------------------------------------------------------------
// k <= 16: up to this many queries group maxima at any length.  Their memory fits the search without a workspace
// then, and no data makes them slow; rows in random order would be filtered as fast: bf16, 64 queries, group
// maxima against levels 179 / 186 us over 393,216 x 1,024, 263 / 252 over 600,000, 408 / 388 over 1 M.
constexpr int kMaximaQueries = 64;
// Most bytes of a launch's group maxima: of up to 64 queries (so that any index length fits the fixed
// array of the search without a workspace), and of larger batches.
constexpr size_t kMaximaBytes = 24ull << 20, kBatchMaximaBytes = 256ull << 20;

// Tile shapes of dense_tile.h.  eff: the rate of the shape's MFMAs at 1,024 queries over 32,768 x
// 1,024 bf16 rows, relative to the largest (1,285 TFLOP/s; 1,088, 1,079, 920 and 671 for the
// smaller ones): fewer MFMAs per byte read from LDS and per barrier.  The 16-query shape serves
// batches of up to 16, where the rows' bytes bound every shape and the smallest epilogue is best.
// fp32: the MFMAs themselves bound every shape, so padded work decides.
// Of each shape forced in turn, 80 to 3,000 queries, the choice is within 3 % of the fastest at 384 to 4,096
// dimensions (32,768 x 1,024, 99,991 x 768, 150,000 x 384, 20,000 x 4,096); at 128, where the epilogue counts
// as much as the two stages, 256 x 256 tiles are up to 25 % slower than 128 x 256 ones (393,000 rows, 256 queries 89 /
// 66 us).
struct ShapeInfo {
  int bm, bn, wm, mt;  // tile rows and queries, waves along the rows, subtiles per wave
  double eff, eff32;
};
constexpr ShapeInfo kShapes[] = {{128, 16, 8, 1, 0.25, 0.9}, {128, 64, 4, 2, 0.52, 1.0},  {128, 128, 2, 4, 0.72, 1.0},
                                 {256, 128, 4, 4, 0.84, 0.}, {128, 256, 2, 4, 0.85, 0.}, {256, 256, 2, 8, 1.0, 0.}};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]), kNumShapes32 = 3;

constexpr long long kDumpRows = 32768;        // up to this many rows every score may be kept (the selection's most)
// k <= 16: up to this many scores of a launch (times the row bytes over kDumpRow, where these are
// more) are kept, 24 MiB at most.  Few scores are read back and selected from sooner than rows are scored
// again, the more so the longer the rows: bf16, k = 10, group maxima against all scores in us:
//   d 128:  64 queries x 10,000 rows 13.3 / 12.3, x 20,000 13.6 / 14.3; 1,024 x 1,000 17.8 / 16.6, x 4,000 18.5 / 23.0
//   d 1024: 16 x 1,000 18.6 / 13.5, 64 x 32,768 22.7 / 22.2, 256 x 10,000 21.7 / 21.4, x 32,768 31.1 / 33.9
//   d 4096: 256 x 20,000 69.3 / 60.3; fp32 d 1024: 16 x 1,000 33.4 / 23.4
constexpr long long kDumpScores = 1ll << 20, kDumpMost = 6ll << 20, kDumpRow = 768;
// Batches of up to 16 over longer indexes keep every score while a chunk's fit in LDS and they add a 16th
// to the index's bytes at most: reading scores back takes 4 us less than scoring rows again, and chunks
// need not end with a tile.  bf16, k = 5, group maxima against all scores in us: 1 query over 65,536 x 1,024
// 30.5 / 26.4, 150,000 57.0 / 53.0, 300,000 121.5 / 116.3, 1 M 353 / 347 (k = 10); 16 queries 30.7 / 27.3 and
// 58.7 / 58.5; f16 168,344 x 512, 4 queries 37.2 / 33.9; 8 queries over 100,000 x 256 20.6 / 18.0.  More tiles than
// LDS holds, stored in two parts: 16 queries over 300,000 x 1,024 123 / 128, 4 over 1 M 354 / 356.
constexpr long long kScoresShare = 4 * 16;
// k <= 16, more than 64 queries: longer indexes filter.  The line is where 512 queries gain from neither;
// fewer queries would cross at some 800,000 rows, more at 300,000.  bf16 x 1,024, group maxima against
// levels in us: 65 queries over 393,216 rows 167 / 195, 600,000 256 / 276, 1 M 410 / 397; 512 queries 377 / 407,
// 565 / 585, 933 / 890; 2,048 queries over 200,000 rows 735 / 811, 393,216 1,462 / 1,345, 600,000 2,218 / 2,001.
constexpr long long kMaximaRows = 393216;
// Up to this many groups (one pass of the rescoring workgroup) are searched directly, which saves a
// dependent read (1.5 us of a call; batch 1 over 32,768 rows, by group maxima, 21.3 -> 20.0 us), unless the batch is so
// large that the maxima's bytes count (batch 1,024: 15.6 us, 14.5 through the coarse ones).
constexpr int kOneLevel = 8192;
constexpr long long kFilterMin = 4096;        // fewest rows of the first level
constexpr long long kFilterFirst = 32000;     // most rows of the first level
// Row growth between levels.  A level's hits cost its tiles time in proportion (at 16-fold growth and k
// = 100, a hit in 5,000 scores, a fifth of it), a level itself two launches.
constexpr long long filter_grow(int k) { return k <= 16 ? 8 : 4; }
// Filter, k <= 16: candidate slots per query.  A query whose best rows only the first and the last level have
// (a topic that lies between two tiles of the others) collects about 64 k, 1,024 at k = 16, but the sample of
// k rows varies: of 300 such queries 2 overflowed 2,048 slots.
constexpr long long kSmallCap = 3072;

size_t align_up256(size_t x) { return (x + 255) & ~(size_t)255; }
int elem_bytes(int dtype) { return dtype == kDtypeF32 ? 4 : 2; }
int log2i(long long x) {
  int l = 0;
  while ((1ll << (l + 1)) <= x) ++l;
  return l;
}

// The row tiles of a launch (DenseArgs): all of the index, or some of them.
struct TileSet {
  long long tiles, tile_pitch;
  int row_pitch = 1, skip = 0;
};
TileSet all_tiles(const ShapeInfo& sh, long long rows) { return {std::max(1ll, (rows + sh.bm - 1) / sh.bm), sh.bm}; }

constexpr long long kChunkBytes = 1ll << 30;

// Most row tiles of a chunk: 32-bit byte offsets reach past it, and its row offsets fit the
// kChunkRowBits bits that a queued hit has for them (fp32 rows of up to 12 dimensions are the ones
// short enough for that to count).
long long max_tiles(const ShapeInfo& sh, int dtype, int d, const TileSet& set) {
  long long by_offset = kChunkBytes / (set.tile_pitch * d * elem_bytes(dtype));
  if (set.skip > 0) by_offset = by_offset * set.skip / (set.skip + 1);
  return std::max(1ll, std::min(by_offset, (1ll << kChunkRowBits) / sh.bm));
}

// Chunks of one launch: row tiles divided as evenly as they go over at most one workgroup per CU
// (rounded down, so that the grid is one round), and no more tiles per chunk than max_tiles.
struct TileGrid {
  int n_qblocks = 1, n_chunks = 1;
  long long tiles = 0, most = 0, grid = 0;  // row tiles, the most of a chunk, workgroups
};

TileGrid tile_grid(int shape, int dtype, int d, const TileSet& set, int nq, int n_cus) {
  const ShapeInfo& sh = kShapes[shape];
  TileGrid g;
  g.n_qblocks = (nq + sh.bn - 1) / sh.bn;
  g.tiles = set.tiles;
  const long long chunks = std::max(1ll, (long long)n_cus / g.n_qblocks), mt = max_tiles(sh, dtype, d, set);
  g.n_chunks = (int)std::min(g.tiles, std::max(chunks, (g.tiles + mt - 1) / mt));
  g.most = (g.tiles + g.n_chunks - 1) / g.n_chunks;
  g.grid = (long long)g.n_chunks * g.n_qblocks;
  return g;
}
TileGrid tile_grid(int shape, int dtype, int d, long long rows, int nq, int n_cus) {
  return tile_grid(shape, dtype, d, all_tiles(kShapes[shape], rows), nq, n_cus);
}

// The shape whose slowest CU finishes its MFMAs first.  (A short index or a small batch wants small
// tiles, so that every CU has one; the padding of the last query block counts too.)  bm: only among the
// shapes with so many rows a tile.
int pick_shape(int dtype, int d, long long rows, int nq, int n_cus, int bm = 0) {
  int best = -1;
  double cost = 0.0;
  for (int i = 0; i < (dtype == kDtypeF32 ? kNumShapes32 : kNumShapes); ++i) {
    // (the bounds of the groups' memory rely on it; for up to 64 queries the larger tiles never cost less)
    if ((nq > kMaximaQueries) != (kShapes[i].mt >= 4) || (bm != 0 && bm != kShapes[i].bm)) continue;
    const TileGrid g = tile_grid(i, dtype, d, rows, nq, n_cus);
    const double rounds = (double)((g.grid + n_cus - 1) / n_cus);
    const double c = rounds * (double)g.most * kShapes[i].bm * kShapes[i].bn /
                     (dtype == kDtypeF32 ? kShapes[i].eff32 : kShapes[i].eff);
    if (best < 0 || c < cost) {
      best = i;
      cost = c;
    }
  }
  return best;
}

// Rows per group, k <= 16.  A query's maxima are written once (4 N / G bytes) and its k best
// groups' rows read again (k G rows): the power of two nearest to the least sum, 4 at least.
long long maxima_group(int dtype, int d, long long rows, int k) {
  const long long row_bytes = (long long)d * elem_bytes(dtype);
  long long g = 4;
  while (g < 32 && g * g * k * row_bytes < 2 * rows) g *= 2;
  return g;
}

// The maxima of a launch with groups of G rows (or as many as a lane has of a tile); unit_sh > 0: of
// all that a lane has of 1 << unit_sh tiles.
MaxGroups max_groups(int shape, int dtype, int d, long long rows, int nq, int n_cus, long long G, int unit_sh = 0) {
  const ShapeInfo& sh = kShapes[shape];
  const TileGrid g = tile_grid(shape, dtype, d, rows, nq, n_cus);
  MaxGroups m;
  m.gs = unit_sh > 0 ? sh.mt : (int)std::min<long long>(G / 4, sh.mt);
  m.per_tile = sh.wm * 4 * (sh.mt / m.gs);
  m.unit_sh = unit_sh;
  m.upc = unit_sh > 0 ? (int)((g.most + (1ll << unit_sh) - 1) >> unit_sh) : 0;
  m.count = rows > 0 ? (int)((unit_sh > 0 ? (long long)g.n_chunks * m.upc : g.tiles) * m.per_tile) : 0;
  m.ld = (m.count + 3) & ~3ll;
  m.coarse = rows > 0 ? g.n_chunks * sh.wm * 4 : 0;
  m.cld = (m.coarse + 3) & ~3ll;
  return m;
}

// The maxima of a k <= 16 search: groups of maxima_group rows, and larger ones while they take more
// memory than they may.  Writing fewer of them is faster as well: 8.45 M rows of 384 fp16, 64 queries, 2.00 ms
// with 8 rows a group (271 MB), 1.37 with 128 (17 MB); 16 queries, 1.52 ms with 4 rows (135 MB), 1.11 with 32.
MaxGroups search_groups(int shape, int dtype, int d, long long rows, int nq, int k, int n_cus) {
  const bool small = nq <= kMaximaQueries;
  long long G = maxima_group(dtype, d, rows, k);
  int unit_sh = 0;
  for (;;) {
    MaxGroups m = max_groups(shape, dtype, d, rows, nq, n_cus, G, unit_sh);
    const bool fits = (size_t)nq * (size_t)m.ld * 4 <= (small ? kMaximaBytes : kBatchMaximaBytes);
    if (fits || (m.gs == kShapes[shape].mt && (!small || m.upc == 1))) return m;
    if (m.gs < kShapes[shape].mt)
      G = 8 * m.gs;
    else
      ++unit_sh;
  }
}

long long dump_scores(int dtype, int d) {  // k <= 16
  const long long row_bytes = (long long)d * elem_bytes(dtype);
  return std::min(kDumpMost, kDumpScores * std::max(kDumpRow, row_bytes) / kDumpRow);
}
bool use_dump(int dtype, int d, long long rows, int nq, int k) {
  return rows <= kDumpRows && (k > 16 || nq * rows <= dump_scores(dtype, d));
}
bool use_scores(int dtype, int d, long long rows, int nq, int k, int n_cus) {
  return k <= 16 && rows > kDumpRows && nq <= 16 && kScoresShare * nq <= (long long)d * elem_bytes(dtype) &&
         nq * tile_grid(0, dtype, d, rows, nq, n_cus).most <= kHeldTiles;
}
bool use_maxima(long long rows, int nq, int k) { return k <= 16 && (nq <= kMaximaQueries || rows <= kMaximaRows); }

// Candidate slots per query of the filter levels.  A level adds about (growth - 1) k of them (the first
// one growth k).
long long filter_cap(int k) { return k <= 16 ? kSmallCap : std::max(4096ll, 64ll * k); }

// Workspace.  Maxima: groups [nq][ld] | coarse [nq][cld].  Filter: candidate buffers [nq][cap] (in the
// same memory, before them the first level's groups and after them the fallback's coarse maxima) |
// counts [nq] | overflow flags.
size_t maxima_bytes(int nq, long long ld, long long cld) {
  return align_up256((size_t)nq * (size_t)ld * 4) + align_up256((size_t)nq * (size_t)cld * 4);
}
size_t filter_body(int nq, int k) {
  return align_up256((size_t)nq * (size_t)filter_cap(k) * 8) + align_up256((size_t)nq * 4);
}
// Short index: the scores; k > 16: room for a 64-bit key per row and query, more than they take.
size_t dump_bytes(int nq, long long rows, int k) {
  if (k <= 16) return align_up256((size_t)nq * (size_t)((rows + 3) & ~3ll) * 4);
  return align_up256((size_t)nq * (size_t)std::max(1ll, rows) * 8) + align_up256((size_t)nq * 4) + 256;
}

}  // namespace

DensePlan plan_dense(int dtype, int d, long long n_rows, int nq, int k, int n_cus) {
  DensePlan p;
  p.n_cus = n_cus;
  p.shape = pick_shape(dtype, d, n_rows, nq, n_cus);
  p.kind = use_dump(dtype, d, n_rows, nq, k) ? DensePlan::kDump
           : use_maxima(n_rows, nq, k)       ? DensePlan::kMaxima
                                             : DensePlan::kFilter;
  if (use_scores(dtype, d, n_rows, nq, k, n_cus)) {
    p.kind = DensePlan::kScores;
    p.shape = 0;
    p.ld = (n_rows + 3) & ~3ll;
    p.groups = max_groups(p.shape, dtype, d, n_rows, nq, n_cus, 4);
  } else if (p.kind == DensePlan::kMaxima) {
    p.groups = search_groups(p.shape, dtype, d, n_rows, nq, k, n_cus);
    if (p.groups.count <= kOneLevel && nq <= 2 * n_cus) p.groups.coarse = p.groups.cld = 0;
  } else if (p.kind == DensePlan::kDump) {
    p.ld = (n_rows + 3) & ~3ll;
  } else {
    // Levels from the end: each holds a fixed share of the next one's tiles, every 4th or 8th of them,
    // down to a first level of at most kFilterFirst rows.
    const int bm = kShapes[p.shape].bm;
    const long long tiles = (n_rows + bm - 1) / bm;
    long long back[16], rows = n_rows;
    int nb = 0;
    for (long long stride = 1; nb < 15; stride *= filter_grow(k)) {
      back[nb++] = stride;
      rows = std::max(kFilterMin, (rows + filter_grow(k) - 1) / filter_grow(k));
      if (rows <= kFilterFirst) break;
    }
    p.n_levels = nb + 1;
    for (int l = 1; l <= nb; ++l) {
      p.level_pitch[l] = back[nb - l] * bm;
      p.level_rows[l] = std::min(n_rows, (tiles + back[nb - l] - 1) / back[nb - l] * bm);
    }
    // The first level only hands thresholds on, so its rows need not be among the second one's: single rows
    // spread over the index (an odd number apart: of documents of 2^n rows not always the same one), in
    // tiles as long as 32-bit offsets allow.
    p.shape0 = pick_shape(dtype, d, std::min(rows, n_rows), nq, n_cus);
    const int bm0 = kShapes[p.shape0].bm;
    const long long tiles0 = std::min(rows, n_rows) / bm0;
    p.level_pitch[0] = n_rows / tiles0;
    p.row_pitch0 = (int)std::min(p.level_pitch[0] / bm0, kChunkBytes / ((long long)bm0 * d * elem_bytes(dtype)));
    p.row_pitch0 -= p.row_pitch0 % 2 == 0 ? 1 : 0;
    p.level_rows[0] = tiles0 * bm0;
    // the first level's groups, as many as their memory and one pass of the selection allow: the k best
    // rows then mostly fall in groups of their own, and the k-th maximum is close to the k-th score
    p.cap = filter_cap(k);
    const long long most = std::min(2 * p.cap, 8192ll);
    for (long long G = 4; G <= 32; G *= 2) {
      p.groups = max_groups(p.shape0, dtype, d, p.level_rows[0], nq, n_cus, G);
      if (p.groups.count <= most) break;
    }
    p.groups.coarse = 0;
    p.groups.cld = 0;
    // exact fallback: the coarse maxima of the whole index, in chunks as short as the candidate
    // buffers' memory allows
    const ShapeInfo& sh = kShapes[p.shape];
    p.cus_all = (int)(most / (sh.wm * 4)) * ((nq + sh.bn - 1) / sh.bn);
    p.groups_all = max_groups(p.shape, dtype, d, n_rows, nq, p.cus_all, 4);
    p.groups_all.count = 0;
    p.groups_all.ld = 0;
  }
  return p;
}

size_t dense_workspace_bytes(const DensePlan& p, int dtype, int d, int nq, long long n_rows, int k) {
  if (p.kind == DensePlan::kMaxima) return maxima_bytes(nq, p.groups.ld, p.groups.cld);
  if (p.kind == DensePlan::kScores) return maxima_bytes(nq, p.ld, p.groups.cld);
  if (p.kind == DensePlan::kDump) return dump_bytes(nq, n_rows, k);
  return filter_body(nq, k) + 256;
}

// The caller splits a batch until every part fits this.  A workspace for nq queries and k results
// serves every smaller batch and k.
size_t dense_workspace_bound(int dtype, int d, long long capacity, int nq, int k, int n_cus) {
  const long long row_bytes = (long long)d * elem_bytes(dtype);
  const int k1 = std::min(k, 16);  // of maxima; larger k: of k = 16
  // The most groups any row count up to `rows` is split into: at the last row count of each group
  // size (tiles of more than 64 queries allow groups of 16, smaller ones may have only 4 rows)
  auto maxima = [&](int queries, long long rows) {
    const bool small = queries <= kMaximaQueries;
    long long groups = 0;
    const long long top = small ? 4 : std::min(16ll, maxima_group(dtype, d, rows, k1));
    for (long long g = 4; g <= top; g *= 2)
      groups = std::max(groups, ((g == top ? rows : std::min(rows, g * g * k1 * row_bytes / 2)) + g - 1) / g + 64);
    // coarse: a lane's per chunk and query, 32 lanes in the 16-query tiles and 16 at most in those of
    // 128 and 256 queries, where a CU serves 128 or more queries of a chunk; more chunks than CUs only
    // where 32-bit offsets ask for them
    const long long longest =
        std::max(1ll, std::min((1ll << 30) / (256ll * row_bytes), (1ll << kChunkRowBits) / 256)) * 256;
    const long long by_len = (rows + longest - 1) / longest;
    const size_t coarse = 4 * (small ? (size_t)queries * 32 * (size_t)std::max<long long>(n_cus, by_len)
                                     : (size_t)16 * std::min(queries, 512) * (size_t)n_cus +
                                           (size_t)queries * 16 * (size_t)by_len);
    const size_t most = small ? std::max(kMaximaBytes, coarse) : kBatchMaximaBytes;  // (small: a unit per chunk at least)
    size_t fine = std::min((size_t)queries * (size_t)((groups + 3) & ~3ll) * 4, most);
    // kScores: as many as the CUs hold, in as many chunks
    fine = std::max(fine, (size_t)std::min(std::min(queries, 16) * rows, (long long)kHeldTiles * 128 * n_cus) * 4 + 256);
    return align_up256(fine) + align_up256(coarse + (size_t)queries * 16);
  };
  size_t b = maxima(std::min(nq, kMaximaQueries), capacity);
  if (nq > kMaximaQueries) {
    b = std::max(b, maxima(nq, std::min(capacity, kMaximaRows)));
    if (capacity > kMaximaRows) b = std::max(b, filter_body(nq, k1) + 256);
  }
  // k <= 16, every score: of one row a query at least
  b = std::max(b, align_up256((size_t)std::min(nq * std::min(capacity, kDumpRows), dump_scores(dtype, d)) * 4 + (size_t)nq * 16));
  if (k > 16) {
    b = std::max(b, dump_bytes(nq, std::min(capacity, kDumpRows), k));
    if (capacity > kDumpRows) b = std::max(b, filter_body(nq, k) + 256);
  }
  return b;
}

namespace {

hipError_t launch_tiles(int dtype, int shape, int mode, const DenseArgs& a, const TileSet& set, int n_cus, hipStream_t s,
                        hipEvent_t ev0, hipEvent_t ev1) {
  const TileGrid g = tile_grid(shape, dtype, a.d, set, a.nq, n_cus);
  DenseArgs arg = a;
  arg.tile_pitch = (int)set.tile_pitch;
  arg.row_pitch = set.row_pitch;
  arg.skip = set.skip;
  arg.skip_recip = set.skip > 0 ? (unsigned)(((1ull << 32) + set.skip - 1) / set.skip) : 0u;
  arg.n_qblocks = g.n_qblocks;
  arg.n_chunks = g.n_chunks;
  arg.tiles = g.tiles;
  if (dtype == kDtypeBF16) return tile_launch<kDtypeBF16>(shape, mode, g.grid, arg, s, ev0, ev1);
  if (dtype == kDtypeF16) return tile_launch<kDtypeF16>(shape, mode, g.grid, arg, s, ev0, ev1);
  return tile_launch<kDtypeF32>(shape, mode, g.grid, arg, s, ev0, ev1);
}

hipError_t launch_maxima(int dtype, int shape, int mode, const MaxGroups& m, const DenseArgs& a, const TileSet& set, int n_cus,
                         const int* gate, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  DenseArgs arg = a;
  arg.mx = m.count > 0 ? reinterpret_cast<float*>(a.partial) : nullptr;
  arg.mx_ld = m.ld;
  arg.mx_gs = m.gs;
  arg.unit_sh = m.unit_sh;
  arg.upc = m.upc;
  arg.cmx = m.coarse > 0 ? reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(a.partial) +
                                                    align_up256((size_t)a.nq * (size_t)m.ld * 4))
                         : nullptr;
  arg.cmx_ld = m.cld;
  arg.gate = gate;
  return launch_tiles(dtype, shape, mode, arg, set, n_cus, s, ev0, ev1);
}

// scores_ld > 0: from every score (that far apart) and the coarse maxima.
hipError_t launch_rescore(int dtype, int shape, const MaxGroups& m, const DenseArgs& a, int n_cus, const int* gate,
                          hipStream_t s, long long scores_ld = 0) {
  const ShapeInfo& sh = kShapes[shape];
  const TileGrid g = tile_grid(shape, dtype, a.d, a.n_rows, a.nq, n_cus);
  RescoreArgs r;
  r.X = a.X;
  r.Q = a.Q;
  r.n_rows = a.n_rows;
  r.d = a.d;
  r.k = a.k;
  r.fine = m.count > 0 ? reinterpret_cast<const float*>(a.partial) : nullptr;
  r.fine_ld = m.ld;
  r.n_fine = m.count;
  r.coarse = reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>(a.partial) +
                                            align_up256((size_t)a.nq * (size_t)m.ld * 4));
  r.coarse_ld = m.cld;
  r.n_coarse = m.coarse;
  r.two = m.count > 0 && m.coarse > 0;
  if (scores_ld > 0) {
    r.scores = 1;
    r.fine_ld = scores_ld;
    r.n_fine = (int)a.n_rows;
    r.coarse = reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>(a.partial) +
                                              align_up256((size_t)a.nq * (size_t)scores_ld * 4));
  }
  r.tile_rows = sh.bm;
  r.n_chunks = g.n_chunks;
  r.least = (int)(g.tiles / g.n_chunks);
  r.spare = (int)(g.tiles % g.n_chunks);
  r.most = (int)g.most;
  r.lanes_sh = log2i(sh.wm * 4);
  r.gpt_sh = m.count == 0 ? r.lanes_sh : log2i(m.per_tile);
  r.gl_sh = log2i(sh.mt / m.gs);
  r.gs_sh = log2i(m.gs);
  r.mt_sh = log2i(sh.mt);
  r.unit_sh = m.unit_sh;
  r.upc = m.upc;
  r.out_scores = a.out_scores;
  r.out_ids = a.out_ids;
  r.gate = gate;
  if (dtype == kDtypeBF16) return rescore_launch<kDtypeBF16>(r, a.nq, s);
  if (dtype == kDtypeF16) return rescore_launch<kDtypeF16>(r, a.nq, s);
  return rescore_launch<kDtypeF32>(r, a.nq, s);
}

// Exact top-k of each query's candidate buffer (threshold_only: just a valid k-th score).
hipError_t launch_select(int n_cus, const unsigned long long* cbuf, int* ccnt, long long cap, int nq, int k,
                         float* out_scores, long long* out_ids, int* ovf, const int* gate, bool threshold_only,
                         hipStream_t s) {
  if (nq <= 2 * n_cus)
    hipLaunchKernelGGL((select_topk_kernel<1024, false>), dim3((unsigned)nq), dim3(1024), 0, s, cbuf, 0, ccnt, cap, k,
                       out_scores, out_ids, ovf, gate, threshold_only ? 1 : 0);
  else
    hipLaunchKernelGGL((select_topk_kernel<256, false>), dim3((unsigned)nq), dim3(256), 0, s, cbuf, 0, ccnt, cap, k,
                       out_scores, out_ids, ovf, gate, threshold_only ? 1 : 0);
  return hipGetLastError();
}

// The same from rows of n fp32 scores (n <= 32,768), ccnt (optional) zeroed.
hipError_t launch_select_scores(const float* scores, int n, long long ld, int* ccnt, int nq, int k, float* out_scores,
                                long long* out_ids, bool threshold_only, hipStream_t s) {
  if (n > 8192 || nq <= 512)
    hipLaunchKernelGGL((select_topk_kernel<1024, true>), dim3((unsigned)nq), dim3(1024), 0, s, scores, n, ccnt, ld, k,
                       out_scores, out_ids, nullptr, nullptr, threshold_only ? 1 : 0);
  else
    hipLaunchKernelGGL((select_topk_kernel<256, true>), dim3((unsigned)nq), dim3(256), 0, s, scores, n, ccnt, ld, k,
                       out_scores, out_ids, nullptr, nullptr, threshold_only ? 1 : 0);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_dense(const DensePlan& p, int dtype, const DenseArgs& a, hipStream_t s, hipEvent_t ev0,
                        hipEvent_t ev1) {
  if (p.kind == DensePlan::kMaxima) {
    const hipError_t e = launch_maxima(dtype, p.shape, p.groups.unit_sh > 0 ? kTileUnits : kTileMax, p.groups, a,
                                       all_tiles(kShapes[p.shape], a.n_rows), p.n_cus, nullptr, s, ev0, ev1);
    if (e != hipSuccess) return e;
    return launch_rescore(dtype, p.shape, p.groups, a, p.n_cus, nullptr, s);
  }
  if (p.kind == DensePlan::kScores) {
    DenseArgs arg = a;
    arg.dump = reinterpret_cast<float*>(a.partial);
    arg.dump_ld = p.ld;
    arg.cmx = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(a.partial) +
                                       align_up256((size_t)a.nq * (size_t)p.ld * 4));
    arg.cmx_ld = p.groups.cld;
    const hipError_t e = launch_tiles(dtype, p.shape, kTileScores, arg, all_tiles(kShapes[p.shape], a.n_rows), p.n_cus, s,
                                      ev0, ev1);
    if (e != hipSuccess) return e;
    return launch_rescore(dtype, p.shape, p.groups, a, p.n_cus, nullptr, s, p.ld);
  }
  if (p.kind == DensePlan::kDump) {
    DenseArgs arg = a;
    arg.dump = reinterpret_cast<float*>(a.partial);
    arg.dump_ld = p.ld;
    const hipError_t e = launch_tiles(dtype, p.shape, kTileDump, arg, all_tiles(kShapes[p.shape], a.n_rows), p.n_cus, s,
                                      ev0, ev1);
    if (e != hipSuccess) return e;
    return launch_select_scores(arg.dump, (int)a.n_rows, p.ld, nullptr, a.nq, a.k, a.out_scores, a.out_ids, false, s);
  }
  // (an index so long that 32-bit offsets ask for more chunks than the fallback's memory holds: not
  // within any device's memory)
  if (std::max(p.groups.ld, p.groups_all.cld) > 2 * p.cap) return hipErrorInvalidValue;
  unsigned char* ws = reinterpret_cast<unsigned char*>(a.partial);
  const size_t body = filter_body(a.nq, a.k);
  int* ccnt = reinterpret_cast<int*>(ws + body - align_up256((size_t)a.nq * 4));
  // [0] a query's candidates overflowed, [2] the repair's did.
  int* fl = reinterpret_cast<int*>(ws + body);
  hipLaunchKernelGGL(clear_ints_kernel, dim3(1), dim3(64), 0, s, fl, 4ll, nullptr);
  // The first level's thresholds (its selection also zeroes the counts); out_scores[q k + k - 1]
  // holds a query's threshold between the levels.
  hipError_t e = launch_maxima(dtype, p.shape0, kTileSample, p.groups, a, {p.level_rows[0] / kShapes[p.shape0].bm, p.level_pitch[0],
                                                                p.row_pitch0}, p.n_cus, nullptr, s, nullptr, nullptr);
  if (e == hipSuccess)
    e = launch_select_scores(reinterpret_cast<const float*>(a.partial),
                             p.groups.count, p.groups.ld, ccnt, a.nq, a.k, a.out_scores,
                             a.out_ids, true, s);
  DenseArgs arg = a;
  arg.th = a.out_scores + (a.k - 1);
  arg.th_stride = a.k;
  arg.cbuf = a.partial;
  arg.ccnt = ccnt;
  arg.cap = p.cap;
  const int bm = kShapes[p.shape].bm;
  const TileSet all = all_tiles(kShapes[p.shape], a.n_rows);
  for (int l = 1; l < p.n_levels && e == hipSuccess; ++l) {
    const bool last = l == p.n_levels - 1;
    // Level 1 has every tile of its pitch; later levels take those that the ones before left out and add to
    // their candidates.
    auto of_pitch = [&](long long pitch) { return (all.tiles + pitch / bm - 1) / (pitch / bm); };
    TileSet set{of_pitch(p.level_pitch[l]), p.level_pitch[l]};
    if (l > 1) {
      set.skip = (int)(p.level_pitch[l - 1] / p.level_pitch[l]) - 1;
      set.tiles -= of_pitch(p.level_pitch[l - 1]);
    }
    const int shape = last ? p.shape : pick_shape(dtype, a.d, set.tiles * bm, a.nq, p.n_cus, bm);
    // A tile expects its scores times k / (the previous level's rows) hits: the queue is looked at
    // before they can fill half of it, every 16 tiles at most.
    const double hits = (double)kShapes[shape].bm * kShapes[shape].bn * a.k / (double)p.level_rows[l - 1];
    arg.check_mask = 15;
    while (arg.check_mask > 0 && (arg.check_mask + 1) * hits > 512.0) arg.check_mask >>= 1;
    e = launch_tiles(dtype, shape, kTileFilt, arg, set, p.n_cus, s, last ? ev0 : nullptr, last ? ev1 : nullptr);
    if (e == hipSuccess)
      e = launch_select(p.n_cus, arg.cbuf, ccnt, p.cap, a.nq, a.k, a.out_scores, a.out_ids, last ? fl : nullptr, nullptr,
                        !last, s);
  }
  if (e != hipSuccess) return e;
  // Exactness repair, decided on the device: only a buffer overflow can lose a row.  Then the
  // whole index is filtered again with the current k-th scores as thresholds
  // (the lists are the top-k of a subset of the rows at or above the old thresholds, so
  // their k-th scores are valid thresholds and no lower), and if that overflows too, group
  // maxima over the whole index answer.  Each repair launch returns at once when its flag is
  // clear.
  arg.check_mask = 0;
  arg.gate = fl;
  e = launch_tiles(dtype, p.shape, kTileFilt, arg, all, p.n_cus, s, nullptr, nullptr);
  if (e == hipSuccess)
    e = launch_select(p.n_cus, arg.cbuf, ccnt, p.cap, a.nq, a.k, a.out_scores, a.out_ids, fl + 2, fl, false, s);
  if (e == hipSuccess)
    e = launch_maxima(dtype, p.shape, kTileMax, p.groups_all, a, all, p.cus_all, fl + 2, s, nullptr, nullptr);
  if (e == hipSuccess) e = launch_rescore(dtype, p.shape, p.groups_all, a, p.cus_all, fl + 2, s);
  return e;
}

DensePlan plan_dense_dump(int dtype, int d, long long n_rows, int nq, int n_cus) {
  DensePlan p;
  p.n_cus = n_cus;
  p.kind = DensePlan::kDump;
  p.shape = pick_shape(dtype, d, n_rows, nq, n_cus);
  p.n_chunks = tile_grid(p.shape, dtype, d, n_rows, nq, n_cus).n_chunks;
  return p;
}

int dense_dump_chunks(int dtype, int d, long long capacity, int nq, int n_cus) {
  long long most = 1;
  for (int i = 0; i < kNumShapes; ++i) {
    const ShapeInfo& sh = kShapes[i];
    const long long tiles = (capacity + sh.bm - 1) / sh.bm, mu = max_tiles(sh, dtype, d, all_tiles(sh, capacity));
    most = std::max(most, std::min(tiles, std::max((long long)n_cus / ((nq + sh.bn - 1) / sh.bn), (tiles + mu - 1) / mu)));
  }
  return (int)most;
}

hipError_t launch_dense_dump(const DensePlan& p, int dtype, const DenseArgs& a, hipStream_t s) {
  return launch_tiles(dtype, p.shape, kTileDump, a, all_tiles(kShapes[p.shape], a.n_rows), p.n_cus, s, nullptr, nullptr);
}

hipError_t launch_weighted_fuse(int n_cus, const float* D, const float* B, long long ld, long long n, long long n_lex, int nq,
                                const float* mm_d, int pd, const float* mm_l, int pl, double wd, double wl, int k,
                                unsigned long long* cbuf, int* ccnt, float* out_scores, long long* out_ids,
                                hipStream_t s) {
  hipLaunchKernelGGL(weighted_fuse_kernel, dim3((unsigned)nq), dim3(kFuseThreads), 0, s, D, B, ld, n, n_lex, mm_d, pd,
                     mm_l, pl, wd, wl, k, cbuf, ccnt);
  return launch_select(n_cus, cbuf, ccnt, n, nq, k, out_scores, out_ids, nullptr, nullptr, false, s);
}

}  // namespace oprag

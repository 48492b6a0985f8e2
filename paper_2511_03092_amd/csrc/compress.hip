// compress.hip -- SnapStream compression at the end of prefill (arXiv
// 2511.03092, Sec. III-B): SnapKV window scores (Eq. 3), window + group sum
// (Eq. 1), 1-D pooling and top-K (Eq. 2), then the gather into the fixed-size
// sink / ring / top-K cache (Sec. III-A).
//
// Kernel sequence per call (one stream, no host synchronisation):
//   score_pass<STATS>   per (seq, KV head, key chunk): bf16 MFMA Q_obs x K^T,
//                       per-row running max / sum-exp of the softmax domain
//                       (skipped after the prefill attention, which writes
//                       those statistics itself)
//   stats_reduce        per (seq, KV head): row max + normaliser (fp64), and
//                       the reset of the selection scratch
//   score_pass<COLSUM>  recompute the scores, W = exp(z - c) * inv, column
//                       sums over the G*w window rows -> A[j]
//   pool_hist           P = pool(A) over the candidates, histogram of their
//                       leading bits
//   select_refine       histogram of the next bits within the bin that holds
//                       the K-th largest P
//   select_collect      the candidates next to it are listed, those above
//                       counted
//   select_threshold    per (seq, KV head): the K-th largest P among the
//                       listed ones
//   band_rescore/decide fp64 scores next to the threshold, the final decision
//   select_write        ordered compaction: P > t, plus the lowest-index ties
//   assemble            sinks, ring rows, kept rows, zero padding (+ fp8)
#include <float.h>
#include <math.h>
#include <string.h>

#include "band_grid.h"
#include "lds_dma.h"
#include "snap_internal.h"

namespace snap {

// ============================================================ score passes
struct ScoreArgs {
  const void* q;        // [n_seq][Hq][w][D]
  const void* k;        // [n_seq][Hkv][max_len][D]
  const int32_t* lengths;
  float2* stats;        // [n_seq*Hkv][n_kchunks][rows_pad]  (max, sum exp)
  const float2* rowref; // [n_seq*Hkv][rows_pad]             (c, inv)
  float* A;             // [n_seq*Hkv][max_len]
  int Hq, Hkv, G, w, max_len, sink, recent, norm;
  int rows, rows_pad, key_chunk, n_kchunks, groups;
  float scale2;     // scale * log2(e) rounded to fp32 toward zero: logits in log2 units
  float scale2_lo;  // scale * log2(e) - scale2, > 0 (see split_scale2)
};

struct ScoreLane {
  int rpos[2][4];
  bool rval[2][4];
  float rm[2][4], rz[2][4], rc[2][4], rinv[2][4], rinvl[2][4];  // rinvl = rinv * ln2
};

// Normalised weight of one logit: 2^(y - c) * inv with y = acc * (s2 + s2lo).
// y is formed as the rounded product yh plus its exact error and the part of
// scale*log2(e) that fp32 s2 dropped; that small remainder enters to first
// order, 2^(yh + yl - c) = 2^(yh - c) * (1 + yl*ln2), folded into the row factor.
// No contraction here: fused into fma(acc, s2, -c), yh - c would no longer
// carry the rounding of yh that yl corrects, and for c != 0 that error would
// be counted twice.
__device__ __forceinline__ float weight(float acc, float s2, float s2lo, float c, float inv, float invl) {
#pragma clang fp contract(off)
  const float yh = acc * s2;
  float yl = fmaf(acc, s2, -yh);
  yl = fmaf(acc, s2lo, yl);
  return fast_exp2(yh - c) * fmaf(yl, invl, inv);
}

// Scores of one TK-key tile already resident in LDS against this wave's 32
// rows, then either the running row max / sum of powers of two (STATS) or the
// column sums of the normalised weights written to A (COLSUM).  Logits are
// kept in log2 units, y = <q,k> * scale * log2(e), formed by one rounded
// multiply, so exp(z) = exp2(y).  `interior` (uniform) means every key of the
// tile is a candidate that precedes every window row: no per-element masks.
// The work is split per 16-key sub-block into the products (score_mma_sb) and
// the softmax arithmetic (score_epi_sb), so a caller can run the two halves of
// a tile at different times.
//
// LDS fragment reads issued ahead of their MFMAs (measured: 4 is 4% faster
// than the scheduler's own 2 on the latent shape; 6 is no better).
constexpr int kReadAhead = 4;

// Products of sub-block sb (keys sb*16 .. sb*16+15 of the tile): acc[rb] holds
// rows rb*16 + 4*(lane/16) + e (e = 0..3) against key sb*16 + lane%16.
// Layout of a bf16 tile; lane group lg feeds chunk KSTEPS*lg + t of a key to
// k-step t (the same for the queries): 64- and 128-wide keys row by row
// (row_slot; 128-wide statistics pass of 8 ragged prompts 309 -> 278 us),
// 576-wide ones chunk by chunk (row by row they took 878 instead of 681 us: the
// addresses of 18 k-steps cost registers, and one workgroup per CU has the
// whole L1 for a tile's lines).
template <int KSTEPS, int TK>
__device__ __forceinline__ int fragment_slot(int key, int t, int lg) {
  return KSTEPS <= 4 ? row_slot<KSTEPS * 4>(key, KSTEPS * lg + t) : tile_slot<TK>(key, KSTEPS * lg + t);
}

// Sum over the four lanes l, l^16, l^32, l^48 by the lane-swap instructions (no
// LDS round trip).
__device__ __forceinline__ float lanes4_sum(float x) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

template <typename In, int KSTEPS, int TK>
__device__ __forceinline__ void score_mma_sb(const unsigned char* __restrict__ ktile, const bf16x8 (&qf)[2][KSTEPS],
                                             const float* qlds, int sb, int wave, int lane, bool wave_has_rows,
                                             f32x4 (&acc)[2]) {
  constexpr bool kBF16 = sizeof(In) == 2;
  constexpr int D = KSTEPS * 32;
  const int l16 = lane & 15, lg = lane >> 4;
  const int key = sb * 16 + l16;
  acc[0] = f32x4{0.f, 0.f, 0.f, 0.f};
  acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (kBF16) {
    // waves without score rows multiply zero fragments (only tiny cases have them).
    // Even and odd k-steps accumulate in separate chains (shorter fp32
    // accumulation, two independent MFMA chains), summed at the end.
    f32x4 odd[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < KSTEPS; ++t) {
      bf16x8 kf = __builtin_bit_cast(bf16x8, *(const u32x4*)(ktile + (size_t)fragment_slot<KSTEPS, TK>(key, t, lg) * 16));
      if (t & 1) {
        odd[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[0][t], kf, odd[0], 0, 0, 0);
        odd[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[1][t], kf, odd[1], 0, 0, 0);
      } else {
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[0][t], kf, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[1][t], kf, acc[1], 0, 0, 0);
      }
    }
    // the fragment reads run kReadAhead k-steps ahead of the MFMAs that use
    // them, so their LDS latency hides behind earlier products
    __builtin_amdgcn_sched_group_barrier(0x100, kReadAhead, 0);  // DS reads
#pragma unroll
    for (int t = 0; t < KSTEPS - kReadAhead; ++t) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2 * kReadAhead, 0);
    acc[0] += odd[0];
    acc[1] += odd[1];
  } else if (wave_has_rows) {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float* qrow = qlds + (size_t)(wave * 32 + rb * 16 + lg * 4 + e) * D;
        // fp32 products are exact in fp64; only the final rounding remains
        double sacc = 0.0;
#pragma unroll 4
        for (int d = 0; d < D; ++d) {
          const float kd = *(const float*)(ktile + (size_t)tile_slot<TK>(key, d >> 2) * 16 + (d & 3) * 4);
          sacc = fma((double)qrow[d], (double)kd, sacc);
        }
        acc[rb][e] = (float)sacc;
      }
  }
}

// Softmax arithmetic of sub-block sb from its products: STATS keeps the
// products (masked ones at -inf) in xv for score_stats_tile; COLSUM writes this
// wave's column sums of the normalised weights to colbuf.
template <int NW, bool COLSUM, int TK>
__device__ __forceinline__ void score_epi_sb(const ScoreArgs& a, const f32x4 (&acc)[2], float* colbuf,
                                             const ScoreLane& sl, int t0, int c1, bool interior, int sb, int wave,
                                             int lane, float (&xv)[2][4][TK / 16]) {
  const int l16 = lane & 15, lg = lane >> 4;
  const float s2 = a.scale2, s2lo = a.scale2_lo;
  const int key = sb * 16 + l16;
  const int j = t0 + key;
  if (!COLSUM) {
    // the raw products: score_stats_tile forms each exponent from them with
    // the full scale (s2 + s2lo), as the column-sum weights do
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int e = 0; e < 4; ++e) xv[rb][e][sb] = acc[rb][e];
    if (!interior) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!(sl.rval[rb][e] && j < c1 && j <= sl.rpos[rb][e])) xv[rb][e][sb] = -INFINITY;
    }
  } else {
    float colv[2][4];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        colv[rb][e] = weight(acc[rb][e], s2, s2lo, sl.rc[rb][e], sl.rinv[rb][e], sl.rinvl[rb][e]);
    if (!interior) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!(sl.rval[rb][e] && j < c1 && j <= sl.rpos[rb][e])) colv[rb][e] = 0.f;
    }
    float cs = ((colv[0][0] + colv[0][1]) + (colv[0][2] + colv[0][3])) +
               ((colv[1][0] + colv[1][1]) + (colv[1][2] + colv[1][3]));
    cs = lanes4_sum(cs);
    if (lg == 0) colbuf[wave * TK + sb * 16 + l16] = cs;
  }
}

// STATS: fold one tile's products into the running row max / sum (log2
// units).  The reference mn is the rounded max of acc * s2; each term's
// exponent acc * (s2 + s2lo) - mn is formed with two fused steps, so the row
// sum carries neither the rounding of acc * s2 nor the part of the scale that
// fp32 s2 drops -- the same logits the column-sum weights use, whose sum it
// normalises.  s2lo > 0 keeps a masked -inf product at -inf.
__device__ __forceinline__ float stats_term(float x, float s2, float s2lo, float mn) {
  return fast_exp2(fmaf(x, s2lo, fmaf(x, s2, -mn)));
}
template <int TK>
__device__ __forceinline__ void score_stats_tile(ScoreLane& sl, const float (&xv)[2][4][TK / 16], float s2,
                                                 float s2lo) {
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* x = xv[rb][e];
      float mt, mn;
      if constexpr (TK == 64) {
        mt = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
      } else {
        mt = fmaxf(x[0], x[1]);
      }
      mn = fmaxf(sl.rm[rb][e], mt * s2);
      if (mn == -INFINITY) continue;
      float z = sl.rz[rb][e] * fast_exp2(sl.rm[rb][e] - mn);
      if constexpr (TK == 64) {
        z += (stats_term(x[0], s2, s2lo, mn) + stats_term(x[1], s2, s2lo, mn)) +
             (stats_term(x[2], s2, s2lo, mn) + stats_term(x[3], s2, s2lo, mn));
      } else {
        z += stats_term(x[0], s2, s2lo, mn) + stats_term(x[1], s2, s2lo, mn);
      }
      sl.rz[rb][e] = z;
      sl.rm[rb][e] = mn;
    }
}

// The whole tile in one go: products and softmax arithmetic sub-block by
// sub-block.
template <typename In, int KSTEPS, int NW, bool COLSUM, int TK>
__device__ __forceinline__ void score_tile(const ScoreArgs& a, const unsigned char* __restrict__ ktile,
                                           const bf16x8 (&qf)[2][KSTEPS], const float* qlds, float* colbuf,
                                           ScoreLane& sl, int t0, int c1, bool interior, int bg, int wave,
                                           int lane, bool wave_has_rows) {
  static_assert(TK == 64 || TK == 32, "tile of 64 or 32 keys");
  float xv[2][4][TK / 16];
#pragma unroll
  for (int sb = 0; sb < TK / 16; ++sb) {
    f32x4 acc[2];
    score_mma_sb<In, KSTEPS, TK>(ktile, qf, qlds, sb, wave, lane, wave_has_rows, acc);
    score_epi_sb<NW, COLSUM, TK>(a, acc, colbuf, sl, t0, c1, interior, sb, wave, lane, xv);
  }
  if (!COLSUM) score_stats_tile<TK>(sl, xv, a.scale2, a.scale2_lo);
}

// Column sums of one tile across the NW waves (fixed order), written to A.
// The caller places a barrier between the waves' colbuf writes and this.
template <int NW, int TK>
__device__ __forceinline__ void colsum_finish(const ScoreArgs& a, const float* colbuf, int t0, int c1, int bg) {
  if (tid() < TK) {
    const int j = t0 + tid();
    const float* c = colbuf + tid();
    float sum;
    if constexpr (NW == 4) {
      sum = (c[0] + c[TK]) + (c[2 * TK] + c[3 * TK]);
    } else {
      sum = ((c[0] + c[TK]) + (c[2 * TK] + c[3 * TK])) + ((c[4 * TK] + c[5 * TK]) + (c[6 * TK] + c[7 * TK]));
    }
    if (j < c1) a.A[(size_t)bg * a.max_len + j] = sum;
  }
}

// Row state of one lane: the MFMA 16x16 output gives lane l the rows
// 4*(l/16)+e (e = 0..3) of each 16-row block and the key column l%16.
// NW waves per workgroup; wave w owns score rows [32w, 32w+32).  Key tiles of
// TK keys stream through a ring of STAGES LDS stages with direct loads: while
// a tile is scored, the next STAGES-1 are in flight (the bytes in flight per
// CU, not the compute, bound a pass with fewer stages).
template <typename In, int KSTEPS, int NW, bool COLSUM, int TK, int STAGES>
__global__ __launch_bounds__(NW * 64) void score_pass(ScoreArgs a) {
  constexpr bool kBF16 = sizeof(In) == 2;
  constexpr int D = KSTEPS * 32;
  constexpr int kRowBytes = D * (int)sizeof(In);
  constexpr int CPR = kRowBytes / 16;                 // 16-byte chunks per key row
  constexpr int kTileBytes = TK * kRowBytes;
  __shared__ __align__(16) unsigned char tiles[STAGES][kTileBytes];
  __shared__ float colbuf[2][NW * TK];  // column partials, double-buffered for the ring
  __shared__ float qlds[kBF16 ? 1 : 128 * D];           // fp32 inputs: [rows_pad <= 128][D]

  const int lane = tid() & 63, wave = tid() >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  // the column sums run in the reverse order of the statistics, so that what
  // the last-level cache still holds of the keys is read first
  const int bg = COLSUM ? a.groups - 1 - bid_y() : bid_y();
  const int chunk = COLSUM ? a.n_kchunks - 1 - bid_x() : bid_x();
  const int b = bg / a.Hkv, g = bg % a.Hkv;
  int L = uniform(a.lengths[b]);
  L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
  const int s = a.sink, r = a.recent;
  const int clo = s, chi = L - r;  // candidates [clo, chi)
  int lo, hi;
  if (COLSUM || a.norm == SNAP_NORM_CAND) {
    lo = clo;
    hi = chi;
  } else {
    lo = 0;
    hi = L;
  }
  const int c0 = lo + chunk * a.key_chunk;
  int c1 = min(c0 + a.key_chunk, hi);
  if (!debug_check(c0 >= 0 && c1 <= a.max_len, kDbgScoreRange)) c1 = c0;  // skip the chunk
  const int we = min(a.w, L);
  const bool wave_has_rows = wave * 32 < a.rows;

  ScoreLane sl;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      int rho = wave * 32 + rb * 16 + lg * 4 + e;
      int ii = rho % a.w;
      sl.rval[rb][e] = rho < a.rows && ii >= a.w - we;
      sl.rpos[rb][e] = L - a.w + ii;
    }

  float2* st_out = a.stats + ((size_t)bg * a.n_kchunks + chunk) * a.rows_pad;
  if (c0 >= c1) {
    if (!COLSUM) {
      for (int t = tid(); t < a.rows_pad; t += nthreads()) st_out[t] = make_float2(-INFINITY, 0.f);
    }
    return;
  }

  const unsigned char* kbase =
      (const unsigned char*)a.k + ((size_t)b * a.Hkv + g) * (size_t)a.max_len * kRowBytes;

  // ---- query rows of this wave
  const In* qbase = (const In*)a.q + ((size_t)b * a.Hq + (size_t)g * a.G) * a.w * D;
  bf16x8 qf[2][KSTEPS];
  if constexpr (kBF16) {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      int rho = wave * 32 + rb * 16 + l16;
      int ii = rho % a.w;
      bool ok = rho < a.rows && ii >= a.w - we;
#pragma unroll
      for (int t = 0; t < KSTEPS; ++t) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (ok) v = *(const u32x4*)(qbase + (size_t)rho * D + 8 * (KSTEPS * lg + t));
        qf[rb][t] = __builtin_bit_cast(bf16x8, v);
      }
    }
  } else {
    for (int i = tid(); i < a.rows_pad * D; i += nthreads()) {
      int rho = i / D;
      qlds[i] = rho < a.rows ? ((const float*)qbase)[i] : 0.f;
    }
  }

#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sl.rm[rb][e] = -INFINITY;
      sl.rz[rb][e] = 0.f;
      if (COLSUM) {
        int rho = wave * 32 + rb * 16 + lg * 4 + e;
        float2 rf = rho < a.rows_pad ? a.rowref[(size_t)bg * a.rows_pad + rho] : make_float2(0.f, 0.f);
        sl.rc[rb][e] = sl.rval[rb][e] ? rf.x : 0.f;  // already in log2 units
        sl.rinv[rb][e] = sl.rval[rb][e] ? rf.y : 0.f;
        sl.rinvl[rb][e] = sl.rinv[rb][e] * 0.69314718055994531f;
      }
    }
  // The query fragments and row normalisers must have landed before the first
  // tile load is issued: the loop's waits only count tile loads (stores issued
  // later only add to the count, which makes those waits stricter).
  wait_vm<0>();
  const int nt = (c1 - c0 + TK - 1) / TK;  // tiles of this chunk
  constexpr bool kRowMajor = kBF16 && KSTEPS <= 4;  // as fragment_slot
  static_assert(!kRowMajor || STAGES == 2, "the ring loads chunk-major tiles");
  const int nload = tile_loads<CPR, NW, TK>(__builtin_amdgcn_readfirstlane(wave));
  // a tile is interior when all its keys are in range and precede the first
  // window position (rows of negative position exist only when L < w)
  const int first_row_pos = L - a.w;
  auto interior_of = [&](int t) { return t + TK <= c1 && t + TK - 1 <= first_row_pos; };

  if constexpr (STAGES == 2) {
    TileLoad<CPR, NW, TK> tl;
    if constexpr (kRowMajor) tl.init(wave, lane);
    auto issue = [&](int t0, unsigned char* buf) {
      if constexpr (kRowMajor)
        tl.issue(kbase, t0, c1, buf);
      else
        issue_tile<CPR, NW, TK>(kbase, kRowBytes, t0, c1, buf, wave, lane);
    };
    issue(c0, &tiles[0][0]);
    // Double buffer, one barrier per tile: past the barrier of a tile it has
    // landed for every wave, and every wave is done with the tile before it,
    // whose stage takes the next tile and whose column partials (the other
    // colbuf half) are summed.
    auto step = [&](int t0, int i, unsigned char* cur, unsigned char* nxt) {
      wait_vm<0>();
      lds_barrier();
      if (t0 + TK < c1) issue(t0 + TK, nxt);
      if constexpr (COLSUM) {
        if (t0 > c0) colsum_finish<NW, TK>(a, colbuf[(i - 1) & 1], t0 - TK, c1, bg);
      }
      score_tile<In, KSTEPS, NW, COLSUM, TK>(a, cur, qf, qlds, colbuf[i & 1], sl, t0, c1, interior_of(t0), bg, wave,
                                             lane, wave_has_rows);
    };
    for (int t0 = c0; t0 < c1; t0 += 2 * TK) {
      step(t0, 0, &tiles[0][0], &tiles[1][0]);
      if (t0 + TK < c1) step(t0 + TK, 1, &tiles[1][0], &tiles[0][0]);
    }
    if constexpr (COLSUM) {
      lds_barrier();
      colsum_finish<NW, TK>(a, colbuf[(nt - 1) & 1], c0 + (nt - 1) * TK, c1, bg);
    }
  } else {
    // Ring, one barrier per tile: past the barrier of tile i every wave has
    // finished tile i-1, so its stage takes tile i+STAGES-1 right away and
    // its column partials (the other colbuf half) can be summed.
    for (int st = 0; st < STAGES - 1 && st < nt; ++st)
      issue_tile<CPR, NW, TK>(kbase, kRowBytes, c0 + st * TK, c1, &tiles[st][0], wave, lane);
    for (int i = 0; i < nt; ++i) {
      wait_vm_dyn(min(nt - 1 - i, STAGES - 2) * nload);  // tile i has landed
      lds_barrier();                                      // ... for every wave
      const int t = c0 + i * TK;
      if (i + STAGES - 1 < nt)
        issue_tile<CPR, NW, TK>(kbase, kRowBytes, t + (STAGES - 1) * TK, c1, &tiles[(i + STAGES - 1) % STAGES][0], wave, lane);
      if constexpr (COLSUM) {
        if (i > 0) colsum_finish<NW, TK>(a, colbuf[(i - 1) & 1], t - TK, c1, bg);
      }
      score_tile<In, KSTEPS, NW, COLSUM, TK>(a, &tiles[i % STAGES][0], qf, qlds, colbuf[i & 1], sl, t, c1,
                                             interior_of(t), bg, wave, lane, wave_has_rows);
    }
    if constexpr (COLSUM) {
      lds_barrier();
      colsum_finish<NW, TK>(a, colbuf[(nt - 1) & 1], c0 + (nt - 1) * TK, c1, bg);
    }
  }

  if (!COLSUM) {
    // combine the 16 key columns of each row (lanes with equal l/16)
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float m = sl.rm[rb][e], z = sl.rz[rb][e];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
          float m2 = __shfl_xor(m, o), z2 = __shfl_xor(z, o);
          float mn = fmaxf(m, m2);
          if (mn != -INFINITY) {
            z = z * fast_exp2(m - mn) + z2 * fast_exp2(m2 - mn);
            m = mn;
          }
        }
        const int rho = wave * 32 + rb * 16 + lg * 4 + e;
        if (l16 == 0 && rho < a.rows_pad) st_out[rho] = make_float2(m, z);
      }
  }
}

// ============================================================ streaming score passes
// 64- and 128-wide bf16 keys, at most 64 score rows.  Every wave holds all score
// rows of the group as query fragments (RB blocks of 16 rows, RB * KS * 4
// registers) and streams its own 16 keys at a time from memory into registers:
// no LDS and no barrier in the loop, two tiles in flight while one is scored.
// The product is S^T = K Q^T (A = 16 keys, B = 16 rows), so a lane holds one row
// of each block against 4 * (lane / 16) + e of 16 keys: the row constants are one
// register per block, a row's running (max, sum) is lane-local until the end, and
// the column sums are an in-lane sum over the blocks and a reduction over 16
// lanes.  The statistics' reference moves lazily (kStatsLag), which the LDS pass
// gains nothing from: here it saves the rescale of every block's sums per 16 keys.
template <int N>
__device__ __forceinline__ float row_ror_add(float x) {
  const int r = __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N, 0xf, 0xf, true);
  return x + __int_as_float(r);
}

constexpr float kStatsLag = 8.f;  // log2 units the statistics' reference may lag a row's max

template <int KS, int RB, bool COLSUM>
__global__ __launch_bounds__(256) void score_stream(ScoreArgs a) {
  constexpr int D = KS * 32;
  constexpr int NW = 4;
  __shared__ float2 part[COLSUM ? 1 : NW * RB * 16];
  __shared__ int rpos[RB * 16];  // position of the row, or -1: not a row
  const int lane = tid() & 63, wave = __builtin_amdgcn_readfirstlane(tid() >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  // the column sums run in the reverse order of the statistics, so that what
  // the last-level cache still holds of the keys is read first
  const int bg = COLSUM ? a.groups - 1 - bid_y() : bid_y();
  const int chunk = COLSUM ? a.n_kchunks - 1 - bid_x() : bid_x();
  const int b = bg / a.Hkv, g = bg % a.Hkv;
  int L = uniform(a.lengths[b]);
  L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
  int lo = a.sink, hi = L - a.recent;
  if (!COLSUM && a.norm != SNAP_NORM_CAND) {
    lo = 0;
    hi = L;
  }
  const int c0 = lo + chunk * a.key_chunk;
  int c1 = min(c0 + a.key_chunk, hi);
  if (!debug_check(c0 >= 0 && c1 <= a.max_len, kDbgScoreRange)) c1 = c0;  // skip the chunk
  float2* st_out = a.stats + ((size_t)bg * a.n_kchunks + chunk) * a.rows_pad;
  if (c0 >= c1) {
    if (!COLSUM) {
      for (int t = tid(); t < a.rows_pad; t += nthreads()) st_out[t] = make_float2(-INFINITY, 0.f);
    }
    return;
  }
  const int we = min(a.w, L);
  const unsigned char* kbase =
      (const unsigned char*)a.k + ((size_t)b * a.Hkv + g) * (size_t)a.max_len * (D * 2);

  // 16 keys at t: this lane's chunks of key t + l16 (keys past c1 read key
  // c1 - 1; they are masked)
  auto load = [&](int t, u32x4 (&k)[KS]) {
    const int j = min(t + l16, c1 - 1);
    const unsigned char* p = kbase + (size_t)j * (D * 2) + lg * 16;
#pragma unroll
    for (int s = 0; s < KS; ++s) k[s] = *(const u32x4*)(p + s * 64);
  };
  constexpr int kStep = 16 * NW;  // keys of one turn of the workgroup
  int t = c0 + 16 * wave;
  u32x4 k0[KS], k1[KS], k2[KS];
  if (t < c1) load(t, k0);
  if (t + kStep < c1) load(t + kStep, k1);

  const uint16_t* qbase = (const uint16_t*)a.q + ((size_t)b * a.Hq + (size_t)g * a.G) * a.w * D;
  bf16x8 qf[RB][KS];
  float s0[RB], s1[RB];  // STATS: reference, sum; COLSUM: reference, 1/normaliser
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int rho = rb * 16 + l16;
    const int ii = rho % a.w;
    const bool ok = rho < a.rows && ii >= a.w - we;
    if (wave == 0 && lg == 0) rpos[rho] = ok ? L - a.w + ii : -1;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (ok) v = *(const u32x4*)(qbase + (size_t)rho * D + 8 * (4 * s + lg));
      qf[rb][s] = __builtin_bit_cast(bf16x8, v);
    }
    if (COLSUM) {
      const float2 rf = ok ? a.rowref[(size_t)bg * a.rows_pad + rho] : make_float2(0.f, 0.f);
      s0[rb] = rf.x;
      s1[rb] = rf.y;
    } else {
      s0[rb] = -INFINITY;
      s1[rb] = 0.f;
    }
  }
  __syncthreads();  // rpos
  const float s2 = a.scale2, s2lo = a.scale2_lo;
  const int first_row_pos = L - a.w;

  auto score = [&](int t, const u32x4 (&k)[KS]) {
    // every key in range and before the first window position: nothing masked
    const bool interior = t + 16 <= c1 && t + 15 <= first_row_pos;
    float cs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      // even and odd k-steps in chains of their own, summed at the end
      f32x4 x = {0.f, 0.f, 0.f, 0.f}, od = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; s += 2) {
        x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[s]), qf[rb][s], x, 0, 0, 0);
        od = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[s + 1]), qf[rb][s + 1], od, 0, 0, 0);
      }
      x += od;
      if constexpr (!COLSUM) {
        if (!interior) {
          const int rp = min(rpos[rb * 16 + l16], c1 - 1);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (t + 4 * lg + e > rp) x[e] = -INFINITY;
        }
        // the reference moves only when a term would pass 2^kStatsLag
        const float mt = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])) * s2;
        if (wave_any(mt > s0[rb] + kStatsLag)) {
          const float mn = fmaxf(s0[rb], mt);
          s1[rb] *= fast_exp2(s0[rb] - (mn == -INFINITY ? 0.f : mn));
          s0[rb] = mn;
        }
        const float mu = s0[rb] == -INFINITY ? 0.f : s0[rb];  // nothing seen yet: every term is 0
        s1[rb] += (stats_term(x[0], s2, s2lo, mu) + stats_term(x[1], s2, s2lo, mu)) +
                  (stats_term(x[2], s2, s2lo, mu) + stats_term(x[3], s2, s2lo, mu));
      } else {
        const float invl = s1[rb] * 0.69314718055994531f;
        float wv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) wv[e] = weight(x[e], s2, s2lo, s0[rb], s1[rb], invl);
        if (!interior) {
          const int rp = min(rpos[rb * 16 + l16], c1 - 1);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (t + 4 * lg + e > rp) wv[e] = 0.f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) cs[e] += wv[e];
      }
    }
    if constexpr (COLSUM) {
      // over the 16 rows of a block (lanes of equal lg); lane l16 = e < 4
      // stores key 4lg + e
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        cs[e] = row_ror_add<8>(cs[e]);
        cs[e] = row_ror_add<4>(cs[e]);
        cs[e] = row_ror_add<2>(cs[e]);
        cs[e] = row_ror_add<1>(cs[e]);
      }
      const float lo2 = (l16 & 1) ? cs[1] : cs[0], hi2 = (l16 & 1) ? cs[3] : cs[2];
      const int j = t + 4 * lg + l16;
      if (l16 < 4 && j < c1) a.A[(size_t)bg * a.max_len + j] = (l16 & 2) ? hi2 : lo2;
    }
  };

  // three buffers in turn, two tiles in flight while one is scored
  for (; t < c1; t += 3 * kStep) {
    if (t + 2 * kStep < c1) load(t + 2 * kStep, k2);
    score(t, k0);
    if (t + kStep >= c1) break;
    if (t + 3 * kStep < c1) load(t + 3 * kStep, k0);
    score(t + kStep, k1);
    if (t + 2 * kStep >= c1) break;
    if (t + 4 * kStep < c1) load(t + 4 * kStep, k1);
    score(t + 2 * kStep, k2);
  }

  if constexpr (!COLSUM) {
    // a row's four lane groups, then the waves
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float m = s0[rb], z = s1[rb];
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float m2 = __shfl_xor(m, o), z2 = __shfl_xor(z, o);
        const float mn = fmaxf(m, m2);
        if (mn != -INFINITY) {
          z = z * fast_exp2(m - mn) + z2 * fast_exp2(m2 - mn);
          m = mn;
        }
      }
      if (lg == 0) part[(wave * RB + rb) * 16 + l16] = make_float2(m, z);
    }
    __syncthreads();
    for (int rho = tid(); rho < a.rows_pad; rho += nthreads()) {
      float m = -INFINITY, z = 0.f;
#pragma unroll
      for (int w2 = 0; w2 < NW; ++w2) {
        const float2 p = part[w2 * RB * 16 + rho];
        const float mn = fmaxf(m, p.x);
        if (mn != -INFINITY) {
          z = z * fast_exp2(m - mn) + p.y * fast_exp2(p.x - mn);
          m = mn;
        }
      }
      st_out[rho] = make_float2(m, z);
    }
  }
}

// ============================================================ row normalisers
struct ReduceArgs {
  const float2* stats;
  float2* rowref;
  double2* rowz;       // [groups][rows_pad] (max in log2 units, sum of 2^(y - max)) in fp64
  int32_t* band_n;     // [groups] members of the re-score band (reset here)
  const int32_t* lengths;
  int32_t* list_n;     // [groups] listed candidates (reset here)
  uint32_t* hist;      // [groups][kHistBins + kSubBins]
  RadixState* state;   // [groups]
  int groups, Hkv, max_len, sink, recent, topk;
  int rows_pad, n_kchunks, reset_wgs;  // reset_wgs: workgroups per group
};

// Row max m over every chunk and the normaliser, in log2 units (the stats
// pass keeps m2 = max y and sum 2^(y - m2) with y = z*log2(e)).  The reference
// c2 is 0 when the natural-log max lies in [-20, 64] (then 2^y is taken
// directly, keeping the full fp32 accuracy of small logits), otherwise
// c2 = m2; inv = 1 / sum_j 2^(y_j - c2), accumulated in fp64.  A wave owns a
// row (chunks strided by 64, a few hundred at most) and combines with in-wave
// shuffles; the group's workgroups also reset its selection scratch.
constexpr int kReduceLanes = 64;
constexpr int kReduceRows = 256 / kReduceLanes;  // rows per workgroup
__global__ __launch_bounds__(256) void stats_reduce(ReduceArgs a) {
  const int bg = bid_y(), b = bg / a.Hkv;
  const int sub = tid() % kReduceLanes;
  const int rho = bid_x() * kReduceRows + tid() / kReduceLanes;
  const float2* st = a.stats + (size_t)bg * a.n_kchunks * a.rows_pad;
  if (rho < a.rows_pad) {
    float m = -INFINITY;
    for (int c = sub; c < a.n_kchunks; c += kReduceLanes) m = fmaxf(m, st[(size_t)c * a.rows_pad + rho].x);
#pragma unroll
    for (int o = 1; o < kReduceLanes; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
    double z = 0.0;
    if (m != -INFINITY) {
      for (int c = sub; c < a.n_kchunks; c += kReduceLanes) {
        float2 v = st[(size_t)c * a.rows_pad + rho];
        if (v.x != -INFINITY) z += (double)v.y * exp2((double)v.x - (double)m);
      }
    }
#pragma unroll
    for (int o = 1; o < kReduceLanes; o <<= 1) z += __shfl_xor(z, o);
    if (sub == 0) {
      float2 ref = make_float2(0.f, 0.f);
      if (m != -INFINITY) {
        const double m_nat = (double)m * 0.69314718055994530942;
        if (m_nat >= -20.0 && m_nat <= 64.0) {
          ref.x = 0.f;
          ref.y = (float)(1.0 / (z * exp2((double)m)));
        } else {
          ref.x = m;
          ref.y = (float)(1.0 / z);
        }
      }
      a.rowref[(size_t)bg * a.rows_pad + rho] = ref;
      a.rowz[(size_t)bg * a.rows_pad + rho] = make_double2((double)m, z);
    }
  }
  {
    constexpr int kAll = kHistBins + kSubBins;
    const int per = (kAll + a.reset_wgs - 1) / a.reset_wgs;
    uint32_t* h = a.hist + (size_t)bg * kAll;
    for (int i = bid_x() * per + tid(); i < min((bid_x() + 1) * per, kAll); i += nthreads()) h[i] = 0u;
  }
  if (bid_x() != 0) return;
  if (tid() == 0) {
    a.band_n[bg] = 0;
    a.list_n[bg] = 0;
  }
  if (tid() == 0) {
    int L = uniform(a.lengths[b]);
    L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
    int n = L - a.sink - a.recent;
    n = n < 0 ? 0 : n;
    int keff = n < a.topk ? n : a.topk;
    RadixState s;
    s.prefix = 0u;
    s.krem = keff;
    s.keff = keff;
    s.mode = keff == 0 ? 0 : (keff == n ? 1 : 2);
    s.bin = s.sub = s.pad[0] = s.pad[1] = 0;
    a.state[bg] = s;
  }
}

// ============================================================ pooling + selection
struct SelectArgs {
  const float* A;        // [groups][max_len]
  float* P;              // [groups][max_len]
  float* pooled_out;     // optional [groups][max_len]
  const int32_t* lengths;
  uint32_t* hist;        // [groups][kHistBins + kSubBins]
  uint2* list;           // [groups][kListCap] (score bits, token) of the candidates next to the K-th largest
  int32_t* list_n;       // [groups] how many there are (more than kListCap: the list is not used)
  RadixState* state;     // [groups]
  uint2* counts;         // [groups][n_splits] (greater, equal)
  int32_t* sel;          // [groups][topk]
  int32_t* band_n;       // [groups] candidates in the re-score band
  int32_t* band_idx;     // [groups][kBandCap] their token indices (in arrival order)
  uint32_t* band_above;  // [groups][n_splits] candidates above the band per split
  int groups, Hkv, max_len, sink, recent, topk, pool_kernel, pool, n_splits;
  uint32_t hist_top;     // leading bits of the largest score there can be (the number of score rows)
};

// The re-score band around the K-th largest pooled score tau (fp32 bits of a
// non-negative value): [tau (1 - 2^-17), tau (1 + 2^-17)] as bit patterns.
// The fp32 score path is accurate to under 2e-6 relative (measured up to
// 1.6e-6 anywhere, 1.2e-6 near the threshold with one window row), so a
// candidate outside the band cannot be on the other side of the threshold.
constexpr float kBandRel = 1.0f / 131072.0f;
__device__ __forceinline__ void band_limits(uint32_t tau_bits, uint32_t& lo, uint32_t& hi) {
  const float t = __uint_as_float(tau_bits);
  lo = __float_as_uint(t * (1.0f - kBandRel));
  hi = __float_as_uint(t * (1.0f + kBandRel));
}

// the group's selection state, with every field in scalar registers
__device__ __forceinline__ RadixState load_state(const RadixState* p) {
  RadixState s = *p;
  s.prefix = (uint32_t)uniform((int)s.prefix);
  s.bin = uniform(s.bin);
  s.sub = uniform(s.sub);
  s.krem = uniform(s.krem);
  s.keff = uniform(s.keff);
  s.mode = uniform(s.mode);
  return s;
}

__device__ __forceinline__ void seq_range(const SelectArgs& a, int bg, int& c0, int& c1) {
  int b = bg / a.Hkv;
  int L = uniform(a.lengths[b]);
  L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
  c0 = a.sink;
  c1 = L - a.recent;
  if (c1 < c0) c1 = c0;
}

// Bin of a pooled score: its exponent and six bits of mantissa, the highest bin
// for the largest score there can be (the number of score rows) and above, the
// lowest for everything 64 octaves below that.
__device__ __forceinline__ int hist_bin(uint32_t bits, uint32_t top) {
  const int d = (int)(bits >> 17) - (int)top + (kHistBins - 1);
  return d < 0 ? 0 : (d > kHistBins - 1 ? kHistBins - 1 : d);
}
// The bit patterns [lo, hi] of a bin, and how far they are shifted down (from
// lo) to their place among the bin's kSubBins parts: 6 bits, so that a part is
// at most 2^-17 of its scores wide, except in the two end bins.
__device__ __forceinline__ void bin_limits(int bin, uint32_t top, uint32_t& lo, uint32_t& hi, int& shift) {
  const uint32_t first = (top - (kHistBins - 1) + (uint32_t)bin) << 17;
  lo = bin == 0 ? 0u : first;
  hi = bin == kHistBins - 1 ? 0xffffffffu : first | 0x1ffffu;
  shift = 32 - __builtin_clz(hi - lo) - kSubBits;
}

// block-wide exclusive scan of one value per thread (lds holds one value per wave)
__device__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* lds, uint32_t& total) {
  const int lane = tid() & 63, wave = tid() >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) lds[wave] = x;
  __syncthreads();
  uint32_t base = 0;
  total = 0;
  for (int w2 = 0; w2 < (int)(nthreads() >> 6); ++w2) {
    uint32_t t = lds[w2];
    if (w2 < wave) base += t;
    total += t;
  }
  __syncthreads();
  return base + x - v;
}

constexpr int kPerThread = kCandChunk / kSelThreads;  // candidates per thread

// P = pool(A) on this workgroup's candidates (+ the debug copy) and the
// histogram of their bins.  Bins of 1.6% keep the pooled scores, which crowd
// within an octave or two, from serialising on a few LDS counters, and the
// lanes of a run with one bin (max pooling repeats a score over its window) add
// once for the run, so one histogram serves the workgroup (three radix passes
// with per-wave histograms of eight bins per octave, a scan launch each and a
// count before this, select_refine, select_collect and select_threshold: 109 us
// for 64 groups of up to 128k candidates, 41 us for 8 groups of 48k; now 52 and
// 25 us).
__global__ __launch_bounds__(kSelThreads) void pool_hist(SelectArgs a) {
  __shared__ float la[kCandChunk + 64];
  __shared__ uint32_t lhist[kHistBins];
  const int bg = bid_y(), split = bid_x();
  const int lane = tid() & 63;
  int c0, c1;
  seq_range(a, bg, c0, c1);
  const int half = a.pool_kernel / 2;
  const int j0 = c0 + split * kCandChunk, j1 = min(j0 + kCandChunk, c1);
  const int mode = uniform(a.state[bg].mode);
  float* Pg = a.P + (size_t)bg * a.max_len;

  if (a.pooled_out && split == 0) {
    float* po = a.pooled_out + (size_t)bg * a.max_len;
    for (int j = tid(); j < a.max_len; j += nthreads())
      if (j < c0 || j >= c1) po[j] = __uint_as_float(kQuietNaN);
  }
  if (j0 >= j1) return;
  const float* Ag = a.A + (size_t)bg * a.max_len;
  const float padv = a.pool == SNAP_POOL_MAX ? -INFINITY : 0.f;
#pragma unroll 4
  for (int i = tid(); i < (j1 - j0) + 2 * half; i += nthreads()) {
    int t = j0 - half + i;
    la[i] = (t >= c0 && t < c1) ? Ag[t] : padv;
  }
  if (mode == 2)
    for (int i = tid(); i < kHistBins; i += nthreads()) lhist[i] = 0u;
  __syncthreads();
  for (int jj = j0; jj < j1; jj += nthreads()) {  // whole waves stay in the loop
    const int j = jj + tid();
    const bool in = j < j1;
    float v = 0.f;
    if (in) {
      const float* w = la + (j - j0);
      if (a.pool == SNAP_POOL_MAX) {
        v = w[0];
#pragma unroll 6
        for (int t = 1; t < a.pool_kernel; ++t) v = fmaxf(v, w[t]);
      } else {
#pragma unroll 4
        for (int t = 0; t < a.pool_kernel; ++t) v += w[t];
        v = v / (float)a.pool_kernel;
      }
      Pg[j] = v;
      if (a.pooled_out) a.pooled_out[(size_t)bg * a.max_len + j] = v;
    }
    if (mode == 2) {
      const int d = in ? hist_bin(__float_as_uint(v), a.hist_top) : -1;
      const int prev = __shfl_up(d, 1);
      const bool start = lane == 0 || prev != d;
      const uint64_t starts = __builtin_amdgcn_ballot_w64(start);
      const uint64_t after = lane == 63 ? 0 : starts >> (lane + 1);
      const int run = after ? __builtin_ctzll(after) + 1 : 64 - lane;
      if (start && in) atomicAdd(&lhist[d], (uint32_t)run);
    }
  }
  if (mode != 2) return;
  __syncthreads();
  uint32_t* gh = a.hist + (size_t)bg * (kHistBins + kSubBins);
  for (int i = tid(); i < kHistBins; i += nthreads()) {
    const uint32_t v = lhist[i];
    if (v) atomicAdd(&gh[i], v);
  }
}

// Bin of the want-th largest entry of the histogram h[NB] (counted from the top
// bin down), and what is left of `want` within it.  Thread t owns the bins just
// below those of thread t-1, so its exclusive prefix is the count above its
// bins.  Every thread of the workgroup (kSelThreads) calls it and gets the
// result; it holds two barriers after pick is written.
template <int NB>
__device__ __forceinline__ int find_bin(const uint32_t* h, uint32_t& want, uint32_t* lds, uint32_t* pick) {
  constexpr int kBins = NB / kSelThreads;
  const u32x4* gh = (const u32x4*)(h + (NB - kBins * (tid() + 1)));
  u32x4 hv[kBins / 4];
  uint32_t tot = 0, total;
#pragma unroll
  for (int i = 0; i < kBins / 4; ++i) {
    hv[i] = gh[i];
    tot += (hv[i][0] + hv[i][1]) + (hv[i][2] + hv[i][3]);
  }
  const uint32_t above = block_exclusive_scan(tot, lds, total);
  if (above < want && above + tot >= want) {
    uint32_t cum = above;
    bool done = false;
#pragma unroll
    for (int i = kBins - 1; i >= 0; --i) {
      const uint32_t c = hv[i >> 2][i & 3];
      if (!done && cum + c >= want) {
        pick[0] = (uint32_t)(NB - kBins * (tid() + 1) + i);
        pick[1] = want - cum;
        done = true;
      }
      cum += c;
    }
  }
  __syncthreads();
  const int bin = uniform((int)pick[0]);
  want = (uint32_t)uniform((int)pick[1]);
  __syncthreads();
  return bin;
}

// Every workgroup finds the bin that holds the K_eff-th largest score for
// itself (16 KB of counts from the L2: about what a launch of its own would
// take), then counts its candidates of that bin in kSubBins parts.
__global__ __launch_bounds__(kSelThreads) void select_refine(SelectArgs a) {
  __shared__ uint32_t lds[8], pick[2];
  __shared__ uint32_t lhist[kSubBins];
  const int bg = bid_y(), split = bid_x();
  if (uniform(a.state[bg].mode) != 2) return;
  uint32_t want = (uint32_t)uniform(a.state[bg].keff);
  int c0, c1;
  seq_range(a, bg, c0, c1);
  const int j0 = c0 + split * kCandChunk, j1 = min(j0 + kCandChunk, c1);
  if (j0 >= j1) return;  // never split 0: there are candidates
  const float* Pg = a.P + (size_t)bg * a.max_len;
  uint32_t bits[kPerThread];
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) bits[i] = __float_as_uint(Pg[min(j0 + tid() + i * kSelThreads, j1 - 1)]);
  for (int i = tid(); i < kSubBins; i += nthreads()) lhist[i] = 0u;
  uint32_t* gh = a.hist + (size_t)bg * (kHistBins + kSubBins);
  const int bin = find_bin<kHistBins>(gh, want, lds, pick);
  if (split == 0 && tid() == 0) {
    a.state[bg].bin = bin;
    a.state[bg].krem = (int32_t)want;
  }
  uint32_t lo, hi;
  int shift;
  bin_limits(bin, a.hist_top, lo, hi, shift);
#pragma unroll
  for (int i = 0; i < kPerThread; ++i)
    if (j0 + tid() + i * kSelThreads < j1 && bits[i] >= lo && bits[i] <= hi)
      atomicAdd(&lhist[(bits[i] - lo) >> shift], 1u);
  __syncthreads();
  for (int i = tid(); i < kSubBins; i += nthreads()) {
    const uint32_t v = lhist[i];
    if (v) atomicAdd(&gh[kHistBins + i], v);
  }
}

// The scores that can decide the threshold when it lies in part `sub` of `bin`,
// as bit patterns: that part's, and as far on each side as the re-score band of
// any of them reaches (2^-17 of the score; twice that here).
__device__ __forceinline__ void list_limits(int bin, int sub, uint32_t top, uint32_t& lo, uint32_t& hi) {
  uint32_t blo, bhi;
  int shift;
  bin_limits(bin, top, blo, bhi, shift);
  const uint32_t first = blo + ((uint32_t)sub << shift), last = first + ((1u << shift) - 1u);
  lo = __float_as_uint(__uint_as_float(first) * (1.0f - 2.f * kBandRel));
  hi = last >= 0x7f800000u || last < first ? 0xffffffffu : __float_as_uint(__uint_as_float(last) * (1.0f + 2.f * kBandRel));
  if (first >= 0x7f800000u) lo = first;  // not finite: no band
}

// Every workgroup finds the part of the bin that holds the threshold, lists its
// candidates next to it and counts those above.
__global__ __launch_bounds__(kSelThreads) void select_collect(SelectArgs a) {
  __shared__ uint32_t lds[8], pick[2];
  __shared__ uint2 buf[kCandChunk];
  __shared__ int nbuf, base;
  const int bg = bid_y(), split = bid_x();
  if (uniform(a.state[bg].mode) != 2) return;
  int c0, c1;
  seq_range(a, bg, c0, c1);
  const int j0 = c0 + split * kCandChunk, j1 = min(j0 + kCandChunk, c1);
  if (j0 >= j1) {
    if (tid() == 0) {
      a.counts[(size_t)bg * a.n_splits + split] = make_uint2(0u, 0u);
      a.band_above[(size_t)bg * a.n_splits + split] = 0u;
    }
    return;
  }
  const int bin = uniform(a.state[bg].bin);
  uint32_t want = (uint32_t)uniform(a.state[bg].krem);
  const float* Pg = a.P + (size_t)bg * a.max_len;
  uint32_t bits[kPerThread];
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) bits[i] = __float_as_uint(Pg[min(j0 + tid() + i * kSelThreads, j1 - 1)]);
  if (tid() == 0) nbuf = 0;
  const int sub = find_bin<kSubBins>(a.hist + (size_t)bg * (kHistBins + kSubBins) + kHistBins, want, lds, pick);
  uint32_t lo, hi;
  list_limits(bin, sub, a.hist_top, lo, hi);
  uint32_t above = 0;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    const int j = j0 + tid() + i * kSelThreads;
    if (j >= j1) continue;
    above += bits[i] > hi;
    if (bits[i] >= lo && bits[i] <= hi) buf[atomicAdd(&nbuf, 1)] = make_uint2(bits[i], (uint32_t)j);
  }
  uint32_t ta;
  block_exclusive_scan(above, lds, ta);  // its barriers also complete buf
  if (tid() == 0) {
    a.counts[(size_t)bg * a.n_splits + split] = make_uint2(ta, 0u);
    a.band_above[(size_t)bg * a.n_splits + split] = ta;
    if (split == 0) a.state[bg].sub = sub;
    base = nbuf ? atomicAdd(&a.list_n[bg], nbuf) : 0;
  }
  __syncthreads();
  for (int i = tid(); i < nbuf; i += nthreads())
    if (base + i < kListCap) a.list[(size_t)bg * kListCap + base + i] = buf[i];
}

// One workgroup per group: the K_eff-th largest score among those within the
// list's limits (a radix select in LDS, digits of 8 bits below the highest bit in
// which the limits differ: 10 bits, except in the end bins), then the exact
// counts per split and the members of the re-score band.  A group with more such
// candidates than the list holds (many equal scores) reads all its scores
// instead, kThrU a thread in flight.
constexpr int kThrThreads = 512;
constexpr int kThrBits = 8;
constexpr int kThrU = 8;
__global__ __launch_bounds__(kThrThreads) void select_threshold(SelectArgs a) {
  __shared__ uint2 list[kListCap];
  __shared__ uint32_t cnt[1 << kThrBits];
  __shared__ uint32_t lds[kThrThreads / 64];
  __shared__ uint32_t pick[2];
  __shared__ int nband;
  const int bg = bid_x();
  RadixState st = load_state(&a.state[bg]);
  if (st.mode != 2) return;
  int c0, c1;
  seq_range(a, bg, c0, c1);
  const float* Pg = a.P + (size_t)bg * a.max_len;
  uint2* counts = a.counts + (size_t)bg * a.n_splits;
  uint32_t* band_above = a.band_above + (size_t)bg * a.n_splits;
  const int n = uniform(a.list_n[bg]), lane = tid() & 63;
  const bool listed = n <= kListCap;
  uint32_t lo, hi;
  list_limits(st.bin, st.sub, a.hist_top, lo, hi);
  if (listed)
    for (int i = tid(); i < n; i += nthreads()) list[i] = a.list[(size_t)bg * kListCap + i];
  uint32_t above = 0, total;
  for (int s = tid(); s < a.n_splits; s += nthreads()) above += band_above[s];
  if (tid() == 0) nband = 0;
  block_exclusive_scan(above, lds, total);
  uint32_t want = (uint32_t)st.keff - total;
  // fn(score bits, token) for every candidate within the limits; whole waves
  // call it (in = false: nothing)
  auto each = [&](auto fn) {
    if (listed) {
      for (int i0 = 0; i0 < n; i0 += nthreads()) {
        const int i = i0 + tid();
        const uint2 e = i < n ? list[i] : make_uint2(0u, 0u);
        fn(i < n, e.x, (int)e.y);
      }
    } else {
      for (int j0 = c0; j0 < c1; j0 += kThrU * kThrThreads) {
        uint32_t bits[kThrU];
#pragma unroll
        for (int u = 0; u < kThrU; ++u) bits[u] = __float_as_uint(Pg[min(j0 + u * kThrThreads + tid(), c1 - 1)]);
#pragma unroll
        for (int u = 0; u < kThrU; ++u) {
          const int j = j0 + u * kThrThreads + tid();
          fn(j < c1 && bits[u] >= lo && bits[u] <= hi, bits[u], j);
        }
      }
    }
  };
  // largest first: digit 0 is the highest score's
  uint32_t prefix = 0;
  int shift = 32 - __builtin_clz(hi - lo);  // bits of hi - score still to decide
  while (shift > 0) {
    const int w = shift < kThrBits ? shift : kThrBits;
    const int below = shift - w;
    if (tid() < (1 << kThrBits)) cnt[tid()] = 0u;
    __syncthreads();
    each([&](bool in, uint32_t bits, int) {
      const uint32_t r = hi - bits;
      in = in && (shift == 32 || (r >> shift) == (prefix >> shift));
      const uint32_t d = (r >> below) & ((1u << w) - 1u);
      // equal scores of a wave count once for all
      const uint64_t m = __builtin_amdgcn_ballot_w64(in);
      if (m == 0) return;
      const int first = __builtin_ctzll(m);
      const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, first);
      const uint64_t same = __builtin_amdgcn_ballot_w64(in && d == d0);
      if (lane == first) atomicAdd(&cnt[d0], (uint32_t)__builtin_popcountll(same));
      if (in && d != d0) atomicAdd(&cnt[d], 1u);
    });
    __syncthreads();
    const uint32_t mine = tid() < (1 << kThrBits) ? cnt[tid()] : 0u;
    const uint32_t before = block_exclusive_scan(mine, lds, total);
    if (before < want && before + mine >= want) {
      pick[0] = (uint32_t)tid();
      pick[1] = before;
    }
    __syncthreads();
    prefix |= pick[0] << below;
    want -= pick[1];
    shift = below;
    __syncthreads();
  }
  const uint32_t tau = hi - prefix;
  uint32_t blo, bhi;
  band_limits(tau, blo, bhi);
  each([&](bool in, uint32_t bits, int j) {
    const int s = (j - c0) / kCandChunk;
    const bool gt = in && bits > tau, eq = in && bits == tau, up = in && bits > bhi;
    if (listed) {
      if (gt) atomicAdd(&counts[s].x, 1u);
      if (eq) atomicAdd(&counts[s].y, 1u);
      if (up) atomicAdd(&band_above[s], 1u);
    } else {
      // 64 consecutive candidates, a multiple of 64 from the first: one split
      const uint64_t mg = __builtin_amdgcn_ballot_w64(gt), me = __builtin_amdgcn_ballot_w64(eq),
                     mu = __builtin_amdgcn_ballot_w64(up);
      if (lane == 0) {
        if (mg) atomicAdd(&counts[s].x, (uint32_t)__builtin_popcountll(mg));
        if (me) atomicAdd(&counts[s].y, (uint32_t)__builtin_popcountll(me));
        if (mu) atomicAdd(&band_above[s], (uint32_t)__builtin_popcountll(mu));
      }
    }
    const bool member = in && bits >= blo && bits <= bhi;
    const uint64_t mm = __builtin_amdgcn_ballot_w64(member);
    if (mm == 0) return;
    int base = 0;
    if (lane == 0) base = atomicAdd(&nband, (int)__builtin_popcountll(mm));
    base = uniform(base);
    const int m = base + (int)__builtin_popcountll(mm & ((1ull << lane) - 1ull));
    if (member && m < kBandCap) a.band_idx[(size_t)bg * kBandCap + m] = j;
  });
  __syncthreads();
  if (tid() == 0) {
    a.band_n[bg] = nband;
    st.prefix = tau;
    st.krem = (int32_t)want;
    a.state[bg] = st;
  }
}

// ============================================================ fp64 re-score of the band
// Every candidate in the band gets its pooled score again in fp64 (Eq. 1-3
// with exact products of the bf16 / fp32 inputs, fp64 exponentials and the
// rows' fp64 normalisers), so the selection near the threshold does not rest
// on the fp32 logits of the score passes.  band_rescore forms the summed
// attention A of every key in the members' pooling windows, once per key:
// with the members sorted by token, member m owns the keys of its window
// past the previous member's window.  band_decide then pools, ranks and
// decides.
struct BandArgs {
  const void* q;          // [n_seq][Hq][w][D]
  const void* k;          // [n_seq][Hkv][max_len][D]
  const int32_t* lengths;
  const double2* rowz;    // [groups][rows_pad]
  const RadixState* state;
  const int32_t* band_n;
  const int32_t* band_idx;
  double* A64;            // [groups][max_len] fp64 A of the window keys
  double* band_p;         // [groups][kBandCap] fp64 pooled scores of the members
  float* pooled_out;      // optional debug copy: the members' re-scored values
  float* P;               // [groups][max_len]
  uint2* counts;          // [groups][n_splits]
  const uint32_t* band_above;
  RadixState* state_w;
  int Hq, Hkv, G, w, D, max_len, sink, recent, pool_kernel, pool, rows, rows_pad, n_splits, in_f32;
  int band_wgs;           // workgroups per group of band_rescore (work items strided over them)
  int rows_per_pass;      // score rows per band_rescore pass (kBandThreads / query-dim slices)
  double scale2;          // sm_scale * log2(e) in fp64
};

// Members ranked by token index (the members are distinct): rank[i] = how
// many members precede member i.  One pass over the list per member, no
// barriers; nb <= kBandCap.
__device__ __forceinline__ int token_rank(const int32_t* s, int nb, int i) {
  const int32_t x = s[i];
  int r = 0;
#pragma unroll 8
  for (int u = 0; u < nb; ++u) r += s[u] < x;
  return r;
}

// The keys whose fp64 A the band needs, in token order: with the members
// sorted by token, member m owns the keys of its pooling window (within the
// candidates) that lie past the previous member's window.  Fills first[m] =
// index of member m's first key in that order (first[nb] = the key count) and
// tok[m] = the sorted members; returns the key count.  Every thread calls it.
__device__ int band_keys(const int32_t* members, int nb, int half, int c0, int c1, int32_t* tok, int32_t* first,
                         uint32_t* scan_lds) {
  for (int i = tid(); i < nb; i += nthreads()) tok[token_rank(members, nb, i)] = members[i];
  __syncthreads();
  // owned key counts, then an exclusive scan over the (<= kBandCap) members
  uint32_t total = 0;
  for (int base = 0; base < nb; base += nthreads()) {
    const int m = base + tid();
    uint32_t cnt = 0;
    if (m < nb) {
      const int j = tok[m];
      int t0 = max(j - half, c0);
      if (m > 0) t0 = max(t0, tok[m - 1] + half + 1);
      const int t1 = min(j + half, c1 - 1);
      cnt = t1 >= t0 ? (uint32_t)(t1 - t0 + 1) : 0u;
    }
    uint32_t part;
    const uint32_t ex = block_exclusive_scan(cnt, scan_lds, part);
    if (m < nb) first[m] = (int)(total + ex);
    total += part;
  }
  if (tid() == 0) first[nb] = (int)total;
  __syncthreads();
  return (int)total;
}

// Token of key x in the band's key order (first[] from band_keys).
__device__ __forceinline__ int band_key_token(const int32_t* tok, const int32_t* first, int nb, int half, int c0,
                                              int x) {
  int lo = 0, hi = nb - 1;  // the member m with first[m] <= x < first[m+1]
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= x) lo = mid; else hi = mid - 1;
  }
  const int j = tok[lo];
  int t0 = max(j - half, c0);
  if (lo > 0) t0 = max(t0, tok[lo - 1] + half + 1);
  return t0 + (x - first[lo]);
}

constexpr int kBandKeys = 4;       // keys per block (staged in LDS together)
constexpr int kBandThreads = 512;  // rows x slices of the query dims
constexpr int kBandKeyCap = 1024;  // band keys per group; more keeps the fp32 selection
constexpr int kBandMaxPass = 4;    // row passes of a key block (rows_pad / rows per pass)
// Workgroup of kBandThreads threads: thread = (score row, slice of SLICES of the
// query dims), rows taken kBandThreads / SLICES at a time.  Each block of
// kBandKeys keys is staged in LDS with one load round trip; the thread's
// query slice is loaded once per block and row pass.
template <typename In, int D, int SLICES>
__device__ void band_rescore_body(const BandArgs& a, int bg, int b, int g, int nkeys, const int32_t* tok,
                                  const int32_t* first, int nb, int half, int c0, int L, unsigned char* kl,
                                  double (*red)[kBandKeys]) {
  constexpr int kEl = 16 / (int)sizeof(In);         // elements per 16-byte chunk
  constexpr int kRowChunks = D / kEl;
  constexpr int CH = kRowChunks / SLICES;           // chunks per slice
  constexpr int RPP = kBandThreads / SLICES;        // rows per pass
  const int sl = tid() % SLICES;
  const int we = min(a.w, L);
  const In* qg = (const In*)a.q + ((size_t)b * a.Hq + (size_t)g * a.G) * a.w * D;
  const size_t krow0 = ((size_t)b * a.Hkv + g) * (size_t)a.max_len;
  const int lane = tid() & 63, wave = tid() >> 6;
  const int npass = (a.rows_pad + RPP - 1) / RPP;
  const int nblk = (nkeys + kBandKeys - 1) / kBandKeys;
  // work items (key block, row pass), strided over the group's workgroups
  for (int item = bid_x(); item < nblk * npass; item += a.band_wgs) {
    const int x0 = (item / npass) * kBandKeys, r0 = (item % npass) * RPP;
    const int nk = min(kBandKeys, nkeys - x0);
    // stage the block's key rows (chunk c of key e at kl + (e * kRowChunks + c) * 16)
    for (int i = tid(); i < nk * kRowChunks; i += nthreads()) {
      const int e = i / kRowChunks, c = i % kRowChunks;
      const int t = band_key_token(tok, first, nb, half, c0, x0 + e);
      if (debug_check(t >= c0 && t < L - a.recent, kDbgBand))
        *((u32x4*)kl + i) = *((const u32x4*)((const In*)a.k + (krow0 + t) * D) + c);
    }
    int kt[kBandKeys];
#pragma unroll
    for (int e = 0; e < kBandKeys; ++e) kt[e] = e < nk ? band_key_token(tok, first, nb, half, c0, x0 + e) : 0;
    // this thread's row and its query slice
    const int rho = r0 + tid() / SLICES;
    const int ii = rho % a.w;
    const bool rval = rho < a.rows && ii >= a.w - we;
    const int rpos = L - a.w + ii;
    const double2 nz = rval ? a.rowz[(size_t)bg * a.rows_pad + rho] : make_double2(0.0, 0.0);
    const bool live = rval && nz.y > 0.0;
    u32x4 qv[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c)
      qv[c] = live ? *((const u32x4*)(qg + (size_t)rho * D) + sl * CH + c) : u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kBandKeys; ++e) {
      double s = 0.0;
      if (e < nk) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const u32x4 kv = *((const u32x4*)kl + e * kRowChunks + sl * CH + c);
          if constexpr (sizeof(In) == 2) {
            // a bf16 x bf16 product is exact in fp32; the sums run in fp64
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              s += (double)(bf16_bits_to_f32(qv[c][i] & 0xffffu) * bf16_bits_to_f32(kv[i] & 0xffffu));
              s += (double)(bf16_bits_to_f32(qv[c][i] >> 16) * bf16_bits_to_f32(kv[i] >> 16));
            }
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) s = fma((double)__uint_as_float(qv[c][i]), (double)__uint_as_float(kv[i]), s);
          }
        }
      }
      // the row's dot product: sum of its slices (adjacent lanes)
#pragma unroll
      for (int o = 1; o < SLICES; o <<= 1) s += __shfl_xor(s, o);
      double wv = 0.0;
      if (sl == 0 && live && e < nk && kt[e] <= rpos) wv = exp2(s * a.scale2 - nz.x) / nz.y;
      // summed over this pass's rows (fixed order)
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) wv += __shfl_xor(wv, o);
      if (lane == 0) red[wave][e] = wv;
    }
    __syncthreads();
    if (tid() < nk) {
      double s = 0.0;
      for (int w2 = 0; w2 < kBandThreads / 64; ++w2) s += red[w2][tid()];
      a.A64[((size_t)bg * kBandKeyCap + x0 + tid()) * kBandMaxPass + item % npass] = s;
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kBandThreads) void band_rescore(BandArgs a) {
  __shared__ int32_t mem[kBandCap];
  __shared__ int32_t tok[kBandCap];
  __shared__ int32_t first[kBandCap + 1];
  __shared__ uint32_t scan_lds[kBandThreads / 64];
  __shared__ double red[kBandThreads / 64][kBandKeys];
  __shared__ __align__(16) unsigned char kl[kBandKeys * 576 * 2];
  const int bg = bid_y(), b = bg / a.Hkv, g = bg % a.Hkv;
  const RadixState st = load_state(&a.state[bg]);
  if (st.mode != 2) return;
  const int nb = uniform(a.band_n[bg]);
  if (nb > kBandCap) return;  // too many: the fp32 selection stands
  // at most pool_kernel keys per member, so at most this many work items:
  // workgroups past them have nothing to do
  if (bid_x() >= (nb * a.pool_kernel + kBandKeys - 1) / kBandKeys * kBandMaxPass) return;
  int L = uniform(a.lengths[b]);
  L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
  const int c0 = a.sink, c1 = L - a.recent, half = a.pool_kernel / 2;
  for (int i = tid(); i < nb; i += nthreads()) mem[i] = a.band_idx[(size_t)bg * kBandCap + i];
  __syncthreads();
  const int nkeys = band_keys(mem, nb, half, c0, c1, tok, first, scan_lds);
  if (nkeys > kBandKeyCap) return;
  // threads per score row (rows_pad <= 256, or 128 for fp32 inputs)
  if (a.in_f32) {
    if (a.D == 64) band_rescore_body<float, 64, 8>(a, bg, b, g, nkeys, tok, first, nb, half, c0, L, kl, red);
    else band_rescore_body<float, 128, 8>(a, bg, b, g, nkeys, tok, first, nb, half, c0, L, kl, red);
  } else {
    if (a.D == 64) band_rescore_body<uint16_t, 64, 4>(a, bg, b, g, nkeys, tok, first, nb, half, c0, L, kl, red);
    else if (a.D == 128) band_rescore_body<uint16_t, 128, 4>(a, bg, b, g, nkeys, tok, first, nb, half, c0, L, kl, red);
    else band_rescore_body<uint16_t, 576, 8>(a, bg, b, g, nkeys, tok, first, nb, half, c0, L, kl, red);
  }
}

// One workgroup per group: pool each member from the fp64 A of its window
// (Eq. 2), rank the members by (fp64 pooled score descending, token index
// ascending), keep the first K_eff - (candidates above the band), and
// rewrite the members' P so that the ordered compaction keeps exactly the
// candidates above the band and the kept members: P > hi for kept ones, 0
// for the others, threshold hi, no ties.
__global__ __launch_bounds__(kSelThreads) void band_decide(BandArgs a) {
  __shared__ double sp[kBandCap];
  __shared__ int32_t sj[kBandCap];
  __shared__ int32_t tok[kBandCap];
  __shared__ int32_t first[kBandCap + 1];
  __shared__ double key_A[kBandKeyCap];
  __shared__ uint32_t lds[8];
  const int bg = bid_x();
  RadixState st = load_state(&a.state[bg]);
  if (st.mode != 2) return;
  const int nb = uniform(a.band_n[bg]);
  if (nb > kBandCap) return;
  const int b = bg / a.Hkv;
  int L = uniform(a.lengths[b]);
  L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
  const int c0 = a.sink, c1 = L - a.recent, half = a.pool_kernel / 2;
  for (int i = tid(); i < nb; i += nthreads()) sj[i] = a.band_idx[(size_t)bg * kBandCap + i];
  __syncthreads();
  const int nkeys = band_keys(sj, nb, half, c0, c1, tok, first, lds);
  if (nkeys > kBandKeyCap) return;  // as band_rescore
  // the keys' A from their row passes, all loads in flight together (a thread
  // that gathered a member's window from memory waited for each of its keys)
  {
    const double* Ag = a.A64 + (size_t)bg * kBandKeyCap * kBandMaxPass;
    const int npass = (a.rows_pad + a.rows_per_pass - 1) / a.rows_per_pass;
    for (int x = tid(); x < nkeys; x += nthreads()) {
      double part[kBandMaxPass], At = 0.0;
#pragma unroll
      for (int pp = 0; pp < kBandMaxPass; ++pp) part[pp] = pp < npass ? Ag[(size_t)x * kBandMaxPass + pp] : 0.0;
#pragma unroll
      for (int pp = 0; pp < kBandMaxPass; ++pp) At += part[pp];
      key_A[x] = At;
    }
  }
  uint32_t lo, hi;
  band_limits(st.prefix, lo, hi);
  // candidates above the band (all kept)
  uint32_t above = 0;
  for (int s = tid(); s < a.n_splits; s += nthreads()) above += a.band_above[(size_t)bg * a.n_splits + s];
  uint32_t n_above;
  block_exclusive_scan(above, lds, n_above);
  const int need = st.keff - (int)n_above;  // in [1, nb] (tau itself is a member)
  if (need < 0 || need > nb) return;         // not for finite scores; the fp32 selection stands
  for (int i = tid(); i < nb; i += nthreads()) {
    const int j = sj[i];
    const int t0 = max(j - half, c0), t1 = min(j + half, c1 - 1);
    double pooled = a.pool == SNAP_POOL_MAX ? -1.0 : 0.0;
    for (int t = t0; t <= t1; ++t) {
      // key index of t: the first member (by token) whose window holds t
      // owns it (see band_keys)
      int lo = 0, hi2 = nb - 1;
      while (lo < hi2) {
        const int mid = (lo + hi2) >> 1;
        if (tok[mid] >= t - half) hi2 = mid; else lo = mid + 1;
      }
      int k0 = max(tok[lo] - half, c0);
      if (lo > 0) k0 = max(k0, tok[lo - 1] + half + 1);
      const double At = key_A[first[lo] + (t - k0)];
      if (a.pool == SNAP_POOL_MAX)
        pooled = At > pooled ? At : pooled;
      else
        pooled += At;
    }
    if (a.pool != SNAP_POOL_MAX) pooled /= (double)a.pool_kernel;
    sp[i] = pooled;
    a.band_p[(size_t)bg * kBandCap + i] = pooled;
    if (a.pooled_out) a.pooled_out[(size_t)bg * a.max_len + j] = (float)pooled;
  }
  __syncthreads();
  // rank by (score desc, token asc): kept when fewer than `need` come first
  float* Pg = a.P + (size_t)bg * a.max_len;
  for (int i = tid(); i < nb; i += nthreads()) {
    const double pi = sp[i];
    const int ji = sj[i];
    int r = 0;
#pragma unroll 4
    for (int u = 0; u < nb; ++u) r += sp[u] > pi || (sp[u] == pi && sj[u] < ji);
    tok[i] = r < need;
  }
  __syncthreads();
  // per-split counts of what the compaction keeps: the candidates above the
  // band and the kept members
  uint2* counts = a.counts + (size_t)bg * a.n_splits;
  for (int s = tid(); s < a.n_splits; s += nthreads())
    counts[s] = make_uint2(a.band_above[(size_t)bg * a.n_splits + s], 0u);
  __syncthreads();
  for (int i = tid(); i < nb; i += nthreads())
    if (tok[i]) atomicAdd(&counts[(sj[i] - c0) / kCandChunk].x, 1u);
  for (int i = tid(); i < nb; i += nthreads()) Pg[sj[i]] = __uint_as_float(tok[i] ? hi + 1u : 0u);
  if (tid() == 0) {
    st.prefix = hi;
    st.krem = 0;
    a.state_w[bg] = st;
  }
}

// Ordered compaction: a candidate is kept when P > t, or P == t and it is among
// the krem lowest-index candidates equal to t, and goes to place (candidates
// above t before it) + min(candidates equal to t before it, krem): token order.
// A wave takes 512 consecutive candidates, 64 a load, and counts them by ballot,
// so the workgroup meets once (with 8 candidates in a row per thread, 32-byte
// strides, four block scans and a serial sum over the splits before it, 19 us
// for 64 groups of up to 128k candidates).
__global__ __launch_bounds__(kSelThreads) void select_write(SelectArgs a) {
  constexpr int kWaves = kSelThreads / 64, kWaveCands = kCandChunk / kWaves;
  __shared__ uint2 wcnt[kWaves], before[kWaves];
  const int bg = bid_y(), split = bid_x();
  const int lane = tid() & 63, wave = uniform(tid() >> 6);
  int c0, c1;
  seq_range(a, bg, c0, c1);
  const int j0 = c0 + split * kCandChunk, j1 = min(j0 + kCandChunk, c1);
  if (j0 >= j1) return;
  const float* Pg = a.P + (size_t)bg * a.max_len;
  const int jw = j0 + wave * kWaveCands + lane;
  uint32_t bits[kWaveCands / 64];
#pragma unroll
  for (int i = 0; i < kWaveCands / 64; ++i) bits[i] = __float_as_uint(Pg[min(jw + 64 * i, j1 - 1)]);
  uint32_t gb = 0, eb = 0;  // candidates above / equal in the splits before this one
  for (int t = tid(); t < split; t += nthreads()) {
    const uint2 c = a.counts[(size_t)bg * a.n_splits + t];
    gb += c.x;
    eb += c.y;
  }
  const RadixState st = load_state(&a.state[bg]);
  if (st.mode == 0) return;
  int32_t* sg = a.sel + (size_t)bg * a.topk;
  if (st.mode == 1) {
    for (int j = j0 + tid(); j < j1; j += nthreads()) sg[j - c0] = j;
    return;
  }
  uint64_t gt[kWaveCands / 64], eq[kWaveCands / 64];
  uint32_t ng = 0, ne = 0;
#pragma unroll
  for (int i = 0; i < kWaveCands / 64; ++i) {
    const bool in = jw + 64 * i < j1;
    gt[i] = __builtin_amdgcn_ballot_w64(in && bits[i] > st.prefix);
    eq[i] = __builtin_amdgcn_ballot_w64(in && bits[i] == st.prefix);
    ng += (uint32_t)__builtin_popcountll(gt[i]);
    ne += (uint32_t)__builtin_popcountll(eq[i]);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    gb += (uint32_t)__shfl_xor((int)gb, o);
    eb += (uint32_t)__shfl_xor((int)eb, o);
  }
  if (lane == 0) {
    wcnt[wave] = make_uint2(ng, ne);
    before[wave] = make_uint2(gb, eb);
  }
  __syncthreads();
  uint32_t G = 0, E = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    G += before[w].x + (w < wave ? wcnt[w].x : 0u);
    E += before[w].y + (w < wave ? wcnt[w].y : 0u);
  }
  const uint32_t krem = (uint32_t)st.krem, keff = (uint32_t)st.keff;
  const uint64_t lower = (1ull << lane) - 1ull;
#pragma unroll
  for (int i = 0; i < kWaveCands / 64; ++i) {
    const uint32_t g = G + (uint32_t)__builtin_popcountll(gt[i] & lower);
    const uint32_t e = E + (uint32_t)__builtin_popcountll(eq[i] & lower);
    const bool keep = (gt[i] >> lane & 1) || ((eq[i] >> lane & 1) && e < krem);
    const uint32_t pos = g + (e < krem ? e : krem);
    // never past the group's K slots
    if (keep && debug_check(pos < keff, kDbgSelWrite) && pos < keff) sg[pos] = jw + 64 * i;
    G += (uint32_t)__builtin_popcountll(gt[i]);
    E += (uint32_t)__builtin_popcountll(eq[i]);
  }
}

// ============================================================ assemble
struct AssembleArgs {
  const void* k;       // [n_seq][Hkv][max_len][dk]
  const void* v;       // or NULL
  void* ck;            // [n_slots][Hkv][B][dk]
  void* cv;
  float* k_scale;      // [n_slots][Hkv], fp8 only (written in SNAP_FP8_SCALES_AMAX mode)
  float* v_scale;
  const int32_t* slot_ids;
  const int32_t* lengths;
  const int32_t* sel;  // [groups][topk]
  const RadixState* state;
  int32_t* sel_out;    // optional [groups][topk]
  int32_t* pos;
  int32_t* n_topk;
  float2* amax;        // [groups][n_rowblocks] (K, V) amax of the kept rows, or NULL
  int Hkv, max_len, sink, recent, topk, dk, dv, n_slots, rows_per_block, n_rowblocks;
};

constexpr int kAsmRows = 64;  // cache rows per assemble workgroup
constexpr int kAsmU = 8;      // row pieces a thread has in flight

// First ring token l0 = max(L - r, s) and ring_base = (l0 - s) mod r, the
// ring row of token l0 counted from s (one division per thread, not per row).
struct RingMap {
  int l0, base;
};
__device__ __forceinline__ RingMap ring_map(int L, int s, int r) {
  const int l0 = L - r > s ? L - r : s;
  return RingMap{l0, (l0 - s) % r};
}

// Source token of cache row `row` (or -1 for a zero padding row).
__device__ __forceinline__ int row_source(int row, int L, int s, int r, int keff, const int32_t* sel,
                                          RingMap rm) {
  if (row < s) return row < L ? row : -1;
  if (row < s + r) {
    // token l0 + ((row - s) - base) mod r, with both terms in [0, r)
    int off = (row - s) - rm.base;
    if (off < 0) off += r;
    int t = rm.l0 + off;
    return t < L ? t : -1;
  }
  int m = row - s - r;
  if (m >= keff) return -1;
  const int t = sel[m];
  return debug_check(t >= s && t < L - r, kDbgAsmSource) ? t : -1;
}

// x / scale rounded once to fp32, as an IEEE division gives it, from a
// correctly rounded reciprocal inv = 1 / scale and one fused correction:
// q0 = x * inv, r = x - q0 * scale (exact by fma), q = q0 + r * inv (Markstein's
// theorem: correctly rounded when neither r nor the quotient leaves the
// normal range).  Where q0 is 0 or not finite it is kept: the E4M3 code of a
// zero, of a quotient too small for a non-zero code, or of a saturated one
// does not depend on the correction.  Checked on the host against the
// division for every finite bf16 x over 353 scales (amax / 448 of 256 bf16
// maxima, 64 random magnitudes, powers of two and their neighbours):
// identical E4M3 codes.
__device__ __forceinline__ float div_by_scale(float x, float scale, float inv) {
  const float q0 = x * inv;
  const float r = __builtin_fmaf(-q0, scale, x);
  const float q = __builtin_fmaf(r, inv, q0);
  return (q0 == 0.f || !__builtin_isfinite(q0)) ? q0 : q;
}

// 8 elements of an input row in raw form: 16 bytes of bf16 or 32 of fp32
// (zeros for a NULL source, a padding row).  The gather reads each prompt row
// and writes each cache row once: both carry the non-temporal (streaming)
// hint (measured 1-2% off the compress call).
template <typename In>
struct Raw8In {
  u32x4 w[sizeof(In) / 2];
};
template <typename In>
__device__ __forceinline__ Raw8In<In> load8(const In* src) {
  Raw8In<In> x;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(In) / 2); ++i)
    x.w[i] = src ? __builtin_nontemporal_load((const u32x4*)src + i) : u32x4{0u, 0u, 0u, 0u};
  return x;
}
// ... stored into the cache, quantised to E4M3 codes of x / scale when the
// cache is fp8 (the correctly rounded quotient, then the conversion
// instruction: e4m3x4_hw).
template <typename In, typename Out>
__device__ __forceinline__ void store8(const Raw8In<In>& x, Out* dst, float scale, float inv) {
  if constexpr (sizeof(Out) == 1) {
    float f[8];
    if constexpr (sizeof(In) == 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f[2 * i] = bf16_bits_to_f32(x.w[0][i] & 0xffffu);
        f[2 * i + 1] = bf16_bits_to_f32(x.w[0][i] >> 16);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = __uint_as_float(x.w[i >> 2][i & 3]);
    }
    float qv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) qv[i] = div_by_scale(f[i], scale, inv);
    u32x2 o;
    o[0] = e4m3x4_hw(qv[0], qv[1], qv[2], qv[3]);
    o[1] = e4m3x4_hw(qv[4], qv[5], qv[6], qv[7]);
    __builtin_nontemporal_store(o, (u32x2*)dst);
  } else {
#pragma unroll
    for (int i = 0; i < (int)(sizeof(In) / 2); ++i) __builtin_nontemporal_store(x.w[i], (u32x4*)dst + i);
  }
}

// Largest magnitude of one workgroup's values (LDS across the waves); every
// thread gets it.
__device__ __forceinline__ uint32_t block_max_u32(uint32_t v, uint32_t* lds) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
  __syncthreads();
  if ((tid() & 63) == 0) lds[tid() >> 6] = v;
  __syncthreads();
  v = 0;
  for (int w = 0; w < (int)(nthreads() >> 6); ++w) v = max(v, lds[w]);
  return v;
}

// fp8 scales from the data (SNAP_FP8_SCALES_AMAX): per (group, block of
// rows_per_block cache rows) the largest |K| and |V| among the rows the block
// keeps; padding rows add nothing.  bf16 magnitudes order like their bit
// patterns, so the maxima are taken on the 15 low bits.
__global__ __launch_bounds__(256) void fp8_amax(AssembleArgs a) {
  __shared__ uint32_t lds[4];
  const int bg = bid_y(), b = bg / a.Hkv, g = bg % a.Hkv;
  const int slot = uniform(a.slot_ids[b]);
  if (slot < 0 || slot >= a.n_slots) return;
  const int s = a.sink, r = a.recent, B = s + r + a.topk;
  int L = uniform(a.lengths[b]);
  L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
  const int keff = a.topk == 0 ? 0 : uniform(a.state[bg].keff);
  const int32_t* sg = a.sel + (size_t)bg * a.topk;
  const int row0 = bid_x() * a.rows_per_block;
  const int row1 = min(row0 + a.rows_per_block, B);
  const size_t in_row0 = ((size_t)b * a.Hkv + g) * (size_t)a.max_len;
  const int kp = a.dk / 8, vp = a.v ? a.dv / 8 : 0, per_row = kp + vp;
  const int items = (row1 - row0) * per_row;
  const RingMap rm = ring_map(L, s, r);
  uint32_t mk = 0, mv = 0;
  // as in assemble: kAsmU pieces a thread, all their reads in flight together
  const int step_r = nthreads() / per_row, step_p = nthreads() % per_row;
  int cur_r = tid() / per_row, cur_p = tid() % per_row;
  for (int it0 = tid(); it0 < items; it0 += kAsmU * nthreads()) {
    int piece_u[kAsmU], src_t[kAsmU];
#pragma unroll
    for (int u = 0; u < kAsmU; ++u) {
      piece_u[u] = cur_p;
      src_t[u] = it0 + u * nthreads() < items ? row_source(row0 + cur_r, L, s, r, keff, sg, rm) : -1;
      cur_r += step_r;
      cur_p += step_p;
      if (cur_p >= per_row) {
        cur_p -= per_row;
        ++cur_r;
      }
    }
    u32x4 x[kAsmU];
#pragma unroll
    for (int u = 0; u < kAsmU; ++u) {
      const int piece = piece_u[u], t = src_t[u];
      x[u] = u32x4{0u, 0u, 0u, 0u};
      if (t >= 0)
        x[u] = piece < kp ? *((const u32x4*)((const uint16_t*)a.k + (in_row0 + t) * a.dk) + piece)
                          : *((const u32x4*)((const uint16_t*)a.v + (in_row0 + t) * a.dv) + (piece - kp));
    }
#pragma unroll
    for (int u = 0; u < kAsmU; ++u) {
      uint32_t m = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) m = max(m, max(x[u][i] & 0x7fffu, (x[u][i] >> 16) & 0x7fffu));
      if (piece_u[u] < kp)
        mk = max(mk, m);
      else
        mv = max(mv, m);
    }
  }
  mk = block_max_u32(mk, lds);
  mv = block_max_u32(mv, lds);
  if (tid() == 0)
    a.amax[(size_t)bg * a.n_rowblocks + bid_x()] = make_float2(bf16_bits_to_f32(mk), bf16_bits_to_f32(mv));
}

// Each workgroup rewrites rows_per_block cache rows of one (sequence, KV
// head); threads walk (row, 8-element piece) pairs so every lane copies, kAsmU
// pairs at a time: their selected-index reads, then their row reads, are all
// issued before the first store (two memory round trips per kAsmU pieces).
template <typename In, typename Out>
__global__ __launch_bounds__(256) void assemble(AssembleArgs a) {
  const int bg = bid_y(), b = bg / a.Hkv, g = bg % a.Hkv;
  const int slot = uniform(a.slot_ids[b]);
  const int s = a.sink, r = a.recent, B = s + r + a.topk;
  int L = uniform(a.lengths[b]);
  L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
  const int keff = a.topk == 0 ? 0 : uniform(a.state[bg].keff);  // no selection ran when topk = 0
  const int32_t* sg = a.sel + (size_t)bg * a.topk;
  const int row0 = bid_x() * a.rows_per_block;
  const int row1 = min(row0 + a.rows_per_block, B);

  if (a.sel_out) {
    for (int m = row0 + tid(); m < row1; m += nthreads()) {
      int mm = m - s - r;
      if (mm >= 0) a.sel_out[(size_t)bg * a.topk + mm] = mm < keff ? sg[mm] : -1;
    }
  }
  if (slot < 0 || slot >= a.n_slots) return;
  if (bid_x() == 0 && g == 0 && tid() == 0) {
    a.pos[slot] = L;
    a.n_topk[slot] = keff;
  }
  const size_t in_row0 = ((size_t)b * a.Hkv + g) * (size_t)a.max_len;
  const size_t out_row0 = ((size_t)slot * a.Hkv + g) * (size_t)B;
  float ks = 1.f, vs = 1.f;
  if constexpr (sizeof(Out) == 1) {
    if (a.amax) {
      // scales from the group's amax over every row block: amax / 448, or 1
      // when every kept value is zero; block 0 records them for decoding
      __shared__ uint32_t lds[4];
      uint32_t mk = 0, mv = 0;
      for (int i = tid(); i < a.n_rowblocks; i += nthreads()) {
        const float2 m = a.amax[(size_t)bg * a.n_rowblocks + i];
        mk = max(mk, __float_as_uint(m.x));
        mv = max(mv, __float_as_uint(m.y));
      }
      const float ak = __uint_as_float(block_max_u32(mk, lds));
      const float av = __uint_as_float(block_max_u32(mv, lds));
      ks = ak > 0.f ? ak / 448.f : 1.f;
      vs = av > 0.f ? av / 448.f : 1.f;
      if (bid_x() == 0 && tid() == 0) {
        a.k_scale[(size_t)slot * a.Hkv + g] = ks;
        if (a.v) a.v_scale[(size_t)slot * a.Hkv + g] = vs;
      }
    } else {
      ks = a.k_scale[(size_t)slot * a.Hkv + g];
      if (a.v) vs = a.v_scale[(size_t)slot * a.Hkv + g];
    }
  }
  const float kinv = 1.0f / ks, vinv = 1.0f / vs;
  const RingMap rm = ring_map(L, s, r);
  const int kp = a.dk / 8, vp = a.v ? a.dv / 8 : 0, per_row = kp + vp;
  const int items = (row1 - row0) * per_row;
  // item it = row * per_row + piece; this thread's items advance by
  // nthreads(), i.e. by (step_r rows, step_p pieces) with a carry, so the
  // division runs once per thread
  const int step_r = nthreads() / per_row, step_p = nthreads() % per_row;
  int cur_r = tid() / per_row, cur_p = tid() % per_row;
  for (int it0 = tid(); it0 < items; it0 += kAsmU * nthreads()) {
    int row_u[kAsmU], piece_u[kAsmU], src_t[kAsmU];
#pragma unroll
    for (int u = 0; u < kAsmU; ++u) {
      const int it = it0 + u * nthreads();
      row_u[u] = row0 + cur_r;
      piece_u[u] = cur_p;
      cur_r += step_r;
      cur_p += step_p;
      if (cur_p >= per_row) {
        cur_p -= per_row;
        ++cur_r;
      }
      src_t[u] = it < items ? row_source(row_u[u], L, s, r, keff, sg, rm) : -1;
    }
    Raw8In<In> x[kAsmU];
#pragma unroll
    for (int u = 0; u < kAsmU; ++u) {
      const int it = it0 + u * nthreads();
      const int piece = piece_u[u], t = src_t[u];
      const In* src = nullptr;
      if (it < items && t >= 0)
        src = piece < kp ? (const In*)a.k + (in_row0 + t) * a.dk + 8 * piece
                         : (const In*)a.v + (in_row0 + t) * a.dv + 8 * (piece - kp);
      x[u] = load8<In>(src);
    }
#pragma unroll
    for (int u = 0; u < kAsmU; ++u) {
      const int it = it0 + u * nthreads();
      if (it >= items) break;
      const int row = row_u[u], piece = piece_u[u];
      if (piece < kp)
        store8<In, Out>(x[u], (Out*)a.ck + (out_row0 + row) * a.dk + 8 * piece, ks, kinv);
      else
        store8<In, Out>(x[u], (Out*)a.cv + (out_row0 + row) * a.dv + 8 * (piece - kp), vs, vinv);
    }
  }
}

// ============================================================ host side
static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// scale * log2(e) as hi + lo: hi the fp32 value rounded toward zero, lo the
// rest, strictly positive (a tiny positive value when hi is exact, where it
// changes no finite product): a masked -inf product times lo stays -inf.
void split_scale2(float scale, float& hi, float& lo) {
  const double x = (double)scale * 1.4426950408889634074;
  float h = (float)x;
  if ((double)h > x) h = nextafterf(h, 0.f);
  const float l = (float)(x - (double)h);
  hi = h;
  lo = l > 0.f ? l : 1e-30f;
}

SNAP_DEBUG_READER(debug_flags_compress)

Geometry compress_geometry(const snap_params& p, int n_seq, int max_len) {
  Geometry g{};
  int G = p.n_q_heads / p.n_kv_heads;
  g.rows = G * p.obs_window;
  g.rows_pad = (g.rows + 31) / 32 * 32;
  int groups = n_seq * p.n_kv_heads;
  // Key chunks: enough workgroups to cover the 256 CUs several times, but each
  // chunk several keys per score row, so that its keys outweigh the query
  // fragments every workgroup loads first.  The 256-row latent shape (a query
  // block of 295 KB) is fastest at 4096-key chunks.  64- and 128-wide keys:
  // prompts of a batch differ in length, so a batch wants many short chunks, or
  // CUs wait for the longest prompt's (8 ragged prompts padded to 128k, 64
  // groups of 128 rows: statistics 278 us at 2048 keys, 267 at 1024, 274 at
  // 512; column sums 310, 288, 268 -- the statistics also write a (max, sum)
  // per row and chunk for stats_reduce, 10 / 13 / 28 us, so their chunks are
  // longer).  A single 50k prompt: statistics 28 us at 512 keys, 32 at 384;
  // column sums 35 and 29 us.
  const bool latent = p.d_qk > 128, narrow = !latent && p.in_dtype == SNAP_BF16;
  auto chunk = [&](long target, long least) {
    const long per_group = (target + groups - 1) / (groups > 0 ? groups : 1);
    long kc = (max_len + per_group - 1) / (per_group > 0 ? per_group : 1);
    if (kc < least) kc = least;
    kc = (kc + kKeyTile - 1) / kKeyTile * kKeyTile;
    return (int)(kc > 16384 ? 16384 : kc);
  };
  const long rp = g.rows_pad;
  g.key_chunk = narrow ? chunk(8192, rp > 64 ? 4 * rp : 256) : chunk(4096, (rp > 128 ? 16 : 4) * rp);
  g.col_chunk = narrow && rp > 64 ? chunk(16384, 3 * rp) : g.key_chunk;
  g.n_kchunks = (max_len + g.key_chunk - 1) / g.key_chunk;
  g.n_colchunks = (max_len + g.col_chunk - 1) / g.col_chunk;
  if (g.n_kchunks < 1) g.n_kchunks = 1;
  if (g.n_colchunks < 1) g.n_colchunks = 1;
  int ncand = max_len - p.sink - p.recent;
  if (ncand < 1) ncand = 1;
  g.n_splits = (ncand + kCandChunk - 1) / kCandChunk;
  size_t off = 0;
  g.off_stats = off;
  off = align256(off + (size_t)groups * g.n_kchunks * g.rows_pad * sizeof(float2));
  g.off_rowref = off;
  off = align256(off + (size_t)groups * g.rows_pad * sizeof(float2));
  g.off_A = off;
  off = align256(off + (size_t)groups * max_len * sizeof(float));
  g.off_P = off;
  off = align256(off + (size_t)groups * max_len * sizeof(float));
  g.off_hist = off;
  off = align256(off + (size_t)groups * (kHistBins + kSubBins) * sizeof(uint32_t));
  g.off_list = off;
  off = align256(off + (size_t)groups * kListCap * sizeof(uint2));
  g.off_list_n = off;
  off = align256(off + (size_t)groups * sizeof(int32_t));
  g.off_state = off;
  off = align256(off + (size_t)groups * sizeof(RadixState));
  g.off_counts = off;
  off = align256(off + (size_t)groups * g.n_splits * sizeof(uint2));
  g.off_sel = off;
  off = align256(off + (size_t)groups * (p.topk > 0 ? p.topk : 1) * sizeof(int32_t));
  // per (group, assemble row block): amax of the kept K and V rows (fp8 scales)
  g.n_rowblocks = (p.sink + p.recent + p.topk + kAsmRows - 1) / kAsmRows;
  g.off_amax = off;
  off = align256(off + (size_t)groups * g.n_rowblocks * sizeof(float2));
  g.off_rowz = off;
  off = align256(off + (size_t)groups * g.rows_pad * sizeof(double2));
  g.off_band_n = off;
  off = align256(off + (size_t)groups * sizeof(int32_t));
  g.off_band_idx = off;
  off = align256(off + (size_t)groups * kBandCap * sizeof(int32_t));
  g.off_band_p = off;
  off = align256(off + (size_t)groups * kBandCap * sizeof(double));
  g.off_band_above = off;
  off = align256(off + (size_t)groups * g.n_splits * sizeof(uint32_t));
  g.off_A64 = off;
  off = align256(off + (size_t)groups * kBandKeyCap * kBandMaxPass * sizeof(double));
  g.compress_bytes = off;
  return g;
}

template <typename In, int KS, int NW, int TK, int STAGES>
static hipError_t launch_score_nw(const ScoreArgs& sa, bool colsum, int groups, int n_kchunks, hipStream_t st) {
  dim3 grid(n_kchunks, groups), block(64 * NW);
  if (colsum)
    hipLaunchKernelGGL((score_pass<In, KS, NW, true, TK, STAGES>), grid, block, 0, st, sa);
  else
    hipLaunchKernelGGL((score_pass<In, KS, NW, false, TK, STAGES>), grid, block, 0, st, sa);
  return hipGetLastError();
}

template <int KS>
static hipError_t launch_stream(const ScoreArgs& sa, bool colsum, int groups, int n_kchunks, hipStream_t st) {
  dim3 grid(n_kchunks, groups);
  void (*k)(ScoreArgs);
  if (sa.rows_pad <= 32)
    k = colsum ? score_stream<KS, 2, true> : score_stream<KS, 2, false>;
  else
    k = colsum ? score_stream<KS, 4, true> : score_stream<KS, 4, false>;
  hipLaunchKernelGGL(k, grid, dim3(256), 0, st, sa);
  return hipGetLastError();
}

// Waves per workgroup: 4 while the score rows fit in 128, else 8.  Tiles and
// stages per shape, as measured: the 576-wide latent rows take 32-key tiles in
// 4 stages (147 KB, one workgroup per CU: three tiles in flight while one is
// scored; 8% faster than two 64-key stages); 64/128-wide bf16 rows keep two
// 64-key stages (three workgroups per CU; three or four stages measured
// slower); fp32 rows 3 or 2 stages next to their fp32 query block.
// Few rows run score_stream: whole compress calls of 1 to 16 prompts of 2000 to
// 131072 tokens against the LDS pass, 64-wide keys, up to 32 rows 0 to 56%
// faster (one 128k prompt 186 -> 126 us at 32 rows), 33 to 64 rows 1% slower to
// 28% faster (16 x 128k 1107 -> 876 us); 128-wide, up to 32 rows 7% slower (a
// short batch of one or two KV heads) to 38% faster (one 128k prompt, 8 KV heads,
// 230 -> 178 us), 33 to 64 rows 9% slower (16 x 16k 326 -> 359 us) to 4% faster
// (4 x 128k 447 -> 433 us).  With 128 rows a wave holds 254 registers and the
// statistics pass of a 128k batch took 344 instead of 278 us.
template <typename In>
static hipError_t launch_score(const ScoreArgs& sa, int dk, bool colsum, int groups, int n_kchunks, hipStream_t st) {
  const bool wide = sa.rows_pad > 128;
  if constexpr (sizeof(In) == 2) {
    if (dk <= 128 && sa.rows_pad <= 64)
      return dk == 64 ? launch_stream<2>(sa, colsum, groups, n_kchunks, st)
                      : launch_stream<4>(sa, colsum, groups, n_kchunks, st);
    if (dk == 64) return wide ? launch_score_nw<In, 2, 8, 64, 2>(sa, colsum, groups, n_kchunks, st)
                              : launch_score_nw<In, 2, 4, 64, 2>(sa, colsum, groups, n_kchunks, st);
    if (dk == 128) return wide ? launch_score_nw<In, 4, 8, 64, 2>(sa, colsum, groups, n_kchunks, st)
                               : launch_score_nw<In, 4, 4, 64, 2>(sa, colsum, groups, n_kchunks, st);
    if (dk == 576) return wide ? launch_score_nw<In, 18, 8, 32, 4>(sa, colsum, groups, n_kchunks, st)
                               : launch_score_nw<In, 18, 4, 32, 4>(sa, colsum, groups, n_kchunks, st);
  } else {
    if (wide) return hipErrorInvalidValue;  // fp32 inputs: at most 128 score rows
    if (dk == 64) return launch_score_nw<In, 2, 4, 64, 3>(sa, colsum, groups, n_kchunks, st);
    if (dk == 128) return launch_score_nw<In, 4, 4, 64, 2>(sa, colsum, groups, n_kchunks, st);
  }
  return hipErrorInvalidValue;
}

snap_status launch_compress(const snap_params& p, const snap_cache& c, int32_t* pos, int32_t* n_topk, int n_seq,
                            const int32_t* slot_ids, const int32_t* lengths, int max_len, const void* q_obs,
                            const void* k, const void* v, int32_t* sel_out, float* pooled_out, void* ws,
                            hipStream_t stream, bool stats_given) {
  Geometry geo = compress_geometry(p, n_seq, max_len);
  const int groups = n_seq * p.n_kv_heads;
  const int G = p.n_q_heads / p.n_kv_heads;
  const float scale = p.sm_scale > 0.f ? p.sm_scale : 1.0f / sqrtf((float)p.d_qk);
  unsigned char* w = (unsigned char*)ws;
  float2* stats = (float2*)(w + geo.off_stats);
  float2* rowref = (float2*)(w + geo.off_rowref);
  float* A = (float*)(w + geo.off_A);
  float* P = (float*)(w + geo.off_P);
  uint32_t* hist = (uint32_t*)(w + geo.off_hist);
  RadixState* state = (RadixState*)(w + geo.off_state);
  uint2* counts = (uint2*)(w + geo.off_counts);
  int32_t* sel = (int32_t*)(w + geo.off_sel);
  double2* rowz = (double2*)(w + geo.off_rowz);
  int32_t* band_n = (int32_t*)(w + geo.off_band_n);
  int32_t* band_idx = (int32_t*)(w + geo.off_band_idx);
  double* band_p = (double*)(w + geo.off_band_p);
  uint32_t* band_above = (uint32_t*)(w + geo.off_band_above);
  double* A64 = (double*)(w + geo.off_A64);

  ScoreArgs sa;
  sa.q = q_obs;
  sa.k = k;
  sa.lengths = lengths;
  sa.stats = stats;
  sa.rowref = rowref;
  sa.A = A;
  sa.Hq = p.n_q_heads;
  sa.Hkv = p.n_kv_heads;
  sa.G = G;
  sa.w = p.obs_window;
  sa.max_len = max_len;
  sa.sink = p.sink;
  sa.recent = p.recent;
  sa.norm = p.norm;
  sa.rows = geo.rows;
  sa.rows_pad = geo.rows_pad;
  sa.key_chunk = geo.key_chunk;
  sa.n_kchunks = geo.n_kchunks;
  sa.groups = groups;
  split_scale2(scale, sa.scale2, sa.scale2_lo);
  const bool bf = p.in_dtype == SNAP_BF16;
  hipError_t e;
  // With no selected rows (StreamingLLM alone) the cache is sinks and ring
  // only: nothing is scored or selected (unless the pooled scores are asked
  // for), the assembly is the whole call.
  const bool select = p.topk > 0 || pooled_out;

  if (select) {
    // stats_given: the prefill attention pass already wrote each window row's
    // (max, sum) over its whole domain, as a single chunk
    if (!stats_given) {
      e = bf ? launch_score<uint16_t>(sa, p.d_qk, false, groups, geo.n_kchunks, stream)
             : launch_score<float>(sa, p.d_qk, false, groups, geo.n_kchunks, stream);
      if (e != hipSuccess) return SNAP_ERR_HIP;
    }

    ReduceArgs ra;
    ra.stats = stats;
    ra.rowref = rowref;
    ra.rowz = rowz;
    ra.band_n = band_n;
    ra.lengths = lengths;
    ra.hist = hist;
    ra.list_n = (int32_t*)(w + geo.off_list_n);
    ra.reset_wgs = (geo.rows_pad + kReduceRows - 1) / kReduceRows;
    ra.state = state;
    ra.groups = groups;
    ra.Hkv = p.n_kv_heads;
    ra.max_len = max_len;
    ra.sink = p.sink;
    ra.recent = p.recent;
    ra.topk = p.topk;
    ra.rows_pad = geo.rows_pad;
    ra.n_kchunks = stats_given ? 1 : geo.n_kchunks;
    hipLaunchKernelGGL(stats_reduce, dim3(ra.reset_wgs, groups), dim3(256), 0, stream, ra);
    if (hipGetLastError() != hipSuccess) return SNAP_ERR_HIP;

    sa.key_chunk = geo.col_chunk;
    sa.n_kchunks = geo.n_colchunks;
    e = bf ? launch_score<uint16_t>(sa, p.d_qk, true, groups, geo.n_colchunks, stream)
           : launch_score<float>(sa, p.d_qk, true, groups, geo.n_colchunks, stream);
    if (e != hipSuccess) return SNAP_ERR_HIP;

    SelectArgs se;
    se.A = A;
    se.P = P;
    se.pooled_out = pooled_out;
    se.lengths = lengths;
    se.hist = hist;
    se.list = (uint2*)(w + geo.off_list);
    se.list_n = (int32_t*)(w + geo.off_list_n);
    {
      const float most = (float)geo.rows;
      uint32_t bits;
      memcpy(&bits, &most, sizeof(bits));
      se.hist_top = bits >> 17;
    }
    se.state = state;
    se.counts = counts;
    se.sel = sel;
    se.band_n = band_n;
    se.band_idx = band_idx;
    se.band_above = band_above;
    se.groups = groups;
    se.Hkv = p.n_kv_heads;
    se.max_len = max_len;
    se.sink = p.sink;
    se.recent = p.recent;
    se.topk = p.topk;
    se.pool_kernel = p.pool_kernel;
    se.pool = p.pool;
    se.n_splits = geo.n_splits;
    dim3 sgrid(geo.n_splits, groups);
    hipLaunchKernelGGL(pool_hist, sgrid, dim3(kSelThreads), 0, stream, se);
    hipLaunchKernelGGL(select_refine, sgrid, dim3(kSelThreads), 0, stream, se);
    hipLaunchKernelGGL(select_collect, sgrid, dim3(kSelThreads), 0, stream, se);
    hipLaunchKernelGGL(select_threshold, dim3(groups), dim3(kThrThreads), 0, stream, se);
    // fp64 re-score of the candidates next to the threshold, then the final
    // decision among them
    BandArgs ba;
    ba.q = q_obs;
    ba.k = k;
    ba.lengths = lengths;
    ba.rowz = rowz;
    ba.state = state;
    ba.band_n = band_n;
    ba.band_idx = band_idx;
    ba.A64 = A64;
    ba.band_p = band_p;
    ba.pooled_out = pooled_out;
    ba.P = P;
    ba.counts = counts;
    ba.band_above = band_above;
    ba.state_w = state;
    ba.Hq = p.n_q_heads;
    ba.Hkv = p.n_kv_heads;
    ba.G = G;
    ba.w = p.obs_window;
    ba.D = p.d_qk;
    ba.max_len = max_len;
    ba.sink = p.sink;
    ba.recent = p.recent;
    ba.pool_kernel = p.pool_kernel;
    ba.pool = p.pool;
    ba.rows = geo.rows;
    ba.rows_pad = geo.rows_pad;
    ba.n_splits = geo.n_splits;
    ba.in_f32 = !bf;
    ba.band_wgs = band_workgroups(p.d_qk, groups);
    // query-dim slices per score row: 8 for 576-wide bf16 rows and for fp32
    // rows, else 4 (as band_rescore dispatches)
    ba.rows_per_pass = kBandThreads / ((!bf || p.d_qk == 576) ? 8 : 4);
    ba.scale2 = (double)scale * 1.4426950408889634074;
    hipLaunchKernelGGL(band_rescore, dim3(ba.band_wgs, groups), dim3(kBandThreads), 0, stream, ba);
    hipLaunchKernelGGL(band_decide, dim3(groups), dim3(kSelThreads), 0, stream, ba);
    hipLaunchKernelGGL(select_write, sgrid, dim3(kSelThreads), 0, stream, se);
    if (hipGetLastError() != hipSuccess) return SNAP_ERR_HIP;
  }

  AssembleArgs aa;
  aa.k = k;
  aa.v = p.v_in_k ? nullptr : v;
  aa.ck = c.k;
  aa.cv = p.v_in_k ? nullptr : c.v;
  aa.k_scale = c.k_scale;
  aa.v_scale = c.v_scale;
  aa.slot_ids = slot_ids;
  aa.lengths = lengths;
  aa.sel = sel;
  aa.state = state;
  aa.sel_out = sel_out;
  aa.pos = pos;
  aa.n_topk = n_topk;
  aa.Hkv = p.n_kv_heads;
  aa.max_len = max_len;
  aa.sink = p.sink;
  aa.recent = p.recent;
  aa.topk = p.topk;
  aa.dk = p.d_qk;
  aa.dv = p.d_v;
  aa.n_slots = c.n_slots;
  aa.rows_per_block = kAsmRows;
  aa.n_rowblocks = geo.n_rowblocks;
  aa.amax = nullptr;
  dim3 agrid(geo.n_rowblocks, groups);
  if (p.kv_dtype == SNAP_FP8_E4M3 && p.fp8_scales == SNAP_FP8_SCALES_AMAX) {
    aa.amax = (float2*)(w + geo.off_amax);
    hipLaunchKernelGGL(fp8_amax, agrid, dim3(256), 0, stream, aa);
  }
  if (p.kv_dtype == SNAP_FP8_E4M3) {
    if (bf)
      hipLaunchKernelGGL((assemble<uint16_t, uint8_t>), agrid, dim3(256), 0, stream, aa);
    else
      hipLaunchKernelGGL((assemble<float, uint8_t>), agrid, dim3(256), 0, stream, aa);
  } else if (bf) {
    hipLaunchKernelGGL((assemble<uint16_t, uint16_t>), agrid, dim3(256), 0, stream, aa);
  } else {
    hipLaunchKernelGGL((assemble<float, float>), agrid, dim3(256), 0, stream, aa);
  }
  if (hipGetLastError() != hipSuccess) return SNAP_ERR_HIP;
  return SNAP_OK;
}

}  // namespace snap

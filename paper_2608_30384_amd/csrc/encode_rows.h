// The fused RSLM encoder on 16-lane rows (rows_dev.h), for D >= 128: residual,
// rotation, EVT scale, nearest centroids, norm correction, both 16-bit scales,
// packing into the scan tile layout, and the second stage or the rotated
// second residual.  One instantiation per codec (bit width, Rslm4Lite, second
// stage) and per (rows per vector, blocks per row).
#pragma once

#include "rows_dev.h"

namespace rslm {

struct EncodeArgs {
  const float *x;
  int64_t n_rows;
  const int64_t *src_row;
  const int32_t *rec_list;
  int64_t n_records;
  const float *cen, *cen_rot;
  int nlist;
  uint8_t *codes;
  uint32_t *scales;
  float *resid;                    // rotated second residual as floats, or null
  uint8_t *codes2;                 // SQ8 codes (with sq8_lo) or second-stage codes
  uint32_t *scales2;
  const float *sq8_lo, *sq8_hi;
  RotParams rp;
  CodecParams cp, cp2;
};

// Bound by VALU issue: about 60 instructions per coordinate (two rotation
// passes 16, quantiser 12 for 1-D codebooks, the rest residual, norms, signs
// and the second residual), 40 % more for 2-D and twice as many for 4-D ones.
// Registers (and with one row per vector LDS) set the wavefronts in flight:
// 24 coordinates per lane run four wavefronts per SIMD where 48 (one row per
// vector) ran three.  Whole calls, us, against one row per vector for D = 128
// NB and 1-D codebooks, and a vector in LDS for the rest: 65,536 x 768 4-bit +
// SQ8 171 -> 123; 524,288 x 768 two-stage 1,314 -> 998; 65,536 x 1,024 2-bit 816
// -> 150; 65,536 x 2,049 4-bit 1,307 -> 288 (kernel); 153,633 x 698
// two-stage 1,425 -> 395.  At D = 128, 256 and 384 with 1-D codebooks (one row
// either way) 400,000 x 128 + SQ8 100 -> 94, 400,000 x 384 276 -> 210.  Calls of a
// few thousand vectors are one wavefront's chain of waits (arguments, tables,
// record, centre, LDS lookups): with the sign words looked up where they are
// used, the quantiser's table counted per workgroup, a record's list loaded
// after its row and one coordinate quantised after the other, 2,000 x 128 took
// 4.8 us and 2,000 x 128 two-stage 6.5; 3.9 and 5.9 here (4.2 and 6.3 with one row
// per vector and the tables of one dimension).
template <int RPV, int NBR, int BITS, bool LITE, bool TWO, bool FULL>
__global__ void __launch_bounds__(256, NBR <= 1 ? 8 : NBR <= 2 ? 6 : NBR <= 3 ? 4 : NBR <= 5 ? 3 : 2) k_encode_rows(EncodeArgs a) {
  constexpr int E = 8 * NBR;
  constexpr int VPW = 4 / RPV;                      // vectors per wavefront
  constexpr int G = BITS == 1 ? 4 : BITS == 2 ? 2 : 1;
  constexpr int K = BITS == 3 ? 8 : 16;
  constexpr int W = BITS == 3 ? 3 : 4;              // bits per code
  constexpr uint32_t kMask = (1u << W) - 1u;
  extern __shared__ float4 lds4[];
  __shared__ __align__(16) uint32_t s1[kSignWords];
  __shared__ float cbs[16], thr[16];
  __shared__ float cb8[LITE ? 16 : 1], thr8[LITE ? 16 : 1];
  __shared__ float4 cb4[G > 1 ? 16 : 1];            // 2-D and 4-D centroids
  __shared__ uint16_t g1t[G == 2 ? kGrid2 * kGrid2 : 1];
  __shared__ float4 cb2[TWO ? 16 : 1];              // second codebook: x, y, |C|^2 / 2
  __shared__ uint16_t g2t[TWO ? kGrid2 * kGrid2 : 1];
  __shared__ uint8_t qtab[G == 1 ? kQuantBuckets : 1];
  __shared__ uint8_t qtab8[LITE ? kQuantBuckets : 1];
  const RotParams &rp = a.rp;
  const CodecParams &cp = a.cp;
  const int D = rp.D;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int stride = rows_stride(D);
  // dynamic LDS: a buffer per vector, the transpose table, the SQ8 ranges
  float *lds = reinterpret_cast<float *>(lds4);
  uint16_t *ts = reinterpret_cast<uint16_t *>(lds + 4 * VPW * stride);
  float *sq = reinterpret_cast<float *>(ts + 128 * RPV * NBR);   // lo, then 255 / (hi - lo)
  const bool has_sq = !TWO && a.sq8_lo;
  const int sq_n = (D + 3) / 4 * 4;
  // with an overlapping block every pass is scaled as it ends; so it is for
  // 2-D and 4-D codebooks (their codes are those of the LDS path)
  const bool mid = (!FULL && rp.overlap) || G > 1;

  // the arguments that the first loads need, in one go (the compiler would fetch
  // each behind the branch on the one before)
  asm volatile("" ::"s"(a.n_records), "s"(a.src_row), "s"(a.cen), "s"(a.rec_list), "s"(rp.passes), "s"(rp.tsrc),
               "s"(cp.qtab));
  const int64_t n_groups = (a.n_records + VPW - 1) / VPW;
  const int64_t step = int64_t(gridDim.x) * 4;
  // source row and list of this lane's record of group g (both loads in
  // flight at once: looked at when the group's turn comes)
  auto fetch = [&](int64_t g, int64_t &row, int &L) {
    const int64_t rec = g * VPW + (lane >> 4) / RPV;
    row = -1;
    L = -1;
    if (rec < a.n_records) {
      row = a.src_row ? a.src_row[rec] : rec;
      if (a.cen) L = a.rec_list[rec];
    }
  };
  int64_t nrow;
  int nL;
  fetch(int64_t(blockIdx.x) * 4 + wid, nrow, nL);

  // Tables: every load first, then the stores, so that a workgroup waits for
  // memory once before its first record.
  RowsTs<128 * RPV * NBR> tload;
  tload.load(rp);
  RowsSigns signs;
  signs.load(rp);
  constexpr int kG2 = kGrid2 * kGrid2 / 256;
  uint16_t gv1[G == 2 ? kG2 : 1], gv2[TWO ? kG2 : 1];
  if (G == 2) {
#pragma unroll
    for (int u = 0; u < kG2; ++u) gv1[u] = cp.g2tab[tid + 256 * u];
  }
  if (TWO) {
#pragma unroll
    for (int u = 0; u < kG2; ++u) gv2[u] = a.cp2.g2tab[tid + 256 * u];
  }
  constexpr int kSq = TWO ? 1 : (128 * RPV * NBR + 255) / 256;
  float lov[kSq], hiv[kSq];
  if (has_sq) {
#pragma unroll
    for (int u = 0; u < kSq; ++u) {
      lov[u] = a.sq8_lo[min(tid + 256 * u, D - 1)];
      hiv[u] = a.sq8_hi[min(tid + 256 * u, D - 1)];
    }
  }
  // quantiser tables of the plan
  const uint8_t qv = G == 1 ? cp.qtab[tid & (kQuantBuckets - 1)] : 0;
  const uint8_t qv8 = LITE ? cp.qtab[kQuantBuckets + (tid & (kQuantBuckets - 1))] : 0;
  // the codebooks (kernel arguments), entry t of 16 by thread t
  const int t16 = tid & 15;
  float cbv[G], thv = 0.f, c8v = 0.f, t8v = 0.f, c2v[3] = {};
#pragma unroll
  for (int t = 0; t < G; ++t) cbv[t] = cp.cb[G * t16 + t];
  if (G == 1) thv = cp.thr[t16];
  if (LITE) {
    c8v = cp.cb_lead[t16 & 7];
    t8v = cp.thr_lead[t16];
  }
  if (TWO) {
    c2v[0] = a.cp2.cb[2 * t16];
    c2v[1] = a.cp2.cb[2 * t16 + 1];
    c2v[2] = a.cp2.cbh[t16];
  }
  tload.store(ts, rp, signs, !mid);
  if (tid < kQuantBuckets) {
    if (G == 1) qtab[tid] = qv;
    if (LITE) qtab8[tid] = qv8;
  }
  if (tid < 16) {
    if constexpr (G == 1) {
      cbs[tid] = cbv[0];
      // sorted decision thresholds, padded with +inf (the comparison after the
      // bucket lookup never passes beyond the last one)
      thr[tid] = (tid + 1 < K) ? thv : __builtin_inff();
    } else if constexpr (G == 2) {
      cb4[tid] = make_float4(cbv[0], cbv[1], 0.f, 0.f);
    } else {
      cb4[tid] = make_float4(cbv[0], cbv[1], cbv[2], cbv[3]);
    }
    if (LITE) {
      cb8[tid] = (tid < 8) ? c8v : 0.f;
      thr8[tid] = t8v;
    }
    if (TWO) cb2[tid] = make_float4(c2v[0], c2v[1], c2v[2], 0.f);
  }
  if (G == 2) {
#pragma unroll
    for (int u = 0; u < kG2; ++u) g1t[tid + 256 * u] = gv1[u];
  }
  if (TWO) {
#pragma unroll
    for (int u = 0; u < kG2; ++u) g2t[tid + 256 * u] = gv2[u];
  }
  if (has_sq) {
#pragma unroll
    for (int u = 0; u < kSq; ++u) {
      const int d = tid + 256 * u;
      if (d < D) {
        sq[d] = lov[u];
        sq[sq_n + d] = sq8_inv(lov[u], hiv[u]);
      }
    }
  }
  signs.fill(s1, rp);
  __syncthreads();

  for (int64_t grp = int64_t(blockIdx.x) * 4 + wid; grp < n_groups; grp += step) {
    const int L = nL;
    const bool none = nrow < 0 || nrow >= a.n_rows || (a.cen && (L < 0 || L >= a.nlist));
    const int64_t row = nrow;
    // the lane's place, opaque here: the compiler would otherwise keep every
    // address and bound derived from it in registers across the loop
    int olane = lane;
    asm volatile("" : "+v"(olane));
    const RowsLane<RPV> ln(olane);
    const int r = ln.r, pv = ln.pv;
    float *vb = lds + (wid * VPW + ln.vslot) * stride;
    const bool lead_lane = LITE && pv == 0 && r < cp.lead / 8;   // block 0 of these lanes is on cb8
    const int64_t rec = grp * VPW + ln.vslot;
    fetch(grp + step, nrow, nL);
    // rows without a vector sit the iteration out (rows of different vectors
    // never exchange data, and no workgroup barrier follows)
    if (none) continue;

    // residual r = x - c, its sums, and S1
    const int c0 = 128 * pv + 8 * r;   // this lane's first coordinate of block j is c0 + 128 RPV j
    const float *xr = a.x + row * D;
    const float *cr = a.cen ? a.cen + int64_t(L) * D : nullptr;
    float z[E];
    float xx = 0.f, rr = 0.f, cc = 0.f;
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      const int c = c0 + 128 * RPV * j;
      float xv[8], cv[8];
      if (j + 1 < NBR || FULL) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const Float4u v = *reinterpret_cast<const Float4u *>(xr + c + 4 * h);
          xv[4 * h] = v.x;
          xv[4 * h + 1] = v.y;
          xv[4 * h + 2] = v.z;
          xv[4 * h + 3] = v.w;
          if (cr) {
            const Float4u w = *reinterpret_cast<const Float4u *>(cr + c + 4 * h);
            cv[4 * h] = w.x;
            cv[4 * h + 1] = w.y;
            cv[4 * h + 2] = w.z;
            cv[4 * h + 3] = w.w;
          } else {
            cv[4 * h] = cv[4 * h + 1] = cv[4 * h + 2] = cv[4 * h + 3] = 0.f;
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int ci = min(c + i, D - 1);
          const float v = xr[ci], w = cr ? cr[ci] : 0.f;
          xv[i] = (c + i < D) ? v : 0.f;
          cv[i] = (c + i < D) ? w : 0.f;
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float d = xv[i] - cv[i];
        xx = fmaf(xv[i], xv[i], xx);
        rr = fmaf(d, d, rr);
        cc = fmaf(cv[i], cv[i], cc);
        xv[i] = d;
      }
      rows_flip(xv, s1, j * RPV + pv, r);
#pragma unroll
      for (int i = 0; i < 8; ++i) z[8 * j + i] = xv[i];
      if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);   // at most 2 blocks of loads in flight
    }
    xx = vec_sum<RPV>(xx);
    rr = vec_sum<RPV>(rr);
    cc = vec_sum<RPV>(cc);
    rows_forward<RPV, NBR, FULL>(z, rp, ts, vb, ln, mid);
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) m = fmaxf(m, fabsf(z[e]));
    m = vec_max<RPV>(m);
    const float inv_s0 = (m > 0.f) ? cp.emax / m : 0.f;

    // Nearest centroids; the codes of a lane's 8 coordinates of block j are
    // the packed word[j].  Centroid values are looked up again where needed.
    // ||c^||^2 accumulates here.  1-D: number of thresholds below u, the count
    // below u's bucket on the quantiser grid plus one comparison with the next
    // threshold (the grid has at most one per bucket).  2-D: the codes listed
    // for u's cell (all that can be nearest there), in ascending order with a
    // strict comparison.  4-D: all 16.
    uint32_t word[NBR];
    float cn2 = 0.f;
    // decoded centroid values of word[j]
    auto decode = [&](int j, float (&v)[8]) {
      uint32_t w = word[j];
      asm volatile("" : "+v"(w));   // looked up where used, not kept from the quantiser
      if constexpr (G == 1) {
        float *cbb = (LITE && j == 0 && lead_lane) ? cb8 : cbs;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = lds_at(cbb, 4u * ((w >> (W * i)) & kMask));
      } else if constexpr (G == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float4 q = cb4[(w >> (4 * k)) & 15u];
          v[2 * k] = q.x;
          v[2 * k + 1] = q.y;
        }
      } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const float4 q = cb4[(w >> (4 * k)) & 15u];
          v[4 * k] = q.x;
          v[4 * k + 1] = q.y;
          v[4 * k + 2] = q.z;
          v[4 * k + 3] = q.w;
        }
      }
    };
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      const int c = c0 + 128 * RPV * j;
      uint32_t w = 0u;
      float v[8];
      if constexpr (G == 1) {
        const bool lb = LITE && j == 0 && lead_lane;
        float *tb = lb ? thr8 : thr;
        float *cbb = lb ? cb8 : cbs;
        const uint8_t *qt = lb ? qtab8 : qtab;
        const float qs = lb ? cp.qs_lead : cp.qs, qo = lb ? cp.qo_lead : cp.qo;
        const int qn = lb ? cp.qn_lead : cp.qn;
        // the three dependent lookups of a coordinate, eight coordinates at a
        // time (left to itself the compiler takes one after the other to save
        // registers: 24 waits for LDS a block, which few wavefronts hide)
        float u[8];
        uint32_t code[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          u[i] = z[8 * j + i] * inv_s0;
          code[i] = qt[quant_bucket(u[i], qs, qo, qn)];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 8; ++i) code[i] += (u[i] > tb[code[i]]) ? 1u : 0u;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          w |= code[i] << (W * i);
          v[i] = cbb[code[i]];
        }
      } else if constexpr (G == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float u0 = z[8 * j + 2 * k] * inv_s0, u1 = z[8 * j + 2 * k + 1] * inv_s0;
          const int gx = int(__builtin_amdgcn_fmed3f(fmaf(u0, cp.g2s, cp.g2o), 0.f, float(kGrid2 - 1)));
          const int gy = int(__builtin_amdgcn_fmed3f(fmaf(u1, cp.g2s, cp.g2o), 0.f, float(kGrid2 - 1)));
          const uint32_t cell = g1t[gx * kGrid2 + gy];
          float best = 3.4e38f;
          uint32_t code = 0u;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const uint32_t kk = (cell >> (4 * t)) & 15u;
            const float4 q = cb4[kk];
            const float e0 = u0 - q.x, e1 = u1 - q.y;
            const float d = fmaf(e1, e1, e0 * e0);
            code = (d < best) ? kk : code;
            best = fminf(best, d);
          }
          w |= code << (4 * k);
          const float4 q = cb4[code];
          v[2 * k] = q.x;
          v[2 * k + 1] = q.y;
        }
      } else {
        float u[8], best[2] = {3.4e38f, 3.4e38f};
        uint32_t code[2] = {0u, 0u};
#pragma unroll
        for (int t = 0; t < 8; ++t) u[t] = z[8 * j + t] * inv_s0;
        int zero = 0;   // opaque: the codebook is read again for every block, not kept
        asm volatile("" : "+v"(zero));
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {   // the same centroid in every lane: broadcast reads
          const float4 q = cb4[kk + zero];
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const float e0 = u[4 * k] - q.x, e1 = u[4 * k + 1] - q.y, e2 = u[4 * k + 2] - q.z,
                        e3 = u[4 * k + 3] - q.w;
            const float d = fmaf(e3, e3, fmaf(e2, e2, fmaf(e1, e1, e0 * e0)));
            code[k] = (d < best[k]) ? uint32_t(kk) : code[k];
            best[k] = fminf(best[k], d);
          }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          w |= code[k] << (4 * k);
          const float4 q = cb4[code[k]];
          v[4 * k] = q.x;
          v[4 * k + 1] = q.y;
          v[4 * k + 2] = q.z;
          v[4 * k + 3] = q.w;
        }
      }
      if (j + 1 < NBR || FULL) {
#pragma unroll
        for (int i = 0; i < 8; ++i) cn2 = fmaf(v[i], v[i], cn2);
      } else {
        // past D: no coordinates, and no codes beyond the last sub-vector
#pragma unroll
        for (int i = 0; i < 8; ++i) cn2 = (c + i < D) ? fmaf(v[i], v[i], cn2) : cn2;
        const int left = (D - c + G - 1) / G;   // sub-vectors of this word (may be <= 0)
        if (left < 8 / G) w &= left > 0 ? (1u << (W * left)) - 1u : 0u;
      }
      word[j] = w;
      __builtin_amdgcn_sched_barrier(0);
    }
    // a zero residual has codes 0 (its sums are multiplied by s^ = 0)
    if (!(m > 0.f)) {
#pragma unroll
      for (int j = 0; j < NBR; ++j) word[j] = 0u;
    }
    cn2 = vec_sum<RPV>(cn2);
    // <R c, c^>
    const float *rcr = (a.cen && a.cen_rot) ? a.cen_rot + int64_t(L) * D : nullptr;
    // the rotated centre's 8 coordinates of block j (0 past D, or without one)
    auto load_rc = [&](int j, float (&v)[8]) {
      const int c = c0 + 128 * RPV * j;
      if (!rcr) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = 0.f;
      } else if (j + 1 < NBR || FULL) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const Float4u w = *reinterpret_cast<const Float4u *>(rcr + c + 4 * h);
          v[4 * h] = w.x;
          v[4 * h + 1] = w.y;
          v[4 * h + 2] = w.z;
          v[4 * h + 3] = w.w;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float w = rcr[min(c + i, D - 1)];
          v[i] = (c + i < D) ? w : 0.f;
        }
      }
    };
    float rcd = 0.f;
    if (rcr) {
#pragma unroll
      for (int j = 0; j < NBR; ++j) {
        float rv[8], cv[8];
        load_rc(j, rv);
        decode(j, cv);
#pragma unroll
        for (int i = 0; i < 8; ++i) rcd = fmaf(rv[i], cv[i], rcd);
        if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
      rcd = vec_sum<RPV>(rcd);
    }
    const float s = (m > 0.f && cn2 > 0.f) ? sqrtf(rr / cn2) : 0.f;
    const uint32_t su = enc_ue7m9(s);
    const float sh = dec_ue7m9(su);
    uint32_t gu = 0x7000u;
    const float den2 = cc + 2.f * sh * rcd + sh * sh * cn2;   // ||c + R^T s^ c^||^2
    if (cp.global) gu = enc_ue4m12((den2 > 0.f) ? sqrtf(xx / den2) : 0.f);
    if (r == 0 && pv == 0) a.scales[rec] = su | (gu << 16);

    // packed words into the scan tile layout: group q = 16 b + r of record n
    // goes to lane stream 16 (r & 3) + n at byte c BITS, c = q / 4
    uint8_t *tile = a.codes + (rec >> 4) * int64_t(cp.tile_bytes) + int(rec & 15) * 16;
    const int q_end = cp.d_pad >> 3;
    auto put = [&](int q, uint32_t w) {
      const int off = (q >> 2) * BITS;
      uint8_t *p = tile + 256 * (q & 3);
      if (BITS == 4) {
        reinterpret_cast<U32u *>(p + (off >> 4) * 1024 + (off & 15))->v = w;
      } else if (BITS == 2) {
        reinterpret_cast<U16u *>(p + (off >> 4) * 1024 + (off & 15))->v = uint16_t(w);
      } else if (BITS == 1) {
        p[(off >> 4) * 1024 + (off & 15)] = uint8_t(w);
      } else {
#pragma unroll
        for (int t = 0; t < 3; ++t)
          p[((off + t) >> 4) * 1024 + ((off + t) & 15)] = uint8_t(w >> (8 * t));
      }
    };
    uint32_t emb = 0u;   // Rslm4Lite: scale byte of this lane spread into bit 3 of each nibble
    if (LITE && lead_lane) {
      const uint32_t byte = ((r < 2 ? su : gu) >> (8 * (r & 1))) & 0xffu;
#pragma unroll
      for (int i = 0; i < 8; ++i) emb |= ((byte >> i) & 1u) << (4 * i + 3);
    }
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      const int q = 16 * (j * RPV + pv) + r;
      if (q < q_end) put(q, j == 0 ? (word[j] | emb) : word[j]);
    }
    // padding chunks past the blocks
    for (int q = 16 * (RPV * NBR) + 16 * pv + r; q < q_end; q += 16 * RPV) put(q, 0u);

    const float gh = dec_ue4m12(gu);
    if constexpr (TWO) {
      // second residual r2 = R x - R a, R a = g^ (R c + s^ c^), kept in z
      float m2 = 0.f, rr2 = 0.f;
#pragma unroll
      for (int j = 0; j < NBR; ++j) {
        float rv[8], cv[8];
        load_rc(j, rv);
        decode(j, cv);
        const int c = c0 + 128 * RPV * j;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int e = 8 * j + i;
          float d = z[e] + rv[i] - gh * (rv[i] + sh * cv[i]);
          if (j + 1 == NBR && !FULL) d = (c + i < D) ? d : 0.f;
          z[e] = d;
          m2 = fmaxf(m2, fabsf(d));
          rr2 = fmaf(d, d, rr2);
        }
        if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
      m2 = vec_max<RPV>(m2);
      rr2 = vec_sum<RPV>(rr2);
      const float inv2 = (m2 > 0.f) ? a.cp2.emax / m2 : 0.f;
      // Nearest 2-D centroid: argmin_k |c_k|^2 / 2 - <u, c_k> (lower k on
      // ties) over the (at most four) codes listed for u's cell of the grid,
      // in ascending order with a strict comparison: the same code as a scan
      // of all K (the lists hold every code that can be nearest in the cell).
      // With the codes of a block: ||c2^||^2, <c^, c2^> and <R c, c2^>.  A
      // zero r2 (m2 = 0) gets codes 0 and s2^ = 0, which removes these sums
      // from g2^, so they need no guard.
      uint32_t w2[NBR];
      float cn22 = 0.f, c12 = 0.f, rc2 = 0.f;
#pragma unroll
      for (int j = 0; j < NBR; ++j) {
        const int c = c0 + 128 * RPV * j;
        float rv[8], cv[8], v2[8];
        load_rc(j, rv);
        w2[j] = 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float u0 = z[8 * j + 2 * k] * inv2, u1 = z[8 * j + 2 * k + 1] * inv2;
          const int gx = int(__builtin_amdgcn_fmed3f(fmaf(u0, a.cp2.g2s, a.cp2.g2o), 0.f, float(kGrid2 - 1)));
          const int gy = int(__builtin_amdgcn_fmed3f(fmaf(u1, a.cp2.g2s, a.cp2.g2o), 0.f, float(kGrid2 - 1)));
          const uint32_t cell = g2t[gx * kGrid2 + gy];
          float best = 3.4e38f;
          uint32_t code = 0u;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const uint32_t kk = (cell >> (4 * t)) & 15u;
            const float4 ck = cb2[kk];
            const float d = fmaf(-u1, ck.y, fmaf(-u0, ck.x, ck.z));
            code = (d < best) ? kk : code;
            best = fminf(best, d);
          }
          const float4 ck = cb2[code];
          v2[2 * k] = ck.x;
          v2[2 * k + 1] = ck.y;
          w2[j] |= code << (4 * k);
        }
        decode(j, cv);
        if (j + 1 == NBR && !FULL) {
#pragma unroll
          for (int i = 0; i < 8; ++i) v2[i] = (c + i < D) ? v2[i] : 0.f;
          const int left = (D - c + 1) / 2;
          if (left < 4) w2[j] &= left > 0 ? (1u << (4 * left)) - 1u : 0u;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          cn22 = fmaf(v2[i], v2[i], cn22);
          c12 = fmaf(cv[i], v2[i], c12);
          rc2 = fmaf(rv[i], v2[i], rc2);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (!(m2 > 0.f)) {
#pragma unroll
        for (int j = 0; j < NBR; ++j) w2[j] = 0u;
      }
      cn22 = vec_sum<RPV>(cn22);
      const float rad = gh * vec_sum<RPV>(fmaf(sh, c12, rc2));   // <R a, c2^>
      const float s2 = (m2 > 0.f && cn22 > 0.f) ? sqrtf(rr2 / cn22) : 0.f;
      const uint32_t su2 = enc_ue7m9(s2);
      const float sh2 = dec_ue7m9(su2);
      uint32_t gu2 = 0x7000u;
      if (a.cp2.global) {
        const float dd = gh * gh * den2 + 2.f * sh2 * rad + sh2 * sh2 * cn22;
        gu2 = enc_ue4m12((dd > 0.f) ? sqrtf(xx / dd) : 0.f);
      }
      if (r == 0 && pv == 0) a.scales2[row] = su2 | (gu2 << 16);
      // canonical record: the lane's four codes of block b are bytes 2 q, 2 q + 1
      uint8_t *dst = a.codes2 + row * int64_t(a.cp2.canon_bytes);
#pragma unroll
      for (int j = 0; j < NBR; ++j) {
        const int byte = 2 * (16 * (j * RPV + pv) + r);
        if (byte + 2 <= a.cp2.canon_bytes) reinterpret_cast<U16u *>(dst + byte)->v = uint16_t(w2[j]);
        else if (byte < a.cp2.canon_bytes) dst[byte] = uint8_t(w2[j]);
      }
    } else if (a.resid || has_sq) {
      // the rotated second residual as floats and / or SQ8 codes (the
      // rslm_sq8_encode arithmetic), indexed by source row
#pragma unroll
      for (int j = 0; j < NBR; ++j) {
        const int c = c0 + 128 * RPV * j;
        float rv[8], cv[8], o[8];
        load_rc(j, rv);
        decode(j, cv);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = z[8 * j + i] + rv[i] - gh * (rv[i] + sh * cv[i]);
        const bool full = j + 1 < NBR || FULL;
        if (a.resid) {
          float *p = a.resid + row * D + c;
          if (full) {
            *reinterpret_cast<Float4u *>(p) = Float4u{o[0], o[1], o[2], o[3]};
            *reinterpret_cast<Float4u *>(p + 4) = Float4u{o[4], o[5], o[6], o[7]};
          } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
              if (c + i < D) p[i] = o[i];
          }
        }
        if (has_sq) {
          uint8_t *p = a.codes2 + row * D + c;
          if (full) {
            uint32_t w8[2] = {0u, 0u};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const float4 l4 = *reinterpret_cast<const float4 *>(sq + c + 4 * h);
              const float4 i4 = *reinterpret_cast<const float4 *>(sq + sq_n + c + 4 * h);
              w8[h] = sq8_code_put(w8[h], o[4 * h], l4.x, i4.x, 0);
              w8[h] = sq8_code_put(w8[h], o[4 * h + 1], l4.y, i4.y, 1);
              w8[h] = sq8_code_put(w8[h], o[4 * h + 2], l4.z, i4.z, 2);
              w8[h] = sq8_code_put(w8[h], o[4 * h + 3], l4.w, i4.w, 3);
            }
            *reinterpret_cast<U64u *>(p) = U64u{w8[0], w8[1]};
          } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
              if (c + i < D) p[i] = uint8_t(sq8_code_put(0u, o[i], sq[c + i], sq[sq_n + c + i], 0));
          }
        }
        if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

template <int RPV, int NBR, int BITS, bool LITE, bool TWO, bool FULL>
void launch_encode_one(const EncodeArgs &a, hipStream_t s) {
  const size_t shm = size_t(16 / RPV) * rows_stride(a.rp.D) * 4 + 128 * RPV * NBR * 2 +
                     (!TWO && a.sq8_lo ? size_t(a.rp.D + 3) / 4 * 32 : 0);
  constexpr auto kernel = k_encode_rows<RPV, NBR, BITS, LITE, TWO, FULL>;
  const int64_t groups = (a.n_records + 16 / RPV - 1) / (16 / RPV);
  // one or two blocks: short units, cheap tables (us, one unit each against
  // striding: 150,000 x 128 33.0, 35.3; 300,000 x 128 58.9, 62.1, two-stage 102.7, 108.7;
  // 100,000 x 256 32.1, 35.4; 1,000,000 x 128, 30 units each, 204, 178)
  const unsigned grid = rows_grid<kernel>(shm, groups, RPV * NBR <= 2 ? 12 : 3);
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), shm, s, a);
}

template <int BITS, bool LITE, bool TWO>
void launch_encode_rows(const EncodeArgs &a, hipStream_t s) {
#define RSLM_ENCODE_ROWS(RPV, NBR)                                             \
  {                                                                            \
    if (rows_only_full(RPV, NBR) || a.rp.D == 128 * RPV * NBR)                 \
      launch_encode_one<RPV, NBR, BITS, LITE, TWO, true>(a, s);                \
    else                                                                       \
      launch_encode_one<RPV, NBR, BITS, LITE, TWO, rows_only_full(RPV, NBR)>(a, s); \
  }
  const int nbt = rows_blocks(a.rp);
  RSLM_ROWS_SWITCH(nbt, a.rp.D == 384, RSLM_ENCODE_ROWS)
#undef RSLM_ENCODE_ROWS
}

// one per codec, each in a source file of its own (they compile in parallel)
extern template void launch_encode_rows<4, false, false>(const EncodeArgs &, hipStream_t);
extern template void launch_encode_rows<4, false, true>(const EncodeArgs &, hipStream_t);
extern template void launch_encode_rows<4, true, false>(const EncodeArgs &, hipStream_t);
extern template void launch_encode_rows<4, true, true>(const EncodeArgs &, hipStream_t);
extern template void launch_encode_rows<3, false, false>(const EncodeArgs &, hipStream_t);
extern template void launch_encode_rows<3, false, true>(const EncodeArgs &, hipStream_t);
extern template void launch_encode_rows<2, false, false>(const EncodeArgs &, hipStream_t);
extern template void launch_encode_rows<2, false, true>(const EncodeArgs &, hipStream_t);
extern template void launch_encode_rows<1, false, false>(const EncodeArgs &, hipStream_t);
extern template void launch_encode_rows<1, false, true>(const EncodeArgs &, hipStream_t);

}  // namespace rslm

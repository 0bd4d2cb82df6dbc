// Rotation of vectors spread over 16-lane rows of a wavefront, for any D >=
// 128 (blocks of 128, the last one overlapping its predecessor when 128 does
// not divide D): the device code shared by the encoder and the decoder (the
// stand-alone rotation takes its helpers only).
//
// A vector takes RPV rows (1, 2 or 4) of 16 lanes, 4 / RPV vectors per
// wavefront.  Row pv of a vector holds the 128-blocks b = j RPV + pv (j <
// NBR); in a block, lane r of the row holds the 8 consecutive coordinates
// 128 b + 8 r + i.  Coordinate bits 0..2 are the register index i and bits
// 3..6 the lane r, so three butterfly stages are in registers and four
// exchange lanes inside the row through DPP (quad_perm for lane xor 1 and 2,
// half-mirror + quad_perm for xor 4, row_ror:8 for xor 8).  The strided
// transpose between the passes, and the overlapping block, whose coordinates
// are not aligned to the lanes, go through a per-vector LDS buffer.  More
// rows per vector means fewer registers per lane and less LDS per wavefront,
// and so more wavefronts in flight; fewer rows, less work repeated per row.
#pragma once

#include <algorithm>
#include <atomic>

#include "rslm_internal.h"

namespace rslm {

__device__ __forceinline__ void wave_sync_r() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS float at a byte offset
__device__ __forceinline__ float &lds_at(float *buf, uint32_t byte_off) {
  return *reinterpret_cast<float *>(reinterpret_cast<char *>(buf) + byte_off);
}

// Four floats at any 4-byte alignment (rows of an odd dimension).
struct __attribute__((packed, aligned(4))) Float4u {
  float x, y, z, w;
};
// Words of byte arrays (packed codes) at any alignment.
struct __attribute__((packed, aligned(1))) U16u {
  uint16_t v;
};
struct __attribute__((packed, aligned(1))) U32u {
  uint32_t v;
};
struct __attribute__((packed, aligned(1))) U64u {
  uint32_t a, b;
};

constexpr int kDppQuadXor1 = 0xB1;   // quad_perm [1, 0, 3, 2]
constexpr int kDppQuadXor2 = 0x4E;   // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppRowRor8 = 0x128;

template <int CTRL>
__device__ __forceinline__ float dppf(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
// Sum / maximum over the RPV rows of a vector.  Every step adds the two values
// of a pair in both of its lanes (never a rotation of four partial sums, which
// the lanes would add in different orders), so all lanes get the same bits:
// each derives the scales from them on its own.
template <int RPV>
__device__ __forceinline__ float vec_sum(float v) {
  v += dppf<kDppQuadXor1>(v);
  v += dppf<kDppQuadXor2>(v);
  v += dppf<kDppHalfMirror>(v);   // quads now uniform: + the other quad of the half
  v += dppf<kDppRowRor8>(v);      // halves now uniform: + the other half
  if (RPV >= 2) v += __shfl_xor(v, 16, 64);
  if (RPV == 4) v += __shfl_xor(v, 32, 64);
  return v;
}
template <int RPV>
__device__ __forceinline__ float vec_max(float v) {
  v = fmaxf(v, dppf<kDppQuadXor1>(v));
  v = fmaxf(v, dppf<kDppQuadXor2>(v));
  v = fmaxf(v, dppf<kDppHalfMirror>(v));
  v = fmaxf(v, dppf<kDppRowRor8>(v));
  if (RPV >= 2) v = fmaxf(v, __shfl_xor(v, 16, 64));
  if (RPV == 4) v = fmaxf(v, __shfl_xor(v, 32, 64));
  return v;
}

// The four lane stages of the 8 elements z[o..o+7] of one block, each a DPP
// multiply-add v_fmac_f32_dpp (z += sg[k] * z of the partner lane: lane r ^ 1,
// r ^ 2, r ^ 4, r ^ 8 of the 16-lane row; r ^ 4 as a half-mirror move then a
// quad reversal).  The compiler does not fold a DPP move into the multiplied
// operand of a multiply-add, so the stages are written out here.  A DPP
// operand must not have been written by the two preceding VALU instructions:
// the block opens and closes with two wait states, and inside it every DPP
// read is at least seven instructions after the write of its register.
#define RSLM_DPP_FMAC(I, SG, SRC, CTRL) \
  "v_fmac_f32_dpp %" #I ", %" #SRC ", %" #SG " " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define RSLM_DPP_STAGE(SG, CTRL)                                                           \
  RSLM_DPP_FMAC(0, SG, 0, CTRL) RSLM_DPP_FMAC(1, SG, 1, CTRL) RSLM_DPP_FMAC(2, SG, 2, CTRL) \
  RSLM_DPP_FMAC(3, SG, 3, CTRL) RSLM_DPP_FMAC(4, SG, 4, CTRL) RSLM_DPP_FMAC(5, SG, 5, CTRL) \
  RSLM_DPP_FMAC(6, SG, 6, CTRL) RSLM_DPP_FMAC(7, SG, 7, CTRL)
#define RSLM_DPP_MIRROR(T, I) \
  "v_mov_b32_dpp %" #T ", %" #I " row_half_mirror row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
__device__ __forceinline__ void lane_stages8(float *z, int o, const float (&sg)[4]) {
  float t0, t1, t2, t3, t4, t5, t6, t7;   // half-mirrored copies (stage r ^ 4)
  asm volatile(
      "s_nop 1\n\t"
      RSLM_DPP_STAGE(16, "quad_perm:[1,0,3,2]")
      RSLM_DPP_STAGE(17, "quad_perm:[2,3,0,1]")
      RSLM_DPP_MIRROR(8, 0) RSLM_DPP_MIRROR(9, 1) RSLM_DPP_MIRROR(10, 2) RSLM_DPP_MIRROR(11, 3)
      RSLM_DPP_MIRROR(12, 4) RSLM_DPP_MIRROR(13, 5) RSLM_DPP_MIRROR(14, 6) RSLM_DPP_MIRROR(15, 7)
      RSLM_DPP_FMAC(0, 18, 8, "quad_perm:[3,2,1,0]") RSLM_DPP_FMAC(1, 18, 9, "quad_perm:[3,2,1,0]")
      RSLM_DPP_FMAC(2, 18, 10, "quad_perm:[3,2,1,0]") RSLM_DPP_FMAC(3, 18, 11, "quad_perm:[3,2,1,0]")
      RSLM_DPP_FMAC(4, 18, 12, "quad_perm:[3,2,1,0]") RSLM_DPP_FMAC(5, 18, 13, "quad_perm:[3,2,1,0]")
      RSLM_DPP_FMAC(6, 18, 14, "quad_perm:[3,2,1,0]") RSLM_DPP_FMAC(7, 18, 15, "quad_perm:[3,2,1,0]")
      RSLM_DPP_STAGE(19, "row_ror:8")
      "s_nop 1"
      : "+v"(z[o + 0]), "+v"(z[o + 1]), "+v"(z[o + 2]), "+v"(z[o + 3]), "+v"(z[o + 4]),
        "+v"(z[o + 5]), "+v"(z[o + 6]), "+v"(z[o + 7]), "=&v"(t0), "=&v"(t1), "=&v"(t2),
        "=&v"(t3), "=&v"(t4), "=&v"(t5), "=&v"(t6), "=&v"(t7)
      : "v"(sg[0]), "v"(sg[1]), "v"(sg[2]), "v"(sg[3]));
}
#undef RSLM_DPP_MIRROR
#undef RSLM_DPP_STAGE
#undef RSLM_DPP_FMAC

// Unnormalised FWHT of every 128-block of the row; sg[k] = -1 where bit k of
// r is set.  A lane stage computes own + sg[k] partner, so the exchanged
// value is the multiplied operand and the exchange folds into the
// multiply-add (one DPP multiply-add per element and stage).  In a lane with
// bit k set that is partner - own, the negative of the butterfly's
// difference: after the four lane stages lane r holds (-1)^popcount(r) times
// the transform, which the caller folds into a later sign or scale.
template <int E>
__device__ __forceinline__ void fwht_rows(float (&z)[E], const float (&sg)[4]) {
#pragma unroll
  for (int b = 0; b < E / 8; ++b) {
#pragma unroll
    for (int s = 1; s < 8; s <<= 1) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (i & s) continue;
        const float a = z[8 * b + i], c = z[8 * b + i + s];
        z[8 * b + i] = a + c;
        z[8 * b + i + s] = a - c;
      }
    }
  }
  // lane stages, one block at a time
#pragma unroll
  for (int b = 0; b < E / 8; ++b) lane_stages8(z, 8 * b, sg);
}

// A lane's place: lane r of row pv of vector vslot of the wavefront.
template <int RPV>
struct RowsLane {
  int r, pv, vslot;
  float sg[4];
  __device__ __forceinline__ RowsLane(int lane) {
    r = lane & 15;
    pv = (lane >> 4) & (RPV - 1);
    vslot = (lane >> 4) / RPV;
#pragma unroll
    for (int k = 0; k < 4; ++k) sg[k] = ((r >> k) & 1) ? -1.f : 1.f;
  }
  // the sign that fwht_rows leaves on this lane, times v
  __device__ __forceinline__ float signed_by_lane(float v) const {
    return (__popc(r) & 1) ? -v : v;
  }
};

// S1 sign bits (bit 31) of the coordinates 128 p + 8 r + i (the table repeats
// every 256 coordinates), word (16 p + r) 8 + i of an LDS table: one lane's
// words are two 16-byte reads.
constexpr int kSignWords = 256;
// The sign words of a thread of 256: of S1 at coordinate t, and of S2 at t (S1 at
// t + 127); both repeat every 256.  In two steps as RowsTs: a select among the
// mask's words would be an indexed load from the kernel's arguments at the place
// of use, one wait for memory after another before a workgroup's first record.
struct RowsSigns {
  uint32_t w1, w2;
  __device__ __forceinline__ void load(const RotParams &rp) {
    w1 = rp.s1mask[threadIdx.x >> 5];
    w2 = rp.s1mask[((threadIdx.x + 127) >> 5) & 7];
  }
  __device__ __forceinline__ void fill(uint32_t *tab, const RotParams &rp) const {
    tab[threadIdx.x] = rp.passes > 0 ? (w1 >> (threadIdx.x & 31)) << 31 : 0u;
  }
  __device__ __forceinline__ uint32_t s2() const { return (w2 >> ((threadIdx.x + 127) & 31)) & 1u; }
};
// S1 times the lane's 8 coordinates v of block b.
__device__ __forceinline__ void rows_flip(float (&v)[8], const uint32_t *tab, int b, int r) {
  const uint4 *p = reinterpret_cast<const uint4 *>(tab + 128 * (b & 1) + 8 * r);
  const uint4 s0 = p[0], s1 = p[1];
  const uint32_t w[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = __uint_as_float(__float_as_uint(v[i]) ^ w[i]);
}

// Entries of the LDS transpose table: per coordinate o < 128 RPV NBR, the byte
// offset in the vector buffer of the source of output o of the strided
// transpose, with bit 15 its sign: S2 of o, times the lane sign that fwht_rows
// leaves on the source when `lane_sign` (the forward pass without a scale in
// between).  Entries past D point at the buffer's start and are not used.
// In two steps, so that a workgroup's table loads are all in flight at once.
template <int N>
struct RowsTs {
  int src[(N + 255) / 256];
  __device__ __forceinline__ void load(const RotParams &rp) {
    if (rp.passes != 2) return;
#pragma unroll
    for (int u = 0; u < (N + 255) / 256; ++u)
      src[u] = rp.tsrc[min(int(threadIdx.x) + 256 * u, rp.D - 1)];
  }
  __device__ __forceinline__ void store(uint16_t *ts, const RotParams &rp, const RowsSigns &sg,
                                        bool lane_sign) const {
    if (rp.passes != 2) return;
#pragma unroll
    for (int u = 0; u < (N + 255) / 256; ++u) {
      const int o = threadIdx.x + 256 * u;
      // the tail [128 n_full, D) is not transformed with the full blocks, but
      // with a tail lane_sign is not set
      uint32_t s = sg.s2();
      if (lane_sign) s ^= __popc((src[u] >> 3) & 15) & 1u;
      if (o < N) ts[o] = o < rp.D ? uint16_t(uint32_t(4 * src[u]) | (s << 15)) : uint16_t(0);
    }
  }
};

__host__ __device__ constexpr int rows_stride(int D) { return (D + 3) / 4 * 4 + 4; }

// The registers of block b (the last full one, so j >= NBR - 2) to or from the
// vector buffer; tail: the coordinates of block n_full (j = NBR - 1), element
// by element.
template <int RPV, int NBR>
__device__ __forceinline__ void rows_put_block(const float (&z)[8 * NBR], int b, const RowsLane<RPV> &ln,
                                               float *vb) {
#pragma unroll
  for (int j = NBR > 1 ? NBR - 2 : 0; j < NBR; ++j) {
    if (j * RPV + ln.pv == b) {
      float *p = vb + 128 * b + 8 * ln.r;
      *reinterpret_cast<float4 *>(p) = make_float4(z[8 * j], z[8 * j + 1], z[8 * j + 2], z[8 * j + 3]);
      *reinterpret_cast<float4 *>(p + 4) =
          make_float4(z[8 * j + 4], z[8 * j + 5], z[8 * j + 6], z[8 * j + 7]);
    }
  }
}
template <int RPV, int NBR>
__device__ __forceinline__ void rows_get_block(float (&z)[8 * NBR], int b, const RowsLane<RPV> &ln,
                                               const float *vb) {
#pragma unroll
  for (int j = NBR > 1 ? NBR - 2 : 0; j < NBR; ++j) {
    if (j * RPV + ln.pv == b) {
      const float *p = vb + 128 * b + 8 * ln.r;
      const float4 a = *reinterpret_cast<const float4 *>(p), c = *reinterpret_cast<const float4 *>(p + 4);
      z[8 * j] = a.x;
      z[8 * j + 1] = a.y;
      z[8 * j + 2] = a.z;
      z[8 * j + 3] = a.w;
      z[8 * j + 4] = c.x;
      z[8 * j + 5] = c.y;
      z[8 * j + 6] = c.z;
      z[8 * j + 7] = c.w;
    }
  }
}
template <int RPV, int NBR>
__device__ __forceinline__ void rows_put_tail(const float (&z)[8 * NBR], const RotParams &rp,
                                              const RowsLane<RPV> &ln, float *vb) {
  constexpr int j = NBR - 1;
  if (j * RPV + ln.pv == rp.n_full) {
    const int c = 128 * rp.n_full + 8 * ln.r;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (c + i < rp.D) vb[c + i] = z[8 * j + i];
  }
}
// also clears what lies past D
template <int RPV, int NBR>
__device__ __forceinline__ void rows_get_tail(float (&z)[8 * NBR], const RotParams &rp,
                                              const RowsLane<RPV> &ln, const float *vb) {
  constexpr int j = NBR - 1;
  if (j * RPV + ln.pv == rp.n_full) {
    const int c = 128 * rp.n_full + 8 * ln.r;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[8 * j + i] = (c + i < rp.D) ? vb[c + i] : 0.f;
  }
}

// FWHT of the overlapping block [D - 128, D) in the vector buffer; every row
// of the vector computes it (and writes the same values).
template <int RPV>
__device__ __forceinline__ void rows_overlap(const RotParams &rp, const RowsLane<RPV> &ln, float *vb,
                                             float lane_scale) {
  float t[8];
  float *p = vb + rp.D - 128 + 8 * ln.r;
  wave_sync_r();
#pragma unroll
  for (int i = 0; i < 8; ++i) t[i] = p[i];
  fwht_rows<8>(t, ln.sg);
  wave_sync_r();
#pragma unroll
  for (int i = 0; i < 8; ++i) p[i] = t[i] * lane_scale;
  wave_sync_r();
}

// Forward rotation of z (already multiplied by S1).  ts: the transpose table
// (RowsTs with lane_sign = !mid); vb: the vector's LDS buffer.  mid:
// every pass is scaled by 1 / sqrt(128) as it ends (always so with an
// overlapping block); otherwise both scales are applied at the end, in one
// multiplication.  Registers past D end as 0.  FULL: D = 128 RPV NBR, no tail
// and no row that ends early.
template <int RPV, int NBR, bool FULL>
__device__ __forceinline__ void rows_forward(float (&z)[8 * NBR], const RotParams &rp,
                                             const uint16_t *ts, float *vb, const RowsLane<RPV> &ln,
                                             bool mid) {
  if (rp.passes == 0) return;
  const bool overlap = !FULL && rp.overlap;
  const float inv = ln.signed_by_lane(rp.inv_sqrt_b);
  if (overlap) rows_put_tail<RPV, NBR>(z, rp, ln, vb);
  fwht_rows<8 * NBR>(z, ln.sg);
  float scale = inv;
  if (rp.passes == 2) {
    if (mid) {
#pragma unroll
      for (int e = 0; e < 8 * NBR; ++e) z[e] *= inv;
    }
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      const int b = j * RPV + ln.pv;
      if (FULL || j + 1 < NBR || b < rp.n_full) {
        float *p = vb + 128 * b + 8 * ln.r;
        *reinterpret_cast<float4 *>(p) = make_float4(z[8 * j], z[8 * j + 1], z[8 * j + 2], z[8 * j + 3]);
        *reinterpret_cast<float4 *>(p + 4) =
            make_float4(z[8 * j + 4], z[8 * j + 5], z[8 * j + 6], z[8 * j + 7]);
      }
    }
    if (overlap) rows_overlap<RPV>(rp, ln, vb, inv);
    else wave_sync_r();
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      const uint4 t8 = *reinterpret_cast<const uint4 *>(ts + 128 * (j * RPV + ln.pv) + 8 * ln.r);
      const uint32_t tw[4] = {t8.x, t8.y, t8.z, t8.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t off = (tw[i >> 1] >> (16 * (i & 1))) & 0x7fffu;
        const uint32_t sb = (i & 1) ? tw[i >> 1] & 0x80000000u : (tw[i >> 1] << 16) & 0x80000000u;
        z[8 * j + i] = __uint_as_float(__float_as_uint(lds_at(vb, off)) ^ sb);
      }
      if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    wave_sync_r();
    if (overlap) rows_put_tail<RPV, NBR>(z, rp, ln, vb);
    fwht_rows<8 * NBR>(z, ln.sg);
    if (!mid) scale = ln.signed_by_lane(rp.inv_sqrt_b * rp.inv_sqrt_b);
  }
#pragma unroll
  for (int e = 0; e < 8 * NBR; ++e) z[e] *= scale;
  if (overlap) {
    rows_put_block<RPV, NBR>(z, rp.n_full - 1, ln, vb);
    rows_overlap<RPV>(rp, ln, vb, inv);
    rows_get_block<RPV, NBR>(z, rp.n_full - 1, ln, vb);
    rows_get_tail<RPV, NBR>(z, rp, ln, vb);
    wave_sync_r();
  }
  // a block past the last one (its transposed reads were arbitrary)
  if (RPV > 1 && !FULL) {
    constexpr int j = NBR - 1;
    const bool none = 128 * (j * RPV + ln.pv) >= rp.D;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[8 * j + i] = none ? 0.f : z[8 * j + i];
  }
}

// Inverse rotation R^T of z, without the final S1 (ts without lane signs):
// blocks in reverse, every pass scaled as it ends.
template <int RPV, int NBR, bool FULL>
__device__ __forceinline__ void rows_inverse(float (&z)[8 * NBR], const RotParams &rp,
                                             const uint16_t *ts, float *vb, const RowsLane<RPV> &ln) {
  if (rp.passes == 0) return;
  const float inv = ln.signed_by_lane(rp.inv_sqrt_b);
  const bool overlap = !FULL && rp.overlap;
  for (int pass = 0; pass < rp.passes; ++pass) {
    if (overlap) {
      rows_put_block<RPV, NBR>(z, rp.n_full - 1, ln, vb);
      rows_put_tail<RPV, NBR>(z, rp, ln, vb);
      rows_overlap<RPV>(rp, ln, vb, inv);
      rows_get_block<RPV, NBR>(z, rp.n_full - 1, ln, vb);
    }
    // the tail's values stay in the buffer (its registers are transformed
    // with the rest and read again below)
    fwht_rows<8 * NBR>(z, ln.sg);
#pragma unroll
    for (int e = 0; e < 8 * NBR; ++e) z[e] *= inv;
    if (overlap) rows_get_tail<RPV, NBR>(z, rp, ln, vb);
    wave_sync_r();
    if (pass + 1 == rp.passes) break;
    // inverse transpose (the tail's entries point at themselves)
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      const int c = 128 * (j * RPV + ln.pv) + 8 * ln.r;
      const uint4 t8 = *reinterpret_cast<const uint4 *>(ts + c);
      const uint32_t tw[4] = {t8.x, t8.y, t8.z, t8.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t off = (tw[i >> 1] >> (16 * (i & 1))) & 0x7fffu;
        const uint32_t sb = (i & 1) ? tw[i >> 1] & 0x80000000u : (tw[i >> 1] << 16) & 0x80000000u;
        if (FULL || j + 1 < NBR || c + i < rp.D)
          lds_at(vb, off) = __uint_as_float(__float_as_uint(z[8 * j + i]) ^ sb);
      }
    }
    wave_sync_r();
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      if (FULL || j + 1 < NBR || j * RPV + ln.pv < rp.n_full) {
        const float *p = vb + 128 * (j * RPV + ln.pv) + 8 * ln.r;
        const float4 a = *reinterpret_cast<const float4 *>(p), d = *reinterpret_cast<const float4 *>(p + 4);
        z[8 * j] = a.x;
        z[8 * j + 1] = a.y;
        z[8 * j + 2] = a.z;
        z[8 * j + 3] = a.w;
        z[8 * j + 4] = d.x;
        z[8 * j + 5] = d.y;
        z[8 * j + 6] = d.z;
        z[8 * j + 7] = d.w;
      }
    }
    if (overlap) rows_get_tail<RPV, NBR>(z, rp, ln, vb);
    wave_sync_r();
  }
}

// Rows per vector and blocks per row of a dimension, by its number of blocks
// (full ones and the tail): few rows while a lane holds at most 32
// coordinates (reductions and scalar steps are per row), then four.  Always
// more than RPV (NBR - 1) blocks, so that the blocks j < NBR - 1 of every row
// are full and only the last one can be the tail or past the end; kernels have
// an instantiation (FULL) for D = 128 RPV NBR, where none is.  D = 384 (EXACT)
// has an arrangement of its own: with two rows of two blocks one of the four
// is past the end, and its last blocks are read and written element by element
// (4-bit encode with a 2-bit second stage, us: 8,000 x 384 33.2, 15.7 here; 400,000
// 1,062, 350).
#define RSLM_ROWS_SWITCH(NBT, EXACT, CALL)  \
  if ((NBT) <= 1) CALL(1, 1)         \
  else if ((NBT) <= 2) CALL(1, 2)    \
  else if ((NBT) == 3 && (EXACT)) CALL(1, 3) \
  else if ((NBT) <= 4) CALL(2, 2)    \
  else if ((NBT) <= 6) CALL(2, 3)    \
  else if ((NBT) <= 8) CALL(2, 4)    \
  else if ((NBT) <= 12) CALL(4, 3)   \
  else if ((NBT) <= 16) CALL(4, 4)   \
  else if ((NBT) <= 20) CALL(4, 5)   \
  else if ((NBT) <= 24) CALL(4, 6)   \
  else if ((NBT) <= 28) CALL(4, 7)   \
  else CALL(4, 8)

// Arrangements that are only used where D = 128 RPV NBR.
constexpr bool rows_only_full(int rpv, int nbr) { return rpv == 1 && nbr != 2; }
inline bool rows_ok(const RotParams &rp) { return rp.B == 128 && rp.D >= 128 && rp.D <= kMaxDim; }
inline int rows_blocks(const RotParams &rp) { return rp.n_full + (rp.overlap ? 1 : 0); }

// Workgroups of 256 threads of a kernel whose workgroups stride over `groups`
// units of work, with shm bytes of dynamic LDS: as many as are resident at
// once, so that tables are filled once per workgroup, and up to 8 times that
// while each still has about 8 units to stride over: workgroups that start
// later even out the ends.  Measured (us; 1, 2, 4, 8 times the resident
// workgroups): two-stage encode of 524,288 x 768 1,177, 1,140, 1,095, 1,071 (85
// units each at 1 x); 2-bit encode of 65,536 x 1,024 168, 164, 162, 161 (15);
// 4-bit with SQ8 of 65,536 x 768 130, 132, 134, 140 (11).  Up to `one_each` units
// per resident workgroup, one each: records without a vector (list padding) make
// units uneven, which only starting them one by one evens out (two-stage encode
// of 20,000 x 512 34.7 against 36.4, 4-bit of 38,244 x 256 19.4 against 20.3).
// The resident count of a kernel is kept for the last shm asked for (a query
// takes longer than a small launch).
template <auto kKernel>
inline unsigned rows_grid(size_t shm, int64_t groups, int one_each = 3) {
  static std::atomic<uint64_t> kept{0};   // shm << 16 | workgroups per CU
  int cus = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 256;
  const uint64_t k = kept.load(std::memory_order_relaxed);
  int per_cu = int(k & 0xffff);
  if (per_cu == 0 || (k >> 16) != shm) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kKernel),
                                                     256, shm) != hipSuccess || per_cu < 1)
      per_cu = 2;
    kept.store(uint64_t(shm) << 16 | uint64_t(per_cu), std::memory_order_relaxed);
  }
  const int64_t n = int64_t(per_cu) * cus;
  if (groups <= one_each * n) return unsigned(std::max<int64_t>(1, groups));
  const int64_t over = std::min<int64_t>(8, std::max<int64_t>(1, (groups / n + 4) / 8));
  return unsigned(std::max<int64_t>(1, std::min(groups, n * over)));
}

}  // namespace rslm

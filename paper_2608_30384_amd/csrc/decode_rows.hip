// Decompress on 16-lane rows (rows_dev.h), for D >= 128.
#include "rows_dev.h"

namespace rslm {

// x~ = g^ (c + R^T s^ C[code]): a lane decodes the 8 coordinates of each of its
// blocks from the packed bytes of one group of the tile layout, the rotation
// back runs in registers (rows_inverse), and the centre is added on output.
// 65,536 x 768: 80 us alone in its call, 65 us among others (3.5 TB/s), against
// 294 us for one wavefront per record through LDS, whose butterfly rounds each
// read and wrote every element.
template <int RPV, int NBR, int BITS, bool LITE, bool FULL>
__global__ void __launch_bounds__(256, NBR <= 4 ? 4 : 2) k_decode_rows(
    const uint8_t *__restrict__ codes, const uint32_t *__restrict__ scales, int64_t n,
    const int32_t *__restrict__ rec_list, const float *__restrict__ cen, int nlist,
    float *__restrict__ out, RotParams rp, CodecParams cp) {
  constexpr int VPW = 4 / RPV;
  constexpr int G = BITS == 1 ? 4 : BITS == 2 ? 2 : 1;
  constexpr int W = BITS == 3 ? 3 : 4;
  constexpr uint32_t kMask = (1u << W) - 1u;
  extern __shared__ float4 lds4[];
  __shared__ __align__(16) uint32_t s1[kSignWords];
  __shared__ float cbs[16], cb8[LITE ? 16 : 1];
  __shared__ float4 cb4[G > 1 ? 16 : 1];
  const int D = rp.D;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int stride = rows_stride(D);
  float *lds = reinterpret_cast<float *>(lds4);
  uint16_t *ts = reinterpret_cast<uint16_t *>(lds + 4 * VPW * stride);
  RowsTs<128 * RPV * NBR> tload;
  tload.load(rp);
  RowsSigns signs;
  signs.load(rp);
  if (tid < 16) {
    if (G == 1) cbs[tid] = cp.cb[tid];
    if (G == 2) cb4[tid] = make_float4(cp.cb[2 * tid], cp.cb[2 * tid + 1], 0.f, 0.f);
    if (G == 4) cb4[tid] = make_float4(cp.cb[4 * tid], cp.cb[4 * tid + 1], cp.cb[4 * tid + 2], cp.cb[4 * tid + 3]);
    if (LITE) cb8[tid] = cp.cb_lead[tid & 7];
  }
  tload.store(ts, rp, signs, false);
  signs.fill(s1, rp);
  __syncthreads();
  const int64_t n_groups = (n + VPW - 1) / VPW;
  for (int64_t grp = int64_t(blockIdx.x) * 4 + wid; grp < n_groups; grp += int64_t(gridDim.x) * 4) {
    int olane = lane;   // opaque: nothing derived from it is kept across the loop
    asm volatile("" : "+v"(olane));
    const RowsLane<RPV> ln(olane);
    const int r = ln.r, pv = ln.pv;
    float *vb = lds + (wid * VPW + ln.vslot) * stride;
    const int64_t rec = grp * VPW + ln.vslot;
    if (rec >= n) continue;   // the rows of this vector sit out; no workgroup barrier follows
    const uint32_t sc = scales[rec];
    const float sh = dec_ue7m9(sc & 0xffffu);
    const float gh = cp.global ? dec_ue4m12(sc >> 16) : 1.f;
    int L = -1;
    if (cen) {
      L = rec_list[rec];
      if (L < 0 || L >= nlist) L = -1;
    }
    // the lane's groups q = 16 b + r of the tile layout (see store in the encoder)
    const uint8_t *tile = codes + (rec >> 4) * int64_t(cp.tile_bytes) + int(rec & 15) * 16;
    const int q_end = cp.d_pad >> 3;
    uint32_t word[NBR];
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      const int q = min(16 * (j * RPV + pv) + r, q_end - 1);
      const int off = (q >> 2) * BITS;
      const uint8_t *p = tile + 256 * (q & 3);
      if (BITS == 4) word[j] = reinterpret_cast<const U32u *>(p + (off >> 4) * 1024 + (off & 15))->v;
      else if (BITS == 2) word[j] = reinterpret_cast<const U16u *>(p + (off >> 4) * 1024 + (off & 15))->v;
      else if (BITS == 1) word[j] = p[(off >> 4) * 1024 + (off & 15)];
      else
        word[j] = uint32_t(p[(off >> 4) * 1024 + (off & 15)]) |
                  (uint32_t(p[((off + 1) >> 4) * 1024 + ((off + 1) & 15)]) << 8) |
                  (uint32_t(p[((off + 2) >> 4) * 1024 + ((off + 2) & 15)]) << 16);
    }
    float z[8 * NBR];
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      float v[8];
      if constexpr (G == 1) {
        const bool lb = LITE && j == 0 && pv == 0 && r < cp.lead / 8;
        float *cbb = lb ? cb8 : cbs;   // bit 3 of a leading code is a scale bit
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = cbb[(word[j] >> (W * i)) & (lb ? 7u : kMask)];
      } else if constexpr (G == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float4 c = cb4[(word[j] >> (4 * k)) & 15u];
          v[2 * k] = c.x;
          v[2 * k + 1] = c.y;
        }
      } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const float4 c = cb4[(word[j] >> (4 * k)) & 15u];
          v[4 * k] = c.x;
          v[4 * k + 1] = c.y;
          v[4 * k + 2] = c.z;
          v[4 * k + 3] = c.w;
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) z[8 * j + i] = sh * v[i];
      if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    rows_inverse<RPV, NBR, FULL>(z, rp, ts, vb, ln);
    const int c0 = 128 * pv + 8 * r;
    const float *cr = L >= 0 ? cen + int64_t(L) * D : nullptr;
    float *orow = out + rec * D;
#pragma unroll
    for (int j = 0; j < NBR; ++j) {
      const int c = c0 + 128 * RPV * j;
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = z[8 * j + i];
      rows_flip(v, s1, j * RPV + pv, r);
      if (j + 1 < NBR || FULL) {
        float b[8] = {};
        if (cr) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const Float4u w = *reinterpret_cast<const Float4u *>(cr + c + 4 * h);
            b[4 * h] = w.x;
            b[4 * h + 1] = w.y;
            b[4 * h + 2] = w.z;
            b[4 * h + 3] = w.w;
          }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
          *reinterpret_cast<Float4u *>(orow + c + 4 * h) =
              Float4u{gh * (b[4 * h] + v[4 * h]), gh * (b[4 * h + 1] + v[4 * h + 1]),
                      gh * (b[4 * h + 2] + v[4 * h + 2]), gh * (b[4 * h + 3] + v[4 * h + 3])};
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (c + i < D) orow[c + i] = gh * ((cr ? cr[c + i] : 0.f) + v[i]);
      }
      if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

struct DecodeCall {
  const rslm_plan *p;
  const uint8_t *codes;
  const uint32_t *scales;
  int64_t n;
  const int32_t *rec_list;
  const float *cen;
  int nlist;
  float *out;
  hipStream_t s;
};

template <int RPV, int NBR, int BITS, bool LITE, bool FULL>
static void launch_decode_one(const DecodeCall &c) {
  const size_t shm = size_t(16 / RPV) * rows_stride(c.p->rot.D) * 4 + 128 * RPV * NBR * 2;
  constexpr auto kernel = k_decode_rows<RPV, NBR, BITS, LITE, FULL>;
  const int64_t groups = (c.n + 16 / RPV - 1) / (16 / RPV);
  hipLaunchKernelGGL(kernel, dim3(rows_grid<kernel>(shm, groups)), dim3(256), shm, c.s, c.codes,
                     c.scales, c.n, c.rec_list, c.cen, c.nlist, c.out, c.p->rot, c.p->codec);
}

template <int BITS, bool LITE>
static void launch_decode_t(const DecodeCall &c) {
  const int D = c.p->rot.D;
#define RSLM_DECODE_ROWS(RPV, NBR)                                                     \
  {                                                                                    \
    if (rows_only_full(RPV, NBR) || D == 128 * RPV * NBR)                              \
      launch_decode_one<RPV, NBR, BITS, LITE, true>(c);                                \
    else                                                                               \
      launch_decode_one<RPV, NBR, BITS, LITE, rows_only_full(RPV, NBR)>(c);            \
  }
  const int nbt = rows_blocks(c.p->rot);
  RSLM_ROWS_SWITCH(nbt, D == 384, RSLM_DECODE_ROWS)
#undef RSLM_DECODE_ROWS
}

bool launch_decode_rows(const rslm_plan *p, const uint8_t *codes, const uint32_t *scales, int64_t n,
                        const int32_t *rec_list, const float *cen, int nlist, float *out,
                        hipStream_t s) {
  if (!rows_ok(p->rot)) return false;
  const DecodeCall c{p, codes, scales, n, rec_list, cen, nlist, out, s};
  switch (p->codec.bits) {
    case 4: p->codec.lead > 0 ? launch_decode_t<4, true>(c) : launch_decode_t<4, false>(c); break;
    case 3: launch_decode_t<3, false>(c); break;
    case 2: launch_decode_t<2, false>(c); break;
    default: launch_decode_t<1, false>(c);
  }
  return true;
}

}  // namespace rslm

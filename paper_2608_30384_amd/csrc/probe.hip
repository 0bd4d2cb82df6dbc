// IVF routing: assignment of vectors to their nearest partition centre and
// probing of the partitions with the largest dot product with a query
// (paper, Section "End-to-End Comparison", Setup: Euclidean partitions,
// routing by the dot product with the centres).
//
// Both modes are a dense [n x D] x [D x nlist] contraction in float32 on the
// matrix cores (v_mfma_f32_16x16x4_f32).  Probing writes the dots (64 x 64
// output tiles) and selects the top-nprobe per row.  Assignment keeps a
// running (distance, id) minimum per row across all centre tiles (128 x 128
// output tiles), never writing the product; rows that are not whole 16-byte
// runs take a vector-ALU tile (64 x 64, 4 x 4 outputs per thread) instead.
#include <mutex>

#include "rslm_internal.h"
#include "select_dev.h"

namespace rslm {

constexpr int kTM = 64, kTN = 64, kTK = 16;

__global__ void k_row_norms(const float *__restrict__ c, int n, int D, float *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= n) return;
  float s = 0.f;
  for (int i = lane; i < D; i += 64) {
    const float v = c[int64_t(row) * D + i];
    s += v * v;
  }
  s = wave_sum(s);
  if (lane == 0) out[row] = s;
}

// Loads a 64-row x 16-column slice of a row-major matrix (rows r0.., cols
// k0..) transposed into lds[16][64 + 4] (zero outside the matrix).
__device__ __forceinline__ void load_slice(const float *__restrict__ m, int64_t rows, int D,
                                           int64_t r0, int k0, float (*lds)[kTM + 4]) {
  // 256 threads x 4 elements
  const int t = threadIdx.x;
  const int r = t >> 2;          // 0..63
  const int kk = (t & 3) * 4;    // 0,4,8,12
  const int64_t gr = r0 + r;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int gk = k0 + kk + e;
    float v = 0.f;
    if (gr < rows && gk < D) v = m[gr * D + gk];
    lds[kk + e][r] = v;
  }
}

// acc[i][j] = sum_k A[r0 + ty*4 + i][k] * B[c0 + tx*4 + j][k]
__device__ __forceinline__ void tile_product(const float *__restrict__ A, int64_t n,
                                             const float *__restrict__ Bm, int nb, int D,
                                             int64_t r0, int c0, float (*As)[kTM + 4],
                                             float (*Bs)[kTM + 4], float acc[4][4]) {
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  for (int k0 = 0; k0 < D; k0 += kTK) {
    load_slice(A, n, D, r0, k0, As);
    load_slice(Bm, nb, D, c0, k0, Bs);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < kTK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(256) k_assign(const float *__restrict__ x, int64_t n, int D,
                                                const float *__restrict__ cen, int nlist,
                                                const float *__restrict__ cnorm,
                                                int32_t *__restrict__ out_ids,
                                                float *__restrict__ out_d) {
  __shared__ float As[kTK][kTM + 4];
  __shared__ float Bs[kTK][kTM + 4];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int64_t r0 = int64_t(blockIdx.x) * kTM;
  float best[4];
  int bid[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    best[i] = 3.4e38f;
    bid[i] = 0x7fffffff;
  }
  float acc[4][4];
  for (int c0 = 0; c0 < nlist; c0 += kTN) {
    tile_product(x, n, cen, nlist, D, r0, c0, As, Bs, acc);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = c0 + tx * 4 + j;
      if (c < nlist) {
        const float cn = cnorm[c];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = cn - 2.f * acc[i][j];   // ||c||^2 - 2 <x, c>
          if (v < best[i]) {                      // columns visited in increasing order
            best[i] = v;
            bid[i] = c;
          }
        }
      }
    }
  }
  // reduce over the 16 threads (tx) sharing each row: lexicographic (value, id)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    for (int off = 8; off >= 1; off >>= 1) {
      const float ov = __shfl_xor(best[i], off, 64);
      const int oi = __shfl_xor(bid[i], off, 64);
      if (ov < best[i] || (ov == best[i] && oi < bid[i])) {
        best[i] = ov;
        bid[i] = oi;
      }
    }
  }
  if (tx == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t r = r0 + ty * 4 + i;
      if (r < n) {
        out_ids[r] = bid[i];
        if (out_d) {
          float xx = 0.f;
          for (int k = 0; k < D; ++k) {
            const float v = x[r * D + k];
            xx += v * v;
          }
          out_d[r] = xx + best[i];
        }
      }
    }
  }
}

// Probe dots on the matrix cores (v_mfma_f32_16x16x4_f32, full float32):
// a 32 x 32 output tile per 256-thread workgroup, each wavefront one 16 x 16
// MFMA tile, K staged through LDS in slabs of 32.
typedef float floatx4_t __attribute__((ext_vector_type(4)));
constexpr int kMT = 32, kMK = 32;

__device__ __forceinline__ void stage32(const float *__restrict__ m, int64_t rows, int D,
                                        int64_t r0, int k0, float (*lds)[kMK + 1]) {
  const int t = threadIdx.x;        // 256 threads x 4 elements = 32 rows x 32 k
  const int r = t >> 3;
  const int kk = (t & 7) * 4;
  const int64_t gr = r0 + r;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int gk = k0 + kk + e;
    lds[r][kk + e] = (gr < rows && gk < D) ? m[gr * D + gk] : 0.f;
  }
}

__global__ void __launch_bounds__(256) k_dots_mfma(const float *__restrict__ x, int64_t n, int D,
                                                   const float *__restrict__ cen, int nlist,
                                                   float *__restrict__ dots) {
  __shared__ float As[kMT][kMK + 1];
  __shared__ float Bs[kMT][kMK + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r0 = int64_t(blockIdx.y) * kMT;
  const int c0 = blockIdx.x * kMT;
  const int wr = (wave >> 1) * 16, wc = (wave & 1) * 16;   // this wave's 16 x 16 block
  const int ml = lane & 15, kl = lane >> 4;
  floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < D; k0 += kMK) {
    stage32(x, n, D, r0, k0, As);
    stage32(cen, nlist, D, c0, k0, Bs);
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < kMK; ks += 4) {
      const float a = As[wr + ml][ks + kl];     // A[m][k]: lane -> (m = lane % 16, k = lane / 16)
      const float b = Bs[wc + ml][ks + kl];     // B[k][n]: lane -> (k = lane / 16, n = lane % 16)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
    }
    __syncthreads();
  }
  // lane holds C[4 (lane / 16) + i][lane % 16]
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = r0 + wr + 4 * kl + i;
    const int c = c0 + wc + ml;
    if (r < n && c < nlist) dots[r * nlist + c] = acc[i];
  }
}

// Assignment on the matrix cores (v_mfma_f32_16x16x4f32, full float32) for
// D a multiple of 4 and 16-byte aligned operands.  A workgroup owns 128 rows
// and walks the centres in tiles of 128 (tile128), in increasing order.  After
// each centre tile the distances ||c||^2 - 2 <x, c> update a (distance, id)
// minimum per row and lane (centres visited in increasing order with a
// strict comparison, so the smallest id wins a tie); lanes and the two
// wavefronts sharing a row are merged lexicographically at the end.
constexpr int kAM = 128, kAN = 128, kAK = 32, kAS = kAK + 4;

__device__ __forceinline__ float4 ld4_or_zero(const float *p, bool in) {
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (in) v = *reinterpret_cast<const float4 *>(p);
  return v;
}

// The 128 x 128 product tile of rows (staging offsets aoff, four per thread)
// and centres [c0, c0 + 128) on the matrix cores: four wavefronts of 4 x 4
// v_mfma_f32_16x16x4f32 tiles, k staged through LDS in slabs of 32 (rows
// padded to 36 floats, so that the 16-byte operand reads of eight consecutive
// lanes fall on distinct banks) with the next slab prefetched into registers.
// Within a half slab of 16 both operands use the same permutation of k: lane
// (m, h) supplies k = 4 h + t to MFMA step t, so one 16-byte read covers four
// steps.  Lane (m, h) of wavefront (wr, wc) ends with C[4 h + e][m] of tile
// (i, j): row wr + 16 i + 4 h + e, centre c0 + wc + 16 j + m.
__device__ __forceinline__ void tile128(const float *__restrict__ x, const int64_t (&aoff)[4],
                                        int D, const float *__restrict__ cen, int nlist, int c0,
                                        float (*As)[kAS], float (*Bs)[kAS],
                                        floatx4_t (&acc)[4][4]) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = (wave >> 1) * 64, wc = (wave & 1) * 64;
  const int m = lane & 15, h = lane >> 4;
  const int srow = tid >> 3, scol = (tid & 7) * 4;
  const int nslab = (D + kAK - 1) / kAK;
  int64_t boff[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) boff[u] = int64_t(min(c0 + srow + 32 * u, nlist - 1)) * D + scol;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  float4 pa[4], pb[4];
  const bool in0 = scol < D;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    pa[u] = ld4_or_zero(x + aoff[u], in0);
    pb[u] = ld4_or_zero(cen + boff[u], in0);
  }
  for (int sl = 0; sl < nslab; ++sl) {
    __syncthreads();   // the previous slab's operand reads are done
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      *reinterpret_cast<float4 *>(&As[srow + 32 * u][scol]) = pa[u];
      *reinterpret_cast<float4 *>(&Bs[srow + 32 * u][scol]) = pb[u];
    }
    __syncthreads();
    if (sl + 1 < nslab) {
      const int kn = (sl + 1) * kAK;
      const bool in = kn + scol < D;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        pa[u] = ld4_or_zero(x + aoff[u] + kn, in);
        pb[u] = ld4_or_zero(cen + boff[u] + kn, in);
      }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      float4 a4[4], b4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a4[i] = *reinterpret_cast<const float4 *>(&As[wr + 16 * i + m][16 * s + 4 * h]);
        b4[i] = *reinterpret_cast<const float4 *>(&Bs[wc + 16 * i + m][16 * s + 4 * h]);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float av = t == 0 ? a4[i].x : t == 1 ? a4[i].y : t == 2 ? a4[i].z : a4[i].w;
            const float bv = t == 0 ? b4[j].x : t == 1 ? b4[j].y : t == 2 ? b4[j].z : b4[j].w;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[i][j], 0, 0, 0);
          }
    }
  }
}

__global__ void __launch_bounds__(256) k_assign_mfma(const float *__restrict__ x, int64_t n,
                                                     int D, const float *__restrict__ cen,
                                                     int nlist, const float *__restrict__ cnorm,
                                                     int32_t *__restrict__ out_ids,
                                                     float *__restrict__ out_d) {
  __shared__ float As[kAM][kAS];
  __shared__ float Bs[kAN][kAS];
  __shared__ float red_v[kAM];
  __shared__ int32_t red_i[kAM];
  __shared__ float xx_s[kAM];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = (wave >> 1) * 64, wc = (wave & 1) * 64;
  const int m = lane & 15, h = lane >> 4;
  const int64_t r0 = int64_t(blockIdx.x) * kAM;
  // staging: thread t moves the float4s (row t / 8 + 32 u, column 4 (t % 8)),
  // u = 0..3, of a 128 x 32 slab; rows past the end are clamped (their
  // products are computed and never used)
  const int srow = tid >> 3, scol = (tid & 7) * 4;
  int64_t aoff[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t r = r0 + srow + 32 * u;
    aoff[u] = (r < n ? r : n - 1) * D + scol;
  }
  float best[16];
  int32_t bid[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    best[r] = 3.4e38f;
    bid[r] = 0x7fffffff;
  }
  for (int c0 = 0; c0 < nlist; c0 += kAN) {
    floatx4_t acc[4][4];
    tile128(x, aoff, D, cen, nlist, c0, As, Bs, acc);
    // lane holds C[4 h + e][m] of each 16 x 16 tile: row wr + 16 i + 4 h + e,
    // centre c0 + wc + 16 j + m
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = c0 + wc + 16 * j + m;
      const float cn = c < nlist ? cnorm[c] : __builtin_inff();
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v = cn - 2.f * acc[i][j][e];   // ||c||^2 - 2 <x, c>
          if (v < best[4 * i + e]) {
            best[4 * i + e] = v;
            bid[4 * i + e] = c;
          }
        }
    }
  }
  // merge the 16 lanes (m) holding the same rows: lexicographic (value, id)
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    for (int off = 1; off < 16; off <<= 1) {
      const float ov = __shfl_xor(best[r], off, 64);
      const int oi = __shfl_xor(bid[r], off, 64);
      if (ov < best[r] || (ov == best[r] && oi < bid[r])) {
        best[r] = ov;
        bid[r] = oi;
      }
    }
  }
  if (wc && m == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        red_v[wr + 16 * i + 4 * h + e] = best[4 * i + e];
        red_i[wr + 16 * i + 4 * h + e] = bid[4 * i + e];
      }
  }
  if (out_d) {   // ||x||^2 of the workgroup's rows: 32 rows per wavefront
    for (int rr = 0; rr < 32; ++rr) {
      const int rl = wave * 32 + rr;
      const int64_t row = r0 + rl < n ? r0 + rl : n - 1;
      float s = 0.f;
      for (int k = 4 * lane; k < D; k += 256) {
        const float4 v = *reinterpret_cast<const float4 *>(x + row * D + k);
        s += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
      }
      s = wave_sum(s);
      if (lane == 0) xx_s[rl] = s;
    }
  }
  __syncthreads();
  if (wc || m) return;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int rl = wr + 16 * i + 4 * h + e;
      float v = best[4 * i + e];
      int32_t id = bid[4 * i + e];
      const float ov = red_v[rl];
      const int32_t oi = red_i[rl];
      if (ov < v || (ov == v && oi < id)) {
        v = ov;
        id = oi;
      }
      const int64_t r = r0 + rl;
      if (r < n) {
        out_ids[r] = id;
        if (out_d) out_d[r] = xx_s[rl] + v;
      }
    }
}

// ------------------------------------------------ assignment on split float16
// Large assignments: the float32 matrix instructions are the limit (157
// TFLOP/s; k_assign_mfma runs at 125), so each operand is split into two
// float16 halves, v s = hi + lo with s a power of two per row that puts the
// row's largest magnitude in [2^14, 2^15), and <x, c> is accumulated in
// float32 as hi hi + hi lo + lo hi on v_mfma_f32_16x16x32_f16 (16 times the
// float32 rate per product).  hi + lo carries 22 to 23 significant bits (and
// never less than 2^-39 of the row's largest element); what is dropped, lo lo,
// is below 2^-22 of each product.  Both are smaller than the roundings of the
// float32 sum, which has D / 32 steps here against D / 4 there.  Error of the
// distances against float64 (2-norm, relative): 524,288 x 768 by 4,096 1.7e-7,
// float32 kernel 8.9e-7; 100,000 x 1,447 by 3,000 2.2e-7 and 1.5e-6; 524,288 x
// 100 by 4,096 1.5e-7 and 4.7e-7.
//
// A workgroup of eight wavefronts owns 256 rows of x and walks its share of
// the centres in tiles of 256: with both sides at 256 each operand is read
// from L2 once per 256 rows of the other, which is what the matrix cores leave
// time for.  The centres are split once per call (k_split_centres), the rows
// of x as they are staged (they are too many to keep).  k goes through LDS in
// slabs of 32, two buffers, one barrier per slab.  Centres are the M side, so
// a lane holds 32 centres of each of four rows and keeps four running minima.
// 1,048,576 x 768 by 4,096: 52.6 ms on the float32 kernel, 20.2 ms here (327
// TFLOP/s of distances, 981 TFLOP/s of float16 products; a large bf16 library
// product runs at 1,370 on the same card).  The same tiles with the centres
// staged through registers 30.6 ms, with two slabs of both operands in
// registers 38.8 ms (spills).
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
constexpr int kSpM = 256, kSpN = 256, kSpK = 32, kSpThreads = 512;
constexpr int kSpRow = 4 * kSpK;       // bytes per LDS row: hi, then lo
constexpr int kWaitVm0 = 0x0F70;       // s_waitcnt vmcnt(0), the other counters free
constexpr int kSlowRow = int(0x80000000);   // id of a row left to k_assign_finish

struct __attribute__((packed, aligned(4))) F4u {
  float x, y, z, w;
};

// Power of two s with m s in [2^14, 2^15) (m > 0 finite; the exponent is
// clamped where s would not be a normal number).
__device__ __forceinline__ float split_scale(float m) {
  if (!(m > 0.f) || !(m < __builtin_inff())) return 1.f;
  return ldexpf(1.f, max(-126, min(126, 14 - ilogbf(m))));
}

// One wavefront per centre (nlist rounded up to whole tiles): ||c||^2 (summed
// in float64; +inf past nlist, so padding is never nearest), -2 / s, and the
// halves, slab by slab (32 hi, then 32 lo, zero past D).
__global__ void __launch_bounds__(256) k_split_centres(const float *__restrict__ cen, int nlist, int D,
                                                       int n_slab, float *__restrict__ cnorm,
                                                       float *__restrict__ cmul,
                                                       _Float16 *__restrict__ split) {
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
  const float *row = cen + int64_t(c) * D;
  const bool in = c < nlist;
  double sum = 0.0;
  float m = 0.f;
  for (int i = lane; in && i < D; i += 64) {
    const float v = row[i];
    sum += double(v) * double(v);
    m = fmaxf(m, fabsf(v));
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  const float sc = split_scale(wave_max(m));
  if (lane == 0) {
    cnorm[c] = in ? float(sum) : __builtin_inff();
    cmul[c] = -2.f / sc;
  }
  _Float16 *out = split + int64_t(c) * n_slab * (2 * kSpK);
  for (int i = lane; i < n_slab * kSpK; i += 64) {
    const float v = (in && i < D) ? row[i] * sc : 0.f;
    const _Float16 h = static_cast<_Float16>(v);
    out[(i / kSpK) * (2 * kSpK) + i % kSpK] = h;
    out[(i / kSpK) * (2 * kSpK) + kSpK + i % kSpK] = static_cast<_Float16>(v - static_cast<float>(h));
  }
}

// Workgroup (rows, share): nearest of the centres [tiles t0, t1) of 256 for
// 256 rows; (distance without ||x||^2, id) to best_v / best_i at [share][row].
__global__ void __launch_bounds__(kSpThreads, 2) k_assign_split(
    const float *__restrict__ x, int64_t n, int D, int n_slab, const float *__restrict__ cnorm,
    const float *__restrict__ cmul, const _Float16 *__restrict__ split, int n_tiles,
    int tiles_per_share, float *__restrict__ best_v, int32_t *__restrict__ best_i) {
  // rows of 128 bytes (32 hi, 32 lo): x, then centres; the eight 16-byte units
  // of row r are stored at unit ^ (r % 8), which spreads a column of units
  // over the banks without padding (the centres are written by lanes in order)
  __shared__ __align__(128) uint8_t lds[2][(kSpM + kSpN) * kSpRow];
  __shared__ float xscale[kSpM];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, h = lane >> 4;
  const int wx = (wave & 3) * 64, wc = (wave >> 2) * 128;   // this wave's rows and centres
  const int64_t r0 = int64_t(blockIdx.x) * kSpM;
  const int t0 = blockIdx.y * tiles_per_share, t1 = min(n_tiles, t0 + tiles_per_share);
  // largest magnitude of each row: 32 rows per wavefront, four in flight
  for (int q = 0; q < 32; q += 4) {
    float mx[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = lane; k < D; k += 64) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t r = min(r0 + wave * 32 + q + u, n - 1);
        mx[u] = fmaxf(mx[u], fabsf(x[r * D + k]));
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      mx[u] = wave_max(mx[u]);
      // an infinite row is marked (by a zero scale) and left to k_assign_finish
      if (lane == 0) xscale[wave * 32 + q + u] = mx[u] < __builtin_inff() ? split_scale(mx[u]) : 0.f;
    }
  }
  __syncthreads();
  // Staging, in 16-byte units u < 4 per thread.  x: four coordinates (unit tid
  // % 8) of row tid / 8 + 64 u, through registers and the split.  Centres:
  // straight from memory into LDS, 64 lanes filling eight rows.
  const int srow = tid >> 3, scol = (tid & 7) * 4;
  const float *xrow[4];
  float sc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    xrow[u] = x + min(r0 + srow + 64 * u, n - 1) * D;
    sc[u] = xscale[srow + 64 * u];
  }
  const int xhi = ((((tid & 7) >> 1) ^ (srow & 7)) * 16) + (tid & 1) * 8;   // byte in the row
  const int xlo = (((4 + ((tid & 7) >> 1)) ^ (srow & 7)) * 16) + (tid & 1) * 8;
  float4 pa[4];
  auto load_x = [&](int sl) {
    const int k = sl * kSpK + scol;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (sl * kSpK + kSpK <= D) {   // uniform
        const F4u v = *reinterpret_cast<const F4u *>(xrow[u] + k);
        pa[u] = make_float4(v.x, v.y, v.z, v.w);
      } else {
        pa[u].x = k < D ? xrow[u][min(k, D - 1)] : 0.f;
        pa[u].y = k + 1 < D ? xrow[u][min(k + 1, D - 1)] : 0.f;
        pa[u].z = k + 2 < D ? xrow[u][min(k + 2, D - 1)] : 0.f;
        pa[u].w = k + 3 < D ? xrow[u][min(k + 3, D - 1)] : 0.f;
      }
    }
  };
  auto store_x = [&](int buf) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float v[4] = {pa[u].x * sc[u], pa[u].y * sc[u], pa[u].z * sc[u], pa[u].w * sc[u]};
      half4_t hi, lo;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hi[e] = static_cast<_Float16>(v[e]);
        lo[e] = static_cast<_Float16>(v[e] - static_cast<float>(hi[e]));
      }
      uint8_t *px = &lds[buf][(srow + 64 * u) * kSpRow];
      *reinterpret_cast<half4_t *>(px + xhi) = hi;
      *reinterpret_cast<half4_t *>(px + xlo) = lo;
    }
  };
  // the unit that lands in this lane's place, of row wave * 8 + lane / 8 + 64 u
  const _Float16 *csrc = split + (int64_t(wave * 8 + (lane >> 3)) * n_slab) * (2 * kSpK) +
                         ((lane & 7) ^ (lane >> 3)) * 8;
  auto load_c = [&](int tile, int sl, int buf) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void *)(
              csrc + (int64_t(tile * kSpN + 64 * u) * n_slab + sl) * (2 * kSpK)),
          (__attribute__((address_space(3))) void *)(&lds[buf][(kSpM + wave * 8 + 64 * u) * kSpRow]),
          16, 0, 0);
  };
  floatx4_t acc[8][4];
  float best[4], inv[4];
  int32_t bid[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    best[j] = 3.4e38f;
    bid[j] = 0x7fffffff;
    const float s = xscale[wx + 16 * j + m];
    inv[j] = s > 0.f ? 1.f / s : 0.f;
  }
  // Slabs in one sequence over the tiles.  While slab s is multiplied, the
  // centres of slab s + 1 go to LDS, the coordinates of x of slab s + 1 (loaded
  // during s - 1) are split and stored, and those of slab s + 2 are loaded.
  const int total = (t1 - t0) * n_slab;
  const int hi_unit = (h ^ (m & 7)) * 16, lo_unit = ((4 + h) ^ (m & 7)) * 16;
  int tile = t0, sl = 0;
  load_c(t0, 0, 0);
  load_x(0);
  store_x(0);
  load_x(n_slab > 1 ? 1 : 0);
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __syncthreads();
  for (int it = 0; it < total; ++it) {
    const int buf = it & 1;
    const bool last = sl + 1 == n_slab;
    if (it + 1 < total) {
      load_c(last ? tile + 1 : tile, last ? 0 : sl + 1, buf ^ 1);
      store_x(buf ^ 1);
      load_x((sl + 2) % n_slab);   // past the end: not stored
    }
    if (sl == 0) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    }
    const uint8_t *px = &lds[buf][(wx + m) * kSpRow];
    const uint8_t *pc = &lds[buf][(kSpM + wc + m) * kSpRow];
    half8_t xh[4], xl[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      xh[j] = *reinterpret_cast<const half8_t *>(px + 16 * j * kSpRow + hi_unit);
      xl[j] = *reinterpret_cast<const half8_t *>(px + 16 * j * kSpRow + lo_unit);
    }
    // a slab's products are summed from zero and then added once: the float32
    // accumulator is rounded D / 32 times, not 3 D / 32
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const half8_t ch = *reinterpret_cast<const half8_t *>(pc + 16 * i * kSpRow + hi_unit);
      const half8_t cl = *reinterpret_cast<const half8_t *>(pc + 16 * i * kSpRow + lo_unit);
      floatx4_t t[4];
      const floatx4_t zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(cl, xh[j], zero, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ch, xl[j], t[j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ch, xh[j], t[j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] += t[j];
    }
    if (last) {
      // lane (m, h) holds centres c0 + wc + 16 i + 4 h + e of rows wx + 16 j + m
      const int c0 = tile * kSpN + wc + 4 * h;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float4 cn = *reinterpret_cast<const float4 *>(cnorm + c0 + 16 * i);
        const float4 cm = *reinterpret_cast<const float4 *>(cmul + c0 + 16 * i);
        const float cna[4] = {cn.x, cn.y, cn.z, cn.w}, cma[4] = {cm.x, cm.y, cm.z, cm.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float v = fmaf(acc[i][j][e], cma[e] * inv[j], cna[e]);   // ||c||^2 - 2 <x, c>
            if (v < best[j]) {   // centres visited in increasing order
              best[j] = v;
              bid[j] = c0 + 16 * i + e;
            }
          }
      }
      ++tile;
      sl = 0;
    } else {
      ++sl;
    }
    __builtin_amdgcn_s_waitcnt(kWaitVm0);   // the centres are in LDS
    __syncthreads();
  }
  // merge the four lanes and the two wavefronts holding a row: lexicographic
  // (value, id)
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
      const float ov = __shfl_xor(best[j], off, 64);
      const int oi = __shfl_xor(bid[j], off, 64);
      if (ov < best[j] || (ov == best[j] && oi < bid[j])) {
        best[j] = ov;
        bid[j] = oi;
      }
    }
  float *red_v = reinterpret_cast<float *>(lds[0]);   // the last slab was multiplied before a barrier
  int32_t *red_i = reinterpret_cast<int32_t *>(red_v + kSpM);
  if (wave >= 4 && h == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      red_v[wx + 16 * j + m] = best[j];
      red_i[wx + 16 * j + m] = bid[j];
    }
  }
  __syncthreads();
  if (wave >= 4 || h) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int rl = wx + 16 * j + m;
    if (r0 + rl >= n) continue;
    if (red_v[rl] < best[j] || (red_v[rl] == best[j] && red_i[rl] < bid[j])) {
      best[j] = red_v[rl];
      bid[j] = red_i[rl];
    }
    const int64_t at = int64_t(blockIdx.y) * n + r0 + rl;
    if (best_v) best_v[at] = best[j];
    best_i[at] = inv[j] > 0.f ? bid[j] : kSlowRow;
  }
}

// One wavefront per row: the best of the shares, and ||x||^2 + its value as
// the distance.  A row with an infinite coordinate is compared with every
// centre in float32.
__global__ void __launch_bounds__(256) k_assign_finish(
    const float *__restrict__ x, int64_t n, int D, const float *__restrict__ cen, int nlist,
    const float *__restrict__ cnorm, int shares, const float *best_v, const int32_t *best_i,
    int32_t *out_ids, float *out_d) {
  const int lane = threadIdx.x & 63;
  const int64_t row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  float v = __builtin_inff();
  int32_t id = 0x7fffffff;
  for (int s = lane; s < shares; s += 64) {
    const float ov = best_v ? best_v[int64_t(s) * n + row] : 0.f;
    const int32_t oi = best_i[int64_t(s) * n + row];
    if (oi == kSlowRow || (id != kSlowRow && (ov < v || (ov == v && oi < id)))) {
      v = ov;
      id = oi;
    }
  }
  for (int off = 1; off < 64; off <<= 1) {
    const float ov = __shfl_xor(v, off, 64);
    const int32_t oi = __shfl_xor(id, off, 64);
    if (oi == kSlowRow || (id != kSlowRow && (ov < v || (ov == v && oi < id)))) {
      v = ov;
      id = oi;
    }
  }
  const float *xr = x + row * D;
  if (id == kSlowRow) {
    v = 3.4e38f;
    id = 0x7fffffff;
    for (int c = 0; c < nlist; ++c) {
      float dot = 0.f;
      for (int k = lane; k < D; k += 64) dot += xr[k] * cen[int64_t(c) * D + k];
      dot = wave_sum(dot);
      const float w = cnorm[c] - 2.f * dot;
      if (w < v) {
        v = w;
        id = c;
      }
    }
  }
  if (out_d) {
    double s = 0.0;
    for (int k = lane * 4; k < D; k += 256) {
      if (k + 4 <= D) {
        const F4u q = *reinterpret_cast<const F4u *>(xr + k);
        s += double(q.x) * q.x + double(q.y) * q.y + (double(q.z) * q.z + double(q.w) * q.w);
      } else {
        for (int e = k; e < D; ++e) s += double(xr[e]) * xr[e];
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) out_d[row] = float(s + double(v));
  }
  if (lane == 0) out_ids[row] = id;
}

// Whether an assignment runs on split float16, and its workspace.
struct SplitWs {
  float *cnorm, *cmul;
  _Float16 *split;
  float *part_v;
  int32_t *part_i;
  int tiles, n_slab, shares, tiles_per_share;
  size_t bytes;
};
static bool assign_on_split(int64_t n, int dim, int nlist) {
  // Rows that are whole 16-byte runs have the float32 matrix kernel to beat:
  // up to 128 centres half a tile of 256 or more is padding (us, float32
  // against split: 65,536 x 512 by 128 113, 119; 1,011,082 x 922 by 188 18,536 on
  // the vector ALU, 3,472), and below 128 rows there is too little work (64 x 768
  // by 1,024 91, 104; 256 x 768 by 4,096 149, 105).  Other rows have a vector-ALU
  // kernel, slower from a few microseconds of work on (4,573 x 230 by 21 87, 52;
  // 20,000 x 1,501 by 16 1,114, 242).
  if (dim % 4 == 0) return nlist > 128 && n >= 128;
  return double(n) * double(nlist) * double(dim) >= 1e6;
}
static SplitWs assign_split_ws(void *base, int64_t n, int dim, int nlist) {
  SplitWs w{};
  char *p = static_cast<char *>(base);
  size_t off = 0;
  auto take = [&](size_t b) {
    char *r = p ? p + off : nullptr;
    off += (b + 255) / 256 * 256;
    return r;
  };
  w.tiles = (nlist + kSpN - 1) / kSpN;
  w.n_slab = (dim + kSpK - 1) / kSpK;
  const size_t np = size_t(w.tiles) * kSpN;
  // the centres are shared out where the rows alone leave compute units idle
  const int64_t blocks = (n + kSpM - 1) / kSpM;
  const int64_t want = std::min<int64_t>(w.tiles, (512 + blocks - 1) / blocks);
  w.tiles_per_share = int((w.tiles + want - 1) / want);
  w.shares = (w.tiles + w.tiles_per_share - 1) / w.tiles_per_share;
  w.cnorm = reinterpret_cast<float *>(take(np * 4));
  w.cmul = reinterpret_cast<float *>(take(np * 4));
  w.split = reinterpret_cast<_Float16 *>(take(np * w.n_slab * 2 * kSpK * sizeof(_Float16)));
  if (w.shares > 1) {
    w.part_v = reinterpret_cast<float *>(take(size_t(w.shares) * n * 4));
    w.part_i = reinterpret_cast<int32_t *>(take(size_t(w.shares) * n * 4));
  }
  w.bytes = off;
  return w;
}

// Probe dots for many rows (D a multiple of 4, 16-byte aligned operands): one
// 128 x 128 tile (tile128) per workgroup, written out.
__global__ void __launch_bounds__(256) k_dots_big(const float *__restrict__ x, int n, int D,
                                                  const float *__restrict__ cen, int nlist,
                                                  float *__restrict__ dots) {
  __shared__ float As[kAM][kAS];
  __shared__ float Bs[kAN][kAS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = (wave >> 1) * 64, wc = (wave & 1) * 64;
  const int m = lane & 15, h = lane >> 4;
  const int r0 = blockIdx.y * kAM, c0 = blockIdx.x * kAN;
  const int srow = tid >> 3, scol = (tid & 7) * 4;
  int64_t aoff[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) aoff[u] = int64_t(min(r0 + srow + 32 * u, n - 1)) * D + scol;
  floatx4_t acc[4][4];
  tile128(x, aoff, D, cen, nlist, c0, As, Bs, acc);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = r0 + wr + 16 * i + 4 * h + e;
        const int c = c0 + wc + 16 * j + m;
        if (r < n && c < nlist) dots[int64_t(r) * nlist + c] = acc[i][j][e];
      }
}

// Probe dots for D a multiple of 4 and 16-byte aligned operands: a 64 x 64
// output tile per workgroup, each of the four wavefronts a 32 x 32 block as
// 2 x 2 MFMA tiles; k staged through LDS in slabs of 32 with the next slab
// prefetched into registers, the same permuted k within half slabs as the
// assignment kernel.  Every centre row is read from L2 by n / 64 workgroups.
constexpr int kPT = 64;

__global__ void __launch_bounds__(256) k_dots_tiled(const float *__restrict__ x, int n, int D,
                                                    const float *__restrict__ cen, int nlist,
                                                    float *__restrict__ dots) {
  __shared__ float As[kPT][kAS];
  __shared__ float Bs[kPT][kAS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  const int m = lane & 15, h = lane >> 4;
  const int r0 = blockIdx.y * kPT, c0 = blockIdx.x * kPT;
  // staging: thread t moves the float4s (row t / 8 + 32 u, column 4 (t % 8)),
  // u = 0, 1, of a 64 x 32 slab; rows past the end are clamped
  const int srow = tid >> 3, scol = (tid & 7) * 4;
  int64_t aoff[2], boff[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    aoff[u] = int64_t(min(r0 + srow + 32 * u, n - 1)) * D + scol;
    boff[u] = int64_t(min(c0 + srow + 32 * u, nlist - 1)) * D + scol;
  }
  floatx4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  const int nslab = (D + kAK - 1) / kAK;
  float4 pa[2], pb[2];
  const bool in0 = scol < D;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    pa[u] = ld4_or_zero(x + aoff[u], in0);
    pb[u] = ld4_or_zero(cen + boff[u], in0);
  }
  for (int sl = 0; sl < nslab; ++sl) {
    __syncthreads();   // the previous slab's operand reads are done
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      *reinterpret_cast<float4 *>(&As[srow + 32 * u][scol]) = pa[u];
      *reinterpret_cast<float4 *>(&Bs[srow + 32 * u][scol]) = pb[u];
    }
    __syncthreads();
    if (sl + 1 < nslab) {
      const int kn = (sl + 1) * kAK;
      const bool in = kn + scol < D;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        pa[u] = ld4_or_zero(x + aoff[u] + kn, in);
        pb[u] = ld4_or_zero(cen + boff[u] + kn, in);
      }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      float4 a4[2], b4[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a4[i] = *reinterpret_cast<const float4 *>(&As[wr + 16 * i + m][16 * s + 4 * h]);
        b4[i] = *reinterpret_cast<const float4 *>(&Bs[wc + 16 * i + m][16 * s + 4 * h]);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const float av = t == 0 ? a4[i].x : t == 1 ? a4[i].y : t == 2 ? a4[i].z : a4[i].w;
            const float bv = t == 0 ? b4[j].x : t == 1 ? b4[j].y : t == 2 ? b4[j].z : b4[j].w;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[i][j], 0, 0, 0);
          }
    }
  }
  // lane holds C[4 h + e][m] of each 16 x 16 tile
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = r0 + wr + 16 * i + 4 * h + e;
        const int c = c0 + wc + 16 * j + m;
        if (r < n && c < nlist) dots[int64_t(r) * nlist + c] = acc[i][j][e];
      }
}

struct IdentityId {
  __device__ int32_t operator()(int i) const { return i; }
};

// Top-nprobe of one row of dots (nlist <= 16,384): 1,024 threads hold the
// row in registers.  The dots are binned linearly over [min, max] of the row
// (1,024 bins; the bin index is a non-decreasing function of the dot, so "bin
// >= b" is an up-set of the order), the bin holding the nprobe-th largest dot
// is found, and every dot in it or above is sorted on (dot desc, list asc).
// Value bins spread the row evenly, unlike the leading bits of the float
// keys, which most dots share (LDS atomics on a few bins serialise).  If the
// boundary bin is crowded (equal or clustered dots), 8-bit radix passes over
// the keys take over, and beyond that the block selection.
constexpr int kPSelThreads = 1024;
constexpr int kPSelPer = 16;
constexpr int kPSelBins = 1024;

__global__ void __launch_bounds__(kPSelThreads) k_probe_select_reg(const float *__restrict__ dots,
                                                                   int nlist, int nprobe,
                                                                   int32_t *__restrict__ out_ids,
                                                                   float *__restrict__ out_s) {
  __shared__ SelectSmem sm;   // hist during the counting passes, buf afterwards
  __shared__ float red[2][kPSelThreads / 64];
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t row = blockIdx.x;
  const float *d = dots + row * nlist;
  float val[kPSelPer];
  uint32_t key[kPSelPer];
  float lo = __builtin_inff(), hi = -__builtin_inff();
#pragma unroll
  for (int v = 0; v < kPSelPer; ++v) {
    const int i = v * nt + tid;
    val[v] = (i < nlist) ? d[i] : 0.f;
    key[v] = (i < nlist) ? order_key(val[v]) : 0u;   // every real key is > 0
    if (i < nlist) {
      lo = fminf(lo, val[v]);
      hi = fmaxf(hi, val[v]);
    }
  }
  lo = -wave_max(-lo);
  hi = wave_max(hi);
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = lo;
    red[1][tid >> 6] = hi;
  }
  __syncthreads();
  lo = red[0][0];
  hi = red[1][0];
  for (int w = 1; w < nt / 64; ++w) {
    lo = fminf(lo, red[0][w]);
    hi = fmaxf(hi, red[1][w]);
  }
  const float scale = (hi > lo) ? float(kPSelBins) / (hi - lo) : 0.f;
  auto bin_of = [&](float x) { return min(kPSelBins - 1, int((x - lo) * scale)); };
  bool collect_by_bin = false;
  int bbin = 0;
  uint32_t edge = 0;
  if (scale > 0.f && scale < 3.0e38f) {
    for (int b = tid; b < kPSelBins; b += nt) sm.hist[b] = 0;
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kPSelPer; ++v)
      if (v * nt + tid < nlist) atomicAdd(&sm.hist[bin_of(val[v])], 1u);
    find_boundary(sm, kPSelBins, 0u, uint32_t(nprobe));
    bbin = int(sm.bcast[0]);
    collect_by_bin = sm.bcast[1] + sm.hist[bbin] <= uint32_t(kSelCap);
    __syncthreads();
  }
  if (!collect_by_bin) {
    uint32_t prefix = 0, above = 0;
    for (int shift = 24; shift >= 0; shift -= 8) {
      for (int b = tid; b < 256; b += nt) sm.hist[b] = 0;
      __syncthreads();
#pragma unroll
      for (int v = 0; v < kPSelPer; ++v) {
        const int i = v * nt + tid;
        if (i < nlist && (shift == 24 || (key[v] >> (shift + 8)) == prefix))
          atomicAdd(&sm.hist[(key[v] >> shift) & 255u], 1u);
      }
      find_boundary(sm, 256, above, uint32_t(nprobe));
      const uint32_t bb = sm.bcast[0];
      const uint32_t in_bin = sm.hist[bb];
      above = sm.bcast[1];
      prefix = (prefix << 8) | bb;
      edge = prefix << shift;
      __syncthreads();
      if (above + in_bin <= uint32_t(kSelCap)) break;
      if (shift == 0) {   // more than kSelCap equal keys at the boundary
        block_topk(d, nlist, nprobe, IdentityId(), out_s + row * nprobe, out_ids + row * nprobe,
                   sm);
        return;
      }
    }
  }
  if (tid == 0) sm.count = 0;
  __syncthreads();
#pragma unroll
  for (int v = 0; v < kPSelPer; ++v) {
    const int i = v * nt + tid;
    const bool take = collect_by_bin ? bin_of(val[v]) >= bbin : key[v] >= edge;
    if (i < nlist && take) sm.buf[atomicAdd(&sm.count, 1u)] = composite(key[v], i);
  }
  __syncthreads();
  emit_sorted(sm, int(sm.count), nprobe, out_s + row * nprobe, out_ids + row * nprobe);
}

// Top-nprobe for rows longer than the register-resident kernel holds.
__global__ void __launch_bounds__(kSelThreads) k_probe_select(const float *__restrict__ dots,
                                                              int nlist, int nprobe,
                                                              int32_t *__restrict__ out_ids,
                                                              float *__restrict__ out_s) {
  __shared__ SelectSmem sm;
  const int64_t row = blockIdx.x;
  block_topk(dots + row * nlist, nlist, nprobe, IdentityId(), out_s + row * nprobe,
             out_ids + row * nprobe, sm);
}

// ------------------------------------------------------------- fixed scratch
// Scratch of ivf_assign_probe_noalloc: a static device array, one per GPU
// the library runs on, held until the process ends.  Host code never uses
// its name as an address: the device address is looked up once per device
// (hipGetSymbolAddress, with that device current) and kept in g_scratch_ptr.
constexpr size_t kProbeScratchBytes = (size_t(64) << 20) + (size_t(256) << 10);
static __device__ __align__(256) unsigned char scratch[kProbeScratchBytes];

constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices] = {nullptr};
static std::mutex g_scratch_mu;

// Device address of this GPU's scratch (looked up on first use); nullptr
// with *status set when the lookup fails.
static void *scratch_of_current_device(int *status) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    *status = set_hip_error(e);
    return nullptr;
  }
  if (dev < 0 || dev >= kMaxDevices) {
    *status = RSLM_ERR_UNSUPPORTED;
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      *status = set_hip_error(e != hipSuccess ? e : hipErrorInvalidSymbol);
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *status = RSLM_OK;
  return g_scratch_ptr[dev];
}

}  // namespace rslm

using namespace rslm;

extern "C" {

size_t ivf_assign_probe_workspace(int64_t n, int32_t dim, int32_t nlist, int32_t nprobe,
                                  int mode) {
  (void)nprobe;
  if (n < 0 || nlist < 1) return 0;
  const size_t norms = (size_t(nlist) * sizeof(float) + 255) / 256 * 256;
  if (mode == IVF_ASSIGN_L2 && dim >= 1 && nlist <= 65536 && assign_on_split(n, dim, nlist))
    return assign_split_ws(nullptr, n, dim, nlist).bytes;
  if (mode == IVF_ASSIGN_L2) return norms;
  const size_t dots = size_t(n) * size_t(nlist) * sizeof(float);
  return norms + (dots + 255) / 256 * 256;
}

// The least a call accepts: the float32 kernels' scratch.
static size_t probe_min_workspace(int64_t n, int32_t nlist, int mode) {
  const size_t norms = (size_t(nlist) * sizeof(float) + 255) / 256 * 256;
  if (mode == IVF_ASSIGN_L2) return norms;
  return norms + (size_t(n) * size_t(nlist) * sizeof(float) + 255) / 256 * 256;
}

int ivf_assign_probe(const float *x, int64_t n, int32_t dim, const float *centroids,
                     int32_t nlist, int32_t nprobe, int mode, int32_t *out_ids,
                     float *out_scores, void *ws, size_t ws_bytes, void *stream) {
  if (n < 0 || dim < 1 || nlist < 1 || nlist > 65536) return RSLM_ERR_INVALID_ARG;
  if (mode != IVF_ASSIGN_L2 && mode != IVF_PROBE_IP) return RSLM_ERR_INVALID_ARG;
  if (mode == IVF_ASSIGN_L2 && nprobe != 1) return RSLM_ERR_INVALID_ARG;
  if (mode == IVF_PROBE_IP && (nprobe < 1 || nprobe > nlist || nprobe > kMaxNprobe))
    return RSLM_ERR_INVALID_ARG;
  if (n == 0) return RSLM_OK;
  if (!x || !centroids || !out_ids || (mode == IVF_PROBE_IP && !out_scores))
    return RSLM_ERR_INVALID_ARG;
  if (!ws || ws_bytes < probe_min_workspace(n, nlist, mode)) return RSLM_ERR_WORKSPACE;
  hipStream_t s = as_stream(stream);
  if (mode == IVF_ASSIGN_L2 && (n + 255) / 256 <= 0x7fffffff && (n + 3) / 4 <= 0x7fffffff &&
      assign_on_split(n, dim, nlist)) {
    // (a workspace that has room for the norms only takes the float32 kernels)
    const SplitWs w = assign_split_ws(ws, n, dim, nlist);
    if (ws_bytes >= w.bytes && (reinterpret_cast<uintptr_t>(ws) & 15) == 0) {
      hipLaunchKernelGGL(k_split_centres, dim3(unsigned(w.tiles * kSpN / 4)), dim3(256), 0, s,
                         centroids, nlist, dim, w.n_slab, w.cnorm, w.cmul, w.split);
      int st = check_launch();
      if (st) return st;
      float *bv = w.shares > 1 ? w.part_v : out_scores;
      int32_t *bi = w.shares > 1 ? w.part_i : out_ids;
      hipLaunchKernelGGL(k_assign_split, dim3(unsigned((n + kSpM - 1) / kSpM), unsigned(w.shares)),
                         dim3(kSpThreads), 0, s, x, n, dim, w.n_slab, w.cnorm, w.cmul, w.split,
                         w.tiles, w.tiles_per_share, bv, bi);
      if ((st = check_launch())) return st;
      hipLaunchKernelGGL(k_assign_finish, dim3(unsigned((n + 3) / 4)), dim3(256), 0, s, x, n, dim,
                         centroids, nlist, w.cnorm, w.shares, bv, bi, out_ids, out_scores);
      return check_launch();
    }
  }
  if (mode == IVF_ASSIGN_L2) {
    float *cnorm = static_cast<float *>(ws);
    hipLaunchKernelGGL(k_row_norms, dim3((nlist + 3) / 4), dim3(256), 0, s, centroids, nlist,
                       dim, cnorm);
    int st = check_launch();
    if (st) return st;
    const bool aligned16 = (reinterpret_cast<uintptr_t>(x) % 16 == 0) &&
                           (reinterpret_cast<uintptr_t>(centroids) % 16 == 0);
    if (dim % 4 == 0 && aligned16) {   // rows are whole, aligned float4 runs
      const int64_t grid = (n + kAM - 1) / kAM;
      if (grid > 0x7fffffff) return RSLM_ERR_INVALID_ARG;
      hipLaunchKernelGGL(k_assign_mfma, dim3(unsigned(grid)), dim3(256), 0, s, x, n, dim,
                         centroids, nlist, cnorm, out_ids, out_scores);
      return check_launch();
    }
    const int64_t grid = (n + kTM - 1) / kTM;
    if (grid > 0x7fffffff) return RSLM_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_assign, dim3(unsigned(grid)), dim3(256), 0, s, x, n, dim, centroids,
                       nlist, cnorm, out_ids, out_scores);
    return check_launch();
  }
  const size_t norms = (size_t(nlist) * sizeof(float) + 255) / 256 * 256;
  float *dots = reinterpret_cast<float *>(static_cast<char *>(ws) + norms);
  const int64_t gy32 = (n + kMT - 1) / kMT;
  if (gy32 > 65535) return RSLM_ERR_INVALID_ARG;
  int st;
  const bool aligned16 = (reinterpret_cast<uintptr_t>(x) % 16 == 0) &&
                         (reinterpret_cast<uintptr_t>(centroids) % 16 == 0);
  const int64_t big_tiles = ((n + kAM - 1) / kAM) * ((nlist + kAN - 1) / kAN);
  if (dim % 4 == 0 && aligned16 && big_tiles >= 1024) {   // enough 128 x 128 tiles
    hipLaunchKernelGGL(k_dots_big, dim3(unsigned((nlist + kAN - 1) / kAN),
                                        unsigned((n + kAM - 1) / kAM)),
                       dim3(256), 0, s, x, int(n), dim, centroids, nlist, dots);
  } else if (dim % 4 == 0 && aligned16) {   // rows are whole, aligned float4 runs
    hipLaunchKernelGGL(k_dots_tiled, dim3(unsigned((nlist + kPT - 1) / kPT),
                                          unsigned((n + kPT - 1) / kPT)),
                       dim3(256), 0, s, x, int(n), dim, centroids, nlist, dots);
  } else {
    hipLaunchKernelGGL(k_dots_mfma, dim3((nlist + kMT - 1) / kMT, unsigned(gy32)), dim3(256), 0, s,
                       x, n, dim, centroids, nlist, dots);
  }
  if ((st = check_launch())) return st;
  if (n > 0x7fffffff) return RSLM_ERR_INVALID_ARG;
  if (nlist <= kPSelThreads * kPSelPer)
    hipLaunchKernelGGL(k_probe_select_reg, dim3(unsigned(n)), dim3(kPSelThreads), 0, s, dots, nlist,
                       nprobe, out_ids, out_scores);
  else
    hipLaunchKernelGGL(k_probe_select, dim3(unsigned(n)), dim3(kSelThreads), 0, s, dots, nlist,
                       nprobe, out_ids, out_scores);
  return check_launch();
}

}  // extern "C"

extern "C" {

int ivf_assign_probe_noalloc(const float *x, int64_t n, int32_t dim, const float *centroids,
                             int32_t nlist, int32_t nprobe, int mode, int32_t *out_ids,
                             float *out_scores, void *stream) {
  // the same validation as ivf_assign_probe, then the fixed scratch's limit
  if (n < 0 || dim < 1 || nlist < 1 || nlist > 65536) return RSLM_ERR_INVALID_ARG;
  if (mode != IVF_ASSIGN_L2 && mode != IVF_PROBE_IP) return RSLM_ERR_INVALID_ARG;
  if (mode == IVF_ASSIGN_L2 && nprobe != 1) return RSLM_ERR_INVALID_ARG;
  if (mode == IVF_PROBE_IP && (nprobe < 1 || nprobe > nlist || nprobe > kMaxNprobe))
    return RSLM_ERR_INVALID_ARG;
  if (n == 0) return RSLM_OK;
  if (!x || !centroids || !out_ids || (mode == IVF_PROBE_IP && !out_scores))
    return RSLM_ERR_INVALID_ARG;
  if (probe_min_workspace(n, nlist, mode) > kProbeScratchBytes) return RSLM_ERR_WORKSPACE;
  int st = RSLM_OK;
  void *ws = scratch_of_current_device(&st);
  if (!ws) return st;
  return ivf_assign_probe(x, n, dim, centroids, nlist, nprobe, mode, out_ids, out_scores, ws,
                          kProbeScratchBytes, stream);
}

size_t ivf_assign_probe_noalloc_limit(void) { return kProbeScratchBytes; }

}  // extern "C"

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
#include <algorithm>
#include <mutex>
#include <type_traits>

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
// float32 rate per product).  These products only sort the centres out: with
// every value goes a bound t(x, c) of its distance from the exact
// ||c||^2 - 2 <x, c> (split_margin), a row whose best value beats every other
// one by more than the bounds is decided, and the rows that are left (near
// ties, rows with one coordinate far above the rest, infinities and NaN) are
// evaluated against every centre in float64 (k_assign_exact).  The centre
// returned is thus the nearest one in float64, the lowest id where two are
// equal there, at any D and whatever the values' spread, and the distance is a
// float64 sum rounded once.  A pair's product does not depend on the other
// rows and centres of its tile, so results do not depend on how a call is cut
// into shares, groups and pieces, that is, on the workspace.
//
// A workgroup of eight wavefronts owns 256 rows of x and walks its share of
// the centres in tiles of 256: with both sides at 256 each operand is read
// from L2 once per 256 rows of the other, which is what the matrix cores leave
// time for.  The centres are split once per call (k_split_centres), the rows
// of x as they are staged (they are too many to keep).  k goes through LDS in
// slabs of 32, two buffers, one barrier per slab.  Centres are the M side, so
// a lane holds 32 centres of each of four rows and keeps four running minima.
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
constexpr int kSpM = 256, kSpN = 256, kSpK = 32, kSpThreads = 512;
constexpr int kSpRow = 4 * kSpK;       // bytes per LDS row: hi, then lo
constexpr int kWaitVm0 = 0x0F70;       // s_waitcnt vmcnt(0), the other counters free
constexpr float kFarthest = 3.4e38f;   // values from here on are not chosen
constexpr int32_t kNoCentre = 0x7fffffff;

struct __attribute__((packed, aligned(4))) F4u {
  float x, y, z, w;
};

// Power of two s with m s in [2^14, 2^15) (m > 0 finite; the exponent is
// clamped where s would not be a normal number).
__device__ __forceinline__ float split_scale(float m) {
  if (!(m > 0.f) || !(m < __builtin_inff())) return 1.f;
  return ldexpf(1.f, max(-126, min(126, 14 - ilogbf(m))));
}

// What is kept of a centre besides its halves.
struct CentreTab {
  float *base;     // ||c||^2 less the margin's part without x; +inf where ||c||^2
                   // is not finite and past nlist: never nearest
  float *along;    // the margin's factor of ||x||
  float *margin;   // the margin's part without x
  float *mul;      // -2 / s
  double *norm;    // ||c||^2; +inf as above
};

// t(x, c) = margin + along ||x|| bounds the difference of the computed value
// fma(acc mul, 1 / s_x, ||c||^2) from the exact one, in units u = 2^-24 of
// ||x|| ||c||:
//   operands   what hi + lo leaves out is at most 2^-22 of a coordinate (and
//              2^-25 of the scaled row's unit where lo is subnormal; 2^-14 were
//              subnormal halves read as 0), and lo lo is dropped: 3 2^-22 of
//              every product, and 2 sqrt(D) 2^-28 of the whole, at most 16 u for D
//              <= 16,384                                               12 + 16
//   products   32 exact products per instruction: at most 34 roundings or
//              truncations of 2^-23 of their absolute sum                   68
//   slabs      one float32 addition each                                D / 32
// twice that, since 2 <x, c> is taken, is 192 + D / 16; 16 more for the
// roundings of the norms and of the value itself, which also take 8 u of
// ||c||^2.  2^-100 and 1e-30 cover scales that were clamped and underflow.
constexpr int kSplitMaxDim = 16384;
__device__ __forceinline__ void split_margin(int D, float cnorm, float &along, float &margin) {
  const float u = 0x1p-24f;
  along = u * (208.f + D / 16.f) * (sqrtf(cnorm) * 1.001f + 0x1p-100f);
  margin = u * 8.f * cnorm + 1e-30f;
}

// One wavefront per centre (nlist rounded up to whole tiles): its table
// entries, and the halves of those of the tiles [t0, t1), slab by slab (32 hi,
// then 32 lo, zero past D).  Workgroup 0 also clears the list's length.
__global__ void __launch_bounds__(256) k_split_centres(const float *__restrict__ cen, int nlist, int D,
                                                       int n_slab, int c0, CentreTab tab,
                                                       _Float16 *__restrict__ split,
                                                       int32_t *__restrict__ n_listed) {
  const int lane = threadIdx.x & 63;
  const int cg = blockIdx.x * 4 + (threadIdx.x >> 6);   // within the group
  const int c = c0 + cg;
  if (blockIdx.x == 0 && threadIdx.x == 0) *n_listed = 0;
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
  const float cn = float(sum);
  const bool ok = in && cn < __builtin_inff();   // (not for a NaN)
  const float sc = split_scale(wave_max(ok ? m : 0.f));
  if (lane == 0) {
    float along = 0.f, margin = 0.f;
    if (ok) split_margin(D, cn, along, margin);
    tab.base[c] = ok ? cn - margin : __builtin_inff();
    tab.along[c] = along;
    tab.margin[c] = margin;
    tab.mul[c] = -2.f / sc;
    tab.norm[c] = ok ? sum : double(__builtin_inff());
  }
  _Float16 *out = split + int64_t(cg) * n_slab * (2 * kSpK);
  for (int i = lane; i < n_slab * kSpK; i += 64) {
    const float v = (ok && i < D) ? row[i] * sc : 0.f;
    const _Float16 h = static_cast<_Float16>(v);
    out[(i / kSpK) * (2 * kSpK) + i % kSpK] = h;
    out[(i / kSpK) * (2 * kSpK) + kSpK + i % kSpK] = static_cast<_Float16>(v - static_cast<float>(h));
  }
}

// What a share of the centres leaves of a row: the lowest lower bound w = value
// - t, its centre, and the second lowest w.
struct SplitPart {
  float *w1, *w2;
  int32_t *id;
};

// Takes (w1, id, w2) of disjoint sets of centres together.
__device__ __forceinline__ void merge_part(float &w1, int32_t &id, float &w2, float ow1, int32_t oid,
                                           float ow2) {
  w2 = fminf(fminf(w2, ow2), fmaxf(w1, ow1));
  if (ow1 < w1 || (ow1 == w1 && oid < id)) {
    w1 = ow1;
    id = oid;
  }
}

// Workgroup (rows, share): its share of the tiles [0, n_tiles) of 256 centres
// at `split` (of which the first is centre c0) for 256 of the rows of x, to
// `part` at [share][row], and ||x|| to xnorm.  Whole call, 1,048,576 x 768 by
// 4,096: 52.5 ms on the float32 kernel, 20.4 ms here (324 TFLOP/s of distances,
// 970 TFLOP/s of float16 products; a large bf16 library product runs at 1,370 on
// the same card).  The same tiles with the centres staged through registers took
// 10 ms more, with two slabs of both operands in registers 18 ms (spills).
__global__ void __launch_bounds__(kSpThreads, 2) k_assign_split(
    const float *__restrict__ x, int64_t n, int D, int n_slab, int c0, CentreTab tab,
    const _Float16 *__restrict__ split, int n_tiles, int tiles_per_share, SplitPart part,
    float *__restrict__ xnorm) {
  // rows of 128 bytes (32 hi, 32 lo): x, then centres; the eight 16-byte units
  // of row r are stored at unit ^ (r % 8), which spreads a column of units
  // over the banks without padding (the centres are written by lanes in order)
  __shared__ __align__(128) uint8_t lds[2][(kSpM + kSpN) * kSpRow];
  __shared__ float xscale[kSpM], xlen[kSpM];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, h = lane >> 4;
  const int wx = (wave & 3) * 64, wc = (wave >> 2) * 128;   // this wave's rows and centres
  const int64_t r0 = int64_t(blockIdx.x) * kSpM;
  const int t0 = blockIdx.y * tiles_per_share, t1 = min(n_tiles, t0 + tiles_per_share);
  // largest magnitude and length of each row: 32 rows per wavefront, four in
  // flight.  A row with an infinity or a NaN, or whose ||x||^2 overflows, gets a
  // length of +inf or NaN, with which no value is decided.
  for (int q = 0; q < 32; q += 4) {
    float mx[4] = {0.f, 0.f, 0.f, 0.f}, ss[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = lane; k < D; k += 64) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t r = min(r0 + wave * 32 + q + u, n - 1);
        const float v = x[r * D + k];
        mx[u] = fmaxf(mx[u], fabsf(v));
        ss[u] = fmaf(v, v, ss[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      mx[u] = wave_max(mx[u]);
      ss[u] = wave_sum(ss[u]);
      const int rl = wave * 32 + q + u;
      if (lane == 0) {
        xscale[rl] = split_scale(mx[u]);
        xlen[rl] = sqrtf(ss[u]);
        if (blockIdx.y == 0 && r0 + rl < n) xnorm[r0 + rl] = sqrtf(ss[u]);
      }
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
  float best[4], second[4], inv[4], len[4];
  int32_t bid[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    best[j] = second[j] = __builtin_inff();
    bid[j] = kNoCentre;
    inv[j] = 1.f / xscale[wx + 16 * j + m];
    len[j] = xlen[wx + 16 * j + m];
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
      // lane (m, h) holds centres c + 16 i + 4 h + e of rows wx + 16 j + m
      const int c = c0 + tile * kSpN + wc + 4 * h;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float4 cb = *reinterpret_cast<const float4 *>(tab.base + c + 16 * i);
        const float4 ca = *reinterpret_cast<const float4 *>(tab.along + c + 16 * i);
        const float4 cm = *reinterpret_cast<const float4 *>(tab.mul + c + 16 * i);
        const float cba[4] = {cb.x, cb.y, cb.z, cb.w}, caa[4] = {ca.x, ca.y, ca.z, ca.w},
                    cma[4] = {cm.x, cm.y, cm.z, cm.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            // ||c||^2 - 2 <x, c> - t (the scales one after the other: their
            // product can underflow where the value does not)
            const float w = fmaf(acc[i][j][e] * cma[e], inv[j], fmaf(-caa[e], len[j], cba[e]));
            second[j] = __builtin_amdgcn_fmed3f(best[j], second[j], w);   // of three, as best <= second
            if (w < best[j]) {   // centres visited in increasing order
              best[j] = w;
              bid[j] = c + 16 * i + e;
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
  // merge the four lanes and the two wavefronts holding a row
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int off = 16; off < 64; off <<= 1)
      merge_part(best[j], bid[j], second[j], __shfl_xor(best[j], off, 64), __shfl_xor(bid[j], off, 64),
                 __shfl_xor(second[j], off, 64));
  float *red_v = reinterpret_cast<float *>(lds[0]);   // the last slab was multiplied before a barrier
  float *red_s = red_v + kSpM;
  int32_t *red_i = reinterpret_cast<int32_t *>(red_s + kSpM);
  if (wave >= 4 && h == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int rl = wx + 16 * j + m;
      red_v[rl] = best[j];
      red_s[rl] = second[j];
      red_i[rl] = bid[j];
    }
  }
  __syncthreads();
  if (wave >= 4 || h) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int rl = wx + 16 * j + m;
    if (r0 + rl >= n) continue;
    merge_part(best[j], bid[j], second[j], red_v[rl], red_i[rl], red_s[rl]);
    const int64_t at = int64_t(blockIdx.y) * n + r0 + rl;
    part.w1[at] = best[j];
    part.w2[at] = second[j];
    part.id[at] = bid[j];
  }
}

// One thread per row: the shares taken together; the centre where the row is
// decided, else ~(its place in the list).
__global__ void __launch_bounds__(256) k_assign_decide(int64_t n, int shares, SplitPart part,
                                                       const float *__restrict__ xnorm, CentreTab tab,
                                                       int32_t *__restrict__ list,
                                                       int32_t *__restrict__ n_listed,
                                                       int32_t *__restrict__ out_ids) {
  const int64_t row = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (row >= n) return;
  float w1 = __builtin_inff(), w2 = __builtin_inff();
  int32_t id = kNoCentre;
  for (int s = 0; s < shares; ++s) {
    const int64_t at = int64_t(s) * n + row;
    merge_part(w1, id, w2, part.w1[at], part.id[at], part.w2[at]);
  }
  bool decided = false;
  if (id != kNoCentre) {
    // w1 + 2 t is at least the exact value of the best
    const float up = fmaf(2.f, fmaf(tab.along[id], xnorm[row], tab.margin[id]), w1);
    decided = up < w2 && up < 1e37f;
  }
  if (decided) {
    out_ids[row] = id;
  } else {
    const int32_t at = atomicAdd(n_listed, 1);
    list[at] = int32_t(row);
    out_ids[row] = ~at;
  }
}

// The listed rows against every centre in float64: workgroups take (64 rows,
// share of the centres) items, as many shares as fill the chip.  A share is
// tiles of 16 TJ centres, 4 x TJ values per thread: TJ = 4 for throughput, TJ = 1
// and longer slabs up to 256 listed rows, where the chain of one tile's slabs is
// what a call waits for (22,958 x 475 by 1,581, us: with no row settled here 278, TJ =
// 4 340, TJ = 1 307).  About 41 TFLOP/s, so a call whose rows are mostly near ties
// takes longer than the float32 kernel: 131,072 x 768 by 4,096 2.8 ms with few, 10.3
// where the coordinates are 30 times their spread from 0, 23 with every centre
// twice, float32 6.6 (and 0.6 % of the rows of the second at another centre than
// the nearest, 33 % at 300 times the spread).  Values are ||c||^2 - 2 <x, c>,
// summed over k in order whatever the tile; the lowest and its lowest id, kNoCentre
// where no value is below 3.4e38 (and infinite and NaN products as in float32).
constexpr int kExT = 64, kExGrid = 1024;
constexpr int kExFew = 256;                // rows up to which TJ = 1
constexpr int kExParts = kExGrid * kExT;   // (row, share) results kept at a time
constexpr int kExLds = 5120;               // doubles: 32 x (64 + 64) or 64 x (64 + 16)
__device__ __forceinline__ int exact_tiles(int rows, int nlist) {
  const int t = rows <= kExFew ? 16 : 64;
  return (nlist + t - 1) / t;
}
__device__ __forceinline__ int exact_shares(int rows, int nlist) {
  const int blocks = (rows + kExT - 1) / kExT;
  return max(1, min(kExGrid / max(blocks, 1), exact_tiles(rows, nlist)));
}
template <int TJ>
__device__ __forceinline__ void exact_items(const float *__restrict__ x, int D,
                                            const float *__restrict__ cen, int nlist,
                                            const double *__restrict__ norm,
                                            const int32_t *__restrict__ list, int rows, double *lds,
                                            double *__restrict__ part_v, int32_t *__restrict__ part_i,
                                            int32_t *__restrict__ out_ids) {
  constexpr int K = TJ == 1 ? 64 : 32, T = 16 * TJ;
  constexpr int AE = kExT * K / 256, BE = T * K / 256;   // staged per thread
  static_assert(K * (kExT + T) <= kExLds, "slabs fit");
  double(*As)[kExT] = reinterpret_cast<double(*)[kExT]>(lds);
  double(*Bs)[T] = reinterpret_cast<double(*)[T]>(lds + K * kExT);
  const int blocks = (rows + kExT - 1) / kExT;
  const int shares = exact_shares(rows, nlist);
  const int tiles = (nlist + T - 1) / T, per = (tiles + shares - 1) / shares;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  // staging: row / centre and first k of this thread
  const int ar = threadIdx.x % kExT, ak = threadIdx.x / kExT * AE;
  const int br = threadIdx.x % T, bk = threadIdx.x / T * BE;
  auto load = [&](const float *row, int k, float *v, auto count) {
    constexpr int N = decltype(count)::value;
    if (k + N <= D) {
#pragma unroll
      for (int q = 0; q < N; q += 4) {
        const F4u u = *reinterpret_cast<const F4u *>(row + k + q);
        v[q] = u.x, v[q + 1] = u.y, v[q + 2] = u.z, v[q + 3] = u.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) v[e] = k + e < D ? row[min(k + e, D - 1)] : 0.f;
    }
  };
  for (int item = blockIdx.x; item < blocks * shares; item += gridDim.x) {
    const int blk = item / shares, share = item - blk * shares;
    const float *arow = x + int64_t(list[min(blk * kExT + ar, rows - 1)]) * D;
    double best[4];
    int32_t bid[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      best[i] = double(kFarthest);
      bid[i] = kNoCentre;
    }
    for (int t = share * per; t < min(tiles, share * per + per); ++t) {
      const int c0 = t * T;
      const float *brow = cen + int64_t(min(c0 + br, nlist - 1)) * D;
      double acc[4][TJ] = {};
      float a[AE], b[BE];   // the next slab, on its way while one is multiplied
      load(arow, ak, a, std::integral_constant<int, AE>());
      load(brow, bk, b, std::integral_constant<int, BE>());
      for (int k0 = 0; k0 < D; k0 += K) {
        __syncthreads();   // the previous slab is done with
#pragma unroll
        for (int e = 0; e < AE; ++e) As[ak + e][ar] = double(a[e]);
#pragma unroll
        for (int e = 0; e < BE; ++e) Bs[bk + e][br] = double(b[e]);
        __syncthreads();
        if (k0 + K < D) {
          load(arow, k0 + K + ak, a, std::integral_constant<int, AE>());
          load(brow, k0 + K + bk, b, std::integral_constant<int, BE>());
        }
#pragma unroll 4
        for (int kk = 0; kk < K; ++kk) {
          double av[4], bv[TJ];
#pragma unroll
          for (int i = 0; i < 4; ++i) av[i] = As[kk][ty * 4 + i];
#pragma unroll
          for (int j = 0; j < TJ; ++j) bv[j] = Bs[kk][tx * TJ + j];
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[i][j] = fma(av[i], bv[j], acc[i][j]);
        }
      }
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const int c = c0 + tx * TJ + j;
        const double cn = c < nlist ? norm[c] : double(__builtin_inff());
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double v = fma(-2.0, acc[i][j], cn);
          if (v < best[i]) {   // centres visited in increasing order
            best[i] = v;
            bid[i] = c;
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      for (int off = 8; off >= 1; off >>= 1) {
        const double ov = __shfl_xor(best[i], off, 64);
        const int32_t oi = __shfl_xor(bid[i], off, 64);
        if (ov < best[i] || (ov == best[i] && oi < bid[i])) {
          best[i] = ov;
          bid[i] = oi;
        }
      }
    if (tx == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int at = blk * kExT + ty * 4 + i;
        if (at >= rows) continue;
        if (shares == 1) {
          out_ids[list[at]] = bid[i];
        } else {   // blocks * shares <= kExGrid
          part_v[share * (blocks * kExT) + at] = best[i];
          part_i[share * (blocks * kExT) + at] = bid[i];
        }
      }
    }
  }
}
__global__ void __launch_bounds__(256) k_assign_exact(const float *__restrict__ x, int D,
                                                      const float *__restrict__ cen, int nlist,
                                                      const double *__restrict__ norm,
                                                      const int32_t *__restrict__ list,
                                                      const int32_t *__restrict__ n_listed,
                                                      double *__restrict__ part_v,
                                                      int32_t *__restrict__ part_i,
                                                      int32_t *__restrict__ out_ids) {
  __shared__ double lds[kExLds];
  const int rows = *n_listed;
  if (rows <= kExFew) exact_items<1>(x, D, cen, nlist, norm, list, rows, lds, part_v, part_i, out_ids);
  else exact_items<4>(x, D, cen, nlist, norm, list, rows, lds, part_v, part_i, out_ids);
}
// The listed row at place `at`: its centre (by a whole wavefront, in every lane).
__device__ __forceinline__ int32_t exact_id(int at, int rows, int nlist, const double *part_v,
                                            const int32_t *part_i) {
  const int stride = (rows + kExT - 1) / kExT * kExT, shares = exact_shares(rows, nlist);
  double v = double(kFarthest);
  int32_t id = kNoCentre;
  for (int s = threadIdx.x & 63; s < shares; s += 64) {   // in increasing order of the centres
    const double ov = part_v[s * stride + at];
    const int32_t oi = part_i[s * stride + at];
    if (ov < v) {
      v = ov;
      id = oi;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const double ov = __shfl_xor(v, off, 64);
    const int32_t oi = __shfl_xor(id, off, 64);
    if (ov < v || (ov == v && oi < id)) {
      v = ov;
      id = oi;
    }
  }
  return id;
}

// Without distances: the listed rows' centres from their shares, one wavefront
// per row.
__global__ void __launch_bounds__(256) k_assign_listed(const int32_t *__restrict__ list,
                                                       const int32_t *__restrict__ n_listed, int nlist,
                                                       const double *__restrict__ part_v,
                                                       const int32_t *__restrict__ part_i,
                                                       int32_t *__restrict__ out_ids) {
  const int rows = *n_listed;
  if (exact_shares(rows, nlist) == 1) return;   // already written
  for (int at = blockIdx.x * 4 + (threadIdx.x >> 6); at < rows; at += gridDim.x * 4) {
    const int32_t id = exact_id(at, rows, nlist, part_v, part_i);
    if ((threadIdx.x & 63) == 0) out_ids[list[at]] = id;
  }
}

// With distances: one wavefront per row, the same, and ||x - c||^2 summed in
// float64.  A row with an infinity has no finite distance (NaN, as inf - inf
// in ||x||^2 + (||c||^2 - 2 <x, c>)); one without a centre gets ||x||^2 + 3.4e38.
__global__ void __launch_bounds__(256) k_assign_finish(const float *__restrict__ x, int64_t n, int D,
                                                       const float *__restrict__ cen, int nlist,
                                                       const int32_t *__restrict__ n_listed,
                                                       const double *__restrict__ part_v,
                                                       const int32_t *__restrict__ part_i,
                                                       int32_t *__restrict__ out_ids,
                                                       float *__restrict__ out_d) {
  const int lane = threadIdx.x & 63;
  const int64_t row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  int32_t id = out_ids[row];
  if (id < 0) {
    id = exact_id(~id, *n_listed, nlist, part_v, part_i);
    if (lane == 0) out_ids[row] = id;
  }
  const bool has = id < nlist;
  const float *xr = x + row * D;
  const float *cr = cen + int64_t(has ? id : 0) * D;
  double s = 0.0;
  for (int k = lane * 4; k < D; k += 256) {
    float v[4], c[4];
    if (k + 4 <= D) {
      const F4u a = *reinterpret_cast<const F4u *>(xr + k), b = *reinterpret_cast<const F4u *>(cr + k);
      v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w;
      c[0] = b.x, c[1] = b.y, c[2] = b.z, c[3] = b.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = k + e < D ? xr[k + e] : 0.f;
        c[e] = k + e < D ? cr[k + e] : 0.f;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double d = has ? double(v[e]) - double(c[e]) : double(v[e]);
      s = fma(d, d, s);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) {
    if (!has) out_d[row] = float(s) + kFarthest;
    else out_d[row] = s < double(__builtin_inff()) ? float(s) : __builtin_nanf("");
  }
}

// Whether an assignment runs on split float16: where that was faster than the
// float32 kernels at the numbers of rows measured (128 to 1,000,000).  Us,
// float32 against split: rows that are whole 16-byte runs (matrix kernel, tiles of
// 128 centres) 65,536 x 16 by 1,024 69, 92, by 4,096 201, 184; 65,536 x 128 by 512
// 102, 110, by 768 137, 128; 65,536 x 512 by 300 248, 253, by 512 314, 262; 128 x 768
// by 4,096 1,872, 139; many rows 131,072 x 64 by 200 87, 102, x 128 by 128 92, 123, by
// 200 130, 124; 500,000 x 768 by 128 1,258, 1,481, by 129 2,024, 1,482.  Other rows
// (vector ALU, tiles of 64) 65,536 x 33 by 512 72, 84, by 2,048 230, 147; 8,192 x 99 by
// 60 41, 60, by 256 74, 45; 8,192 x 150 by 60 58, 66; 8,192 x 230 by 16 86, 84; many
// rows 65,536 x 49 by 256 61, 61; x 99 by 60 76, 77, by 128 95, 77; x 150 by 16 136, 87.
// Below 16 coordinates many centres are within the margin of the nearest (65,536
// x 1 by 20,000 770, 2,762).
static bool assign_on_split(int64_t n, int dim, int nlist) {
  if (dim < 16 || dim > kSplitMaxDim || n < 128) return false;
  const int64_t table = int64_t(nlist) * dim;
  if (dim % 4 == 0)
    return nlist >= 4096 || (nlist >= 512 && table >= 98304) || (n >= 131072 && nlist > 128 && dim >= 128);
  return dim >= 200 || table >= 24576 || (n >= 65536 && (dim >= 128 || table >= 12600));
}

// How a call is cut: pieces of `rows` rows, groups of `tiles` tiles of centres
// (whose halves are in the workspace at a time), `shares` workgroups along a
// group's centres.  A plan is made for a number of bytes; what does not fit in
// them at once goes in more pieces and groups, with the same results.
constexpr size_t kSplitBudget = size_t(64) << 20;
struct SplitPlan {
  int64_t rows;   // 0: no plan
  int tiles, groups, shares, per_share, n_slab;
  size_t tab, split, list, parts, exact, bytes;   // offsets
};
static SplitPlan split_layout(int64_t rows, int tiles, int dim, int nlist) {
  SplitPlan p{};
  const int all = (nlist + kSpN - 1) / kSpN;
  p.rows = rows;
  p.tiles = tiles;
  p.groups = (all + tiles - 1) / tiles;
  p.n_slab = (dim + kSpK - 1) / kSpK;
  // the centres are shared out where the rows alone leave compute units idle
  const int64_t blocks = (rows + kSpM - 1) / kSpM;
  const int want = int(std::min<int64_t>(tiles, (512 + blocks - 1) / blocks));
  p.per_share = (tiles + want - 1) / want;
  p.shares = (tiles + p.per_share - 1) / p.per_share;
  size_t off = 0;
  auto take = [&](size_t b) {
    const size_t at = off;
    off += (b + 255) / 256 * 256;
    return at;
  };
  p.exact = take(size_t(kExParts) * (sizeof(double) + sizeof(int32_t)));
  p.tab = take(size_t(all) * kSpN * (4 * sizeof(float) + sizeof(double)));
  p.split = take(size_t(tiles) * kSpN * p.n_slab * 2 * kSpK * sizeof(_Float16));
  p.list = take((size_t(rows) + 64) * 4);   // the length, then the rows
  p.parts = take(size_t(rows) * 4 + size_t(p.groups) * p.shares * rows * 12);
  p.bytes = off;
  return p;
}
static SplitPlan split_plan(int64_t n, int dim, int nlist, size_t budget) {
  const int all = (nlist + kSpN - 1) / kSpN;
  const int64_t least = std::min<int64_t>(n, 4096);   // a smaller piece does not pay
  int64_t rows = std::min<int64_t>(n, int64_t(1) << 24);
  for (int tiles = all; tiles >= 1; tiles = (tiles + 1) / 2) {
    for (int64_t r = rows; r >= least; r = r > least ? std::max(least, (r / 2 + 255) / 256 * 256) : 0) {
      const SplitPlan p = split_layout(r, tiles, dim, nlist);
      if (p.bytes <= budget) return p;
    }
    if (tiles == 1) break;
  }
  return SplitPlan{};
}

static int launch_assign_split(const SplitPlan &p, const float *x, int64_t n, int dim, const float *cen,
                               int nlist, int32_t *out_ids, float *out_d, void *ws, hipStream_t s) {
  char *w = static_cast<char *>(ws);
  const int all = (nlist + kSpN - 1) / kSpN;
  const size_t np = size_t(all) * kSpN;
  double *part_v = reinterpret_cast<double *>(w + p.exact);
  int32_t *part_i = reinterpret_cast<int32_t *>(part_v + kExParts);
  CentreTab tab;
  tab.norm = reinterpret_cast<double *>(w + p.tab);
  tab.base = reinterpret_cast<float *>(tab.norm + np);
  tab.along = tab.base + np;
  tab.margin = tab.along + np;
  tab.mul = tab.margin + np;
  _Float16 *split = reinterpret_cast<_Float16 *>(w + p.split);
  int32_t *n_listed = reinterpret_cast<int32_t *>(w + p.list), *list = n_listed + 64;
  float *xnorm = reinterpret_cast<float *>(w + p.parts);
  const int shares = p.groups * p.shares;
  for (int64_t r0 = 0; r0 < n; r0 += p.rows) {
    const int64_t m = std::min(p.rows, n - r0);
    const float *xp = x + r0 * dim;
    int st;
    SplitPart part;
    part.w1 = xnorm + p.rows;
    part.w2 = part.w1 + int64_t(shares) * m;
    part.id = reinterpret_cast<int32_t *>(part.w2 + int64_t(shares) * m);
    int done = 0;
    for (int g = 0; g < p.groups; ++g) {
      const int t0 = g * p.tiles, nt = std::min(p.tiles, all - t0);
      const int sh = (nt + p.per_share - 1) / p.per_share;
      hipLaunchKernelGGL(k_split_centres, dim3(unsigned(nt * kSpN / 4)), dim3(256), 0, s, cen, nlist, dim,
                         p.n_slab, t0 * kSpN, tab, split, n_listed);
      if ((st = check_launch())) return st;
      SplitPart pg{part.w1 + done * m, part.w2 + done * m, part.id + done * m};
      hipLaunchKernelGGL(k_assign_split, dim3(unsigned((m + kSpM - 1) / kSpM), unsigned(sh)),
                         dim3(kSpThreads), 0, s, xp, m, dim, p.n_slab, t0 * kSpN, tab, split, nt,
                         p.per_share, pg, xnorm);
      if ((st = check_launch())) return st;
      done += sh;
    }
    int32_t *ids = out_ids + r0;
    hipLaunchKernelGGL(k_assign_decide, dim3(unsigned((m + 255) / 256)), dim3(256), 0, s, m, done, part,
                       xnorm, tab, list, n_listed, ids);
    if ((st = check_launch())) return st;
    hipLaunchKernelGGL(k_assign_exact, dim3(kExGrid), dim3(256), 0, s, xp, dim, cen, nlist, tab.norm,
                       list, n_listed, part_v, part_i, ids);
    if ((st = check_launch())) return st;
    if (out_d)
      hipLaunchKernelGGL(k_assign_finish, dim3(unsigned((m + 3) / 4)), dim3(256), 0, s, xp, m, dim, cen,
                         nlist, n_listed, part_v, part_i, ids, out_d + r0);
    else
      hipLaunchKernelGGL(k_assign_listed, dim3(256), dim3(256), 0, s, list, n_listed, nlist, part_v,
                         part_i, ids);
    if ((st = check_launch())) return st;
  }
  return RSLM_OK;
}

// The least workspace a call accepts: the float32 kernels' scratch.
static size_t probe_min_workspace(int64_t n, int32_t nlist, int mode) {
  const size_t norms = (size_t(nlist) * sizeof(float) + 255) / 256 * 256;
  if (mode == IVF_ASSIGN_L2) return norms;
  return norms + (size_t(n) * size_t(nlist) * sizeof(float) + 255) / 256 * 256;
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
  const size_t least = probe_min_workspace(n, nlist, mode);
  if (mode == IVF_ASSIGN_L2 && dim >= 1 && nlist <= 65536 && assign_on_split(n, dim, nlist))
    return std::max(least, split_plan(n, dim, nlist, kSplitBudget).bytes);
  return least;
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
  if (mode == IVF_ASSIGN_L2 && assign_on_split(n, dim, nlist) &&
      (reinterpret_cast<uintptr_t>(ws) & 15) == 0) {
    // (a workspace too small for pieces of a useful size takes the float32 kernels)
    const SplitPlan pl = split_plan(n, dim, nlist, std::min(ws_bytes, kSplitBudget));
    if (pl.rows > 0)
      return launch_assign_split(pl, x, n, dim, centroids, nlist, out_ids, out_scores, ws, s);
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

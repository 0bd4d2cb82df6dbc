// Register-resident rotation for dimensions that are a multiple of the
// 128-element block (D = 128 NB, NB = 1, 2, 3, 4, 6, 8, 12, 16).
//
// Same arithmetic as the general path (paper, Section "Pre-Quantization
// Transformations": S1, block FWHT, permutation + strided transpose, S2,
// block FWHT), different mapping: lane l of a wavefront holds elements
// e = l + 64 j (j < J = D / 64), so element bits 0..5 are the lane and bit 6
// of the block index is j's parity.  The six lane-bit butterfly stages use
// cross-lane exchanges, the seventh is in registers, and LDS is touched only
// by the strided transpose between the passes.
#include "rows_dev.h"

namespace rslm {

__device__ __forceinline__ int px_r(int i) { return i + (i >> 5); }

// Orthonormal FWHT of every 128-block of the register vector.
template <int J>
__device__ __forceinline__ void fwht128_reg(float (&x)[J], int lane) {
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) {
    const float sg = (lane & s) ? -1.f : 1.f;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const float p = __shfl_xor(x[j], s, 64);
      x[j] = fmaf(sg, x[j], p);   // lane bit clear: x + p; set: p - x
    }
  }
  constexpr float kInv = 0.08838834764831845f;   // 1 / sqrt(128)
#pragma unroll
  for (int j = 0; j < J; j += 2) {
    const float a = x[j], b = x[j + 1];
    x[j] = (a + b) * kInv;
    x[j + 1] = (a - b) * kInv;
  }
}

// Per-lane sign words: element j of the lane takes sign word w[j mod 4]
// (the sign index pattern repeats every 256 = 4 x 64 elements).
struct SignWords {
  uint32_t w[4];
};
__device__ __forceinline__ SignWords sign_words(uint32_t bits) {
  SignWords s;
#pragma unroll
  for (int t = 0; t < 4; ++t) s.w[t] = ((bits >> t) & 1u) << 31;
  return s;
}
__device__ __forceinline__ float flipw(float v, const SignWords &s, int j) {
  return __uint_as_float(__float_as_uint(v) ^ s.w[j & 3]);
}

// Forward rotation of x (already multiplied by S1) through buf (LDS, >= D +
// D/32 floats) for the transpose; ts[o] = byte offset in buf of the source of
// output o.
template <int J>
__device__ __forceinline__ void rotate_fwd_reg(float (&x)[J], const RotParams &rp,
                                               const uint16_t *ts, const SignWords &s2, float *buf,
                                               int lane) {
  if (rp.passes == 0) return;
  fwht128_reg<J>(x, lane);
  if (rp.passes == 1) return;
#pragma unroll
  for (int j = 0; j < J; ++j) buf[px_r(lane + 64 * j)] = x[j];
  wave_sync_r();
#pragma unroll
  for (int j = 0; j < J; ++j) x[j] = flipw(lds_at(buf, ts[lane + 64 * j]), s2, j);
  wave_sync_r();
  fwht128_reg<J>(x, lane);
}

// Inverse rotation R^T (without the final S1, applied by the caller).
template <int J>
__device__ __forceinline__ void rotate_inv_reg(float (&x)[J], const RotParams &rp,
                                               const uint16_t *ts, const SignWords &s2, float *buf,
                                               int lane) {
  if (rp.passes == 0) return;
  fwht128_reg<J>(x, lane);
  if (rp.passes == 1) return;
#pragma unroll
  for (int j = 0; j < J; ++j) lds_at(buf, ts[lane + 64 * j]) = flipw(x[j], s2, j);
  wave_sync_r();
#pragma unroll
  for (int j = 0; j < J; ++j) x[j] = buf[px_r(lane + 64 * j)];
  wave_sync_r();
  fwht128_reg<J>(x, lane);
}

// Workgroup prologue: LDS copy of the transpose source table (D entries), as
// byte offsets into the padded per-wave buffer.
// D = 64 J entries, 256 threads: all loads first (clamped index), then the
// stores.
template <int J>
__device__ __forceinline__ void load_tsrc_r(const RotParams &rp, uint16_t *ts) {
  constexpr int D = 64 * J, kU = (D + 255) / 256;
  if (rp.passes == 2) {
    int16_t tv[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) tv[u] = rp.tsrc[min(int(threadIdx.x) + 256 * u, D - 1)];
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (int(threadIdx.x) + 256 * u < D) ts[threadIdx.x + 256 * u] = uint16_t(4 * px_r(tv[u]));
  }
  __syncthreads();
}

template <int J>
__global__ void __launch_bounds__(256) k_rotate_reg(const float *__restrict__ x, float *y,
                                                    int64_t n, RotParams rp, int inverse,
                                                    int dstride) {
  extern __shared__ float lds[];
  __shared__ uint16_t ts[64 * J];
  load_tsrc_r<J>(rp, ts);
  const int lane = threadIdx.x & 63;
  const int wid = threadIdx.x >> 6;
  const int64_t row = int64_t(blockIdx.x) * (blockDim.x >> 6) + wid;
  if (row >= n) return;   // no workgroup barriers below
  float *buf = lds + wid * dstride;
  const uint2 sm = lane_sign_masks(rp, lane);
  const SignWords s1 = sign_words(rp.passes > 0 ? sm.x : 0u), s2 = sign_words(sm.y);
  const float *xr = x + row * (64 * J);
  float v[J];
#pragma unroll
  for (int j = 0; j < J; ++j) v[j] = xr[lane + 64 * j];
  if (!inverse) {
#pragma unroll
    for (int j = 0; j < J; ++j) v[j] = flipw(v[j], s1, j);
    rotate_fwd_reg<J>(v, rp, ts, s2, buf, lane);
  } else {
    rotate_inv_reg<J>(v, rp, ts, s2, buf, lane);
#pragma unroll
    for (int j = 0; j < J; ++j) v[j] = flipw(v[j], s1, j);
  }
  float *yr = y + row * (64 * J);
#pragma unroll
  for (int j = 0; j < J; ++j) yr[lane + 64 * j] = v[j];
}

// Launchers: return false when D is not handled here.
#define RSLM_REG_SWITCH(NB, CALL) \
  switch (NB) {                   \
    case 1: CALL(2); break;       \
    case 2: CALL(4); break;       \
    case 3: CALL(6); break;       \
    case 4: CALL(8); break;       \
    case 6: CALL(12); break;      \
    case 8: CALL(16); break;      \
    case 12: CALL(24); break;     \
    case 16: CALL(32); break;     \
    default: return false;        \
  }

bool reg_path_ok(const RotParams &rp) {
  if (rp.B != 128 || rp.overlap || rp.D % 128) return false;
  const int nb = rp.D / 128;
  return nb == 1 || nb == 2 || nb == 3 || nb == 4 || nb == 6 || nb == 8 || nb == 12 || nb == 16;
}

static int reg_dstride(int D) { return (D + (D >> 5) + 4 + 3) / 4 * 4; }

bool launch_rotate_reg(const rslm_plan *p, const float *x, float *y, int64_t n, int inverse,
                       hipStream_t s) {
  if (!reg_path_ok(p->rot)) return false;
  const int dstride = reg_dstride(p->rot.D);
  const int waves = 4;
  const size_t shm = size_t(waves) * dstride * sizeof(float);
  const unsigned grid = unsigned((n + waves - 1) / waves);
#define CALL(J)                                                                            \
  hipLaunchKernelGGL((k_rotate_reg<J>), dim3(grid), dim3(64 * waves), shm, s, x, y, n, p->rot, \
                     inverse, dstride)
  RSLM_REG_SWITCH(p->rot.D / 128, CALL)
#undef CALL
  return true;
}

}  // namespace rslm

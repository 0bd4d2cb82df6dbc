// IVF partition training: one Lloyd update of the partition centres.
//
// Paper, Section "End-to-End Comparison with Faiss and ScaNN", Setup: the
// collection is partitioned by Euclidean k-means (about 256 sample points
// per centre).  One iteration assigns every point to its nearest centre
// (ivf_assign_probe, IVF_ASSIGN_L2) and then moves each centre to the mean of
// its points; a centre with no points keeps its position.  This file is the
// second half of the iteration.
//
// GPU design.  The point indices are counting-sorted by centre (counts by
// integer atomics, one exclusive scan, placement through a per-centre
// cursor), so each centre's points are one contiguous run of indices.  Then
// one workgroup per (centre, 256 coordinates) walks its run: each thread owns
// one coordinate and adds the points' values in float64 (a point's row is
// read as one coalesced 1 KiB segment per workgroup), and divides once by
// the count.  With float64 sums, the order in which atomics placed a
// centre's points only moves the sum by float64 roundings; the result is
// rounded to float32 once.
//
// Few centres would leave most of the chip idle and every atomic on a handful
// of addresses, so then a centre's run is shared by several workgroups
// (partial float64 sums in the workspace, added by k_km_final) and counts and
// places are taken per workgroup in LDS, with one global atomic per workgroup
// and centre.
#include <algorithm>

#include "rslm_internal.h"

namespace rslm {

constexpr int kKmThreads = 256;
constexpr int kKmScanThreads = 1024;

constexpr int kKmLdsLists = 4096;   // centres counted in LDS

struct KmWs {
  int32_t *counts, *cursor, *offsets, *order;
  double *partial;        // shares x nlist x dim sums
  size_t bytes, min_bytes;   // min_bytes: without the partial sums
};

// Workgroups that share one centre's points: enough for about 2,048 in all, and
// at least 64 points each on average.  Whole update, us, one share and global
// counters against these: 4,000,000 x 64 by 16 56,668 -> 327; 262,794 x 810 by 27
// 2,407 -> 202; 1,011,082 x 922 by 188 2,093 -> 792 (reading x once: 782).
static int km_shares(int64_t n, int dim, int nlist) {
  const int64_t have = int64_t(nlist) * ((dim + kKmThreads - 1) / kKmThreads);
  const int64_t want = (2048 + have - 1) / have, most = n / (int64_t(nlist) * 64);
  return int(std::max<int64_t>(1, std::min<int64_t>({want, most, 256})));
}
// Counting per workgroup in LDS pays where each of its 512 workgroups has
// several points per centre.
static bool km_lds(int64_t n, int nlist) {
  return nlist <= kKmLdsLists && n / 512 >= 4 * int64_t(nlist);
}

static size_t km_align(size_t b) { return (b + 255) / 256 * 256; }

static KmWs km_ws_layout(void *base, int64_t n, int nlist) {
  KmWs w{};
  char *p = static_cast<char *>(base);
  size_t off = 0;
  auto take = [&](size_t b) {
    char *r = p ? p + off : nullptr;
    off += km_align(b);
    return reinterpret_cast<int32_t *>(r);
  };
  w.counts = take(size_t(nlist) * 4);
  w.cursor = take(size_t(nlist) * 4);
  w.offsets = take(size_t(nlist + 1) * 4);
  w.order = take(size_t(n > 0 ? n : 1) * 4);
  w.min_bytes = off;
  // shares > 1 means fewer than 2,048 (centre, 256 coordinates) pairs, doubled at
  // most by rounding the shares up
  if (nlist < 2048 && n >= 128 * int64_t(nlist))
    w.partial = reinterpret_cast<double *>(take(size_t(4096) * kKmThreads * sizeof(double)));
  w.bytes = off;
  return w;
}

__global__ void __launch_bounds__(kKmThreads) k_km_zero(int32_t *__restrict__ counts,
                                                        int32_t *__restrict__ cursor, int nlist) {
  const int i = blockIdx.x * kKmThreads + threadIdx.x;
  if (i < nlist) {
    counts[i] = 0;
    cursor[i] = 0;
  }
}

// Points per centre; assignments outside [0, nlist) are ignored.
__global__ void __launch_bounds__(kKmThreads) k_km_count(const int32_t *__restrict__ assign,
                                                         int64_t n, int nlist,
                                                         int32_t *__restrict__ counts) {
  const int64_t stride = int64_t(gridDim.x) * kKmThreads;
  for (int64_t i = int64_t(blockIdx.x) * kKmThreads + threadIdx.x; i < n; i += stride) {
    const int a = assign[i];
    if (a >= 0 && a < nlist) atomicAdd(&counts[a], 1);
  }
}

// The same for few centres: 512 workgroups, each over a run of consecutive
// points, count in LDS and add what they found once per centre.
__global__ void __launch_bounds__(kKmThreads) k_km_count_lds(const int32_t *__restrict__ assign,
                                                             int64_t n, int nlist,
                                                             int32_t *__restrict__ counts) {
  extern __shared__ int32_t hist[];
  for (int c = threadIdx.x; c < nlist; c += kKmThreads) hist[c] = 0;
  __syncthreads();
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t a = blockIdx.x * per, b = min(n, a + per);
  for (int64_t i = a + threadIdx.x; i < b; i += kKmThreads) {
    const int c = assign[i];
    if (c >= 0 && c < nlist) atomicAdd(&hist[c], 1);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < nlist; c += kKmThreads)
    if (hist[c]) atomicAdd(&counts[c], hist[c]);
}

// Exclusive prefix of the counts (one workgroup): thread t sums a run of
// consecutive centres, the runs' totals are scanned by wavefront shuffles and
// then across the wavefronts, and each thread writes its run's offsets.
__global__ void __launch_bounds__(kKmScanThreads) k_km_scan(const int32_t *__restrict__ counts,
                                                            int nlist,
                                                            int32_t *__restrict__ offsets) {
  __shared__ int32_t part[kKmScanThreads / 64];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int per = (nlist + kKmScanThreads - 1) / kKmScanThreads;
  const int a = min(nlist, t * per), b = min(nlist, a + per);
  int sum = 0;
  for (int i = a; i < b; ++i) sum += counts[i];
  int incl = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(incl, off, 64);
    if (lane >= off) incl += v;
  }
  if (lane == 63) part[wv] = incl;
  __syncthreads();
  int before = 0, total = 0;
  for (int w = 0; w < kKmScanThreads / 64; ++w) {
    before += w < wv ? part[w] : 0;
    total += part[w];
  }
  int run = before + incl - sum;
  for (int i = a; i < b; ++i) {
    offsets[i] = run;
    run += counts[i];
  }
  if (t == 0) offsets[nlist] = total;
}

// Point i takes the next slot of its centre's run.
__global__ void __launch_bounds__(kKmThreads) k_km_place(const int32_t *__restrict__ assign,
                                                         int64_t n, int nlist,
                                                         const int32_t *__restrict__ offsets,
                                                         int32_t *__restrict__ cursor,
                                                         int32_t *__restrict__ order) {
  const int64_t stride = int64_t(gridDim.x) * kKmThreads;
  for (int64_t i = int64_t(blockIdx.x) * kKmThreads + threadIdx.x; i < n; i += stride) {
    const int a = assign[i];
    if (a >= 0 && a < nlist) order[offsets[a] + atomicAdd(&cursor[a], 1)] = int32_t(i);
  }
}

// The same for few centres: each workgroup counts its run of points again,
// reserves its part of every centre's run with one atomic, and places its
// points there through LDS cursors.
__global__ void __launch_bounds__(kKmThreads) k_km_place_lds(const int32_t *__restrict__ assign,
                                                             int64_t n, int nlist,
                                                             const int32_t *__restrict__ offsets,
                                                             int32_t *__restrict__ cursor,
                                                             int32_t *__restrict__ order) {
  extern __shared__ int32_t hist[];
  for (int c = threadIdx.x; c < nlist; c += kKmThreads) hist[c] = 0;
  __syncthreads();
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t a = blockIdx.x * per, b = min(n, a + per);
  for (int64_t i = a + threadIdx.x; i < b; i += kKmThreads) {
    const int c = assign[i];
    if (c >= 0 && c < nlist) atomicAdd(&hist[c], 1);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < nlist; c += kKmThreads)
    if (hist[c]) hist[c] = offsets[c] + atomicAdd(&cursor[c], hist[c]);
  __syncthreads();
  for (int64_t i = a + threadIdx.x; i < b; i += kKmThreads) {
    const int c = assign[i];
    if (c >= 0 && c < nlist) order[atomicAdd(&hist[c], 1)] = int32_t(i);
  }
}

// Workgroup (centre L, coordinate block y, share z): thread d' sums coordinate
// d = 256 y + d' over its share of the centre's points in float64 (eight rows
// in flight), then writes the mean, or with several shares the sum; an empty
// centre is left as it is.
__global__ void __launch_bounds__(kKmThreads) k_km_mean(const float *__restrict__ x, int dim,
                                                        const int32_t *__restrict__ offsets,
                                                        const int32_t *__restrict__ counts,
                                                        const int32_t *__restrict__ order,
                                                        float *__restrict__ centroids,
                                                        double *__restrict__ partial) {
  const int L = blockIdx.x;
  const int d = blockIdx.y * kKmThreads + threadIdx.x;
  const int cnt = counts[L];
  if (cnt <= 0 || d >= dim) return;
  const int32_t *run = order + offsets[L];
  const int per = (cnt + gridDim.z - 1) / gridDim.z;
  int j = min(cnt, int(blockIdx.z) * per);
  const int end = min(cnt, j + per);
  double s[8] = {};
  for (; j + 8 <= end; j += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x[int64_t(run[j + u]) * dim + d];
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u] += double(v[u]);
  }
  if (j + 4 <= end) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = x[int64_t(run[j + u]) * dim + d];
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] += double(v[u]);
    j += 4;
  }
  for (; j < end; ++j) s[0] += double(x[int64_t(run[j]) * dim + d]);
  const double sum = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
  if (partial) partial[(int64_t(blockIdx.z) * gridDim.x + L) * dim + d] = sum;
  else centroids[int64_t(L) * dim + d] = float(sum / double(cnt));
}

// Means from the shares' sums.
__global__ void __launch_bounds__(kKmThreads) k_km_final(const double *__restrict__ partial, int shares,
                                                         int dim, const int32_t *__restrict__ counts,
                                                         float *__restrict__ centroids) {
  const int L = blockIdx.x;
  const int d = blockIdx.y * kKmThreads + threadIdx.x;
  const int cnt = counts[L];
  if (cnt <= 0 || d >= dim) return;
  double sum = 0.0;
  for (int z = 0; z < shares; ++z) sum += partial[(int64_t(z) * gridDim.x + L) * dim + d];
  centroids[int64_t(L) * dim + d] = float(sum / double(cnt));
}

}  // namespace rslm

using namespace rslm;

extern "C" {

size_t ivf_kmeans_update_workspace(int64_t n, int32_t nlist) {
  if (n < 0 || nlist < 1) return 0;
  return km_ws_layout(nullptr, n, nlist).bytes;
}

int ivf_kmeans_update(const float *x, int64_t n, int32_t dim, const int32_t *assign,
                      int32_t nlist, float *centroids, void *ws, size_t ws_bytes,
                      void *stream) {
  if (n < 0 || n > 0x7fffffff || dim < 1 || dim > (1 << 20) || nlist < 1 || nlist > 65536)
    return RSLM_ERR_INVALID_ARG;
  if (!centroids) return RSLM_ERR_INVALID_ARG;
  if (n == 0) return RSLM_OK;
  if (!x || !assign) return RSLM_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(x) & 3) || (reinterpret_cast<uintptr_t>(assign) & 3) ||
      (reinterpret_cast<uintptr_t>(centroids) & 3))
    return RSLM_ERR_INVALID_ARG;
  const KmWs w = km_ws_layout(ws, n, nlist);
  if (!ws || ws_bytes < w.min_bytes) return RSLM_ERR_WORKSPACE;
  // (without room for partial sums, or where they would not be aligned, a
  // centre's points are not shared out)
  const bool part = w.partial && ws_bytes >= w.bytes && (reinterpret_cast<uintptr_t>(ws) & 7) == 0;
  const int shares = part ? km_shares(n, dim, nlist) : 1;
  hipStream_t s = as_stream(stream);
  int st;
  hipLaunchKernelGGL(k_km_zero, dim3(unsigned((nlist + kKmThreads - 1) / kKmThreads)),
                     dim3(kKmThreads), 0, s, w.counts, w.cursor, nlist);
  if ((st = check_launch())) return st;
  const unsigned grid = unsigned(std::min<int64_t>((n + kKmThreads - 1) / kKmThreads, 4096));
  const bool lds = km_lds(n, nlist);
  const size_t shm = size_t(nlist) * 4;
  if (lds)
    hipLaunchKernelGGL(k_km_count_lds, dim3(512), dim3(kKmThreads), shm, s, assign, n, nlist, w.counts);
  else
    hipLaunchKernelGGL(k_km_count, dim3(grid), dim3(kKmThreads), 0, s, assign, n, nlist, w.counts);
  if ((st = check_launch())) return st;
  hipLaunchKernelGGL(k_km_scan, dim3(1), dim3(kKmScanThreads), 0, s, w.counts, nlist, w.offsets);
  if ((st = check_launch())) return st;
  if (lds)
    hipLaunchKernelGGL(k_km_place_lds, dim3(512), dim3(kKmThreads), shm, s, assign, n, nlist, w.offsets,
                       w.cursor, w.order);
  else
    hipLaunchKernelGGL(k_km_place, dim3(grid), dim3(kKmThreads), 0, s, assign, n, nlist, w.offsets,
                       w.cursor, w.order);
  if ((st = check_launch())) return st;
  const unsigned gy = unsigned((dim + kKmThreads - 1) / kKmThreads);
  hipLaunchKernelGGL(k_km_mean, dim3(unsigned(nlist), gy, unsigned(shares)), dim3(kKmThreads), 0, s, x, dim,
                     w.offsets, w.counts, w.order, centroids, shares > 1 ? w.partial : nullptr);
  if (shares > 1) {
    if ((st = check_launch())) return st;
    hipLaunchKernelGGL(k_km_final, dim3(unsigned(nlist), gy), dim3(kKmThreads), 0, s, w.partial, shares,
                       dim, w.counts, centroids);
  }
  return check_launch();
}

}  // extern "C"

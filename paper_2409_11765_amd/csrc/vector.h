// Matrix-vector products of one generation (d = R (m - x*), B z_w), 32 rows a
// workgroup.
#pragma once

#include <hip/hip_runtime.h>

namespace cmx {

// sum of count values, stride apart, in order; eight loads under way at a time
// (a loop over a count that is not known has one)
template <typename T>
__device__ __forceinline__ double sum_strided(const T* __restrict__ p, int64_t stride, int count) {
  double a = 0.0;
  for (int c = 0; c < count; c += 8) {
    T v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = p[stride * min(c + q, count - 1)];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (c + q < count) a += static_cast<double>(v[q]);
  }
  return a;
}

// Row row0 + (thread & 31) of M x, in threads 0..31 of 256 (x(j): column j's
// factor).  A row's sum is the sum over its chunks of 64 columns, in order, of each
// chunk's sum, in order: one chunk to a group of 32 threads, so all of n = 512 at
// once, in one launch where the chunks' sums took a second one (n = 200: 3.9 +
// 3.3 us and the gap between them, now 4-5, most of it the latency of the loads).
// Larger n spread the chunks over the GPU instead (kMvOneMax): 32 workgroups
// cannot draw 8 MB fast enough (n = 1000: 12.2 us against 4.9 and the second launch).
constexpr int kMvRows = 32, kMvGroups = 8, kMvOneMax = 512;
template <class X>
__device__ __forceinline__ double matvec_rows(int row0, int n, const double* __restrict__ M, int ld, X x) {
  constexpr int G = kMvGroups, COLS = 64 * G;
  __shared__ double xs[COLS];
  __shared__ double part[G][kMvRows];
  const int t = threadIdx.x, r = t & 31, g = t >> 5, i = row0 + r;
  const double* row = M + min(i, n - 1);
  double acc = 0.0;
  for (int j0 = 0; j0 < n; j0 += COLS) {
    const int c0 = j0 + 64 * g, c1 = min(n, c0 + 64);
    // half a chunk's loads are under way before the factors are there
    double v[32];
    auto load = [&](int c) {
#pragma unroll
      for (int q = 0; q < 32; ++q) v[q] = row[static_cast<int64_t>(min(c + q, n - 1)) * ld];
    };
    double s = 0.0;
    auto add = [&](int c) {
#pragma unroll
      for (int q = 0; q < 32; ++q)
        if (c + q < c1) s += v[q] * xs[c + q - j0];
    };
    load(c0);
    __syncthreads();
    for (int q = t; q < COLS; q += 32 * G)
      if (j0 + q < n) xs[q] = x(j0 + q);
    __syncthreads();
    add(c0);
    load(c0 + 32);
    add(c0 + 32);
    part[g][r] = s;
    __syncthreads();
    if (g == 0)
      for (int q = 0; q < G && j0 + 64 * q < n; ++q) acc += part[q][r];
  }
  return acc;
}

// d = R (m - x*) (R null: m - x*; x* null: the origin); workgroup b of
// shift_blocks(n, R)
struct ShiftArgs {
  int n;
  const double* R;
  int ldr;
  const double *m, *xstar;
  double *d, *part;  // part: ceil(n / 64) n, scratch for n > kMvOneMax
};
__device__ __forceinline__ double shift_of(const ShiftArgs& a, int j) {
  return a.m[j] - (a.xstar ? a.xstar[j] : 0.0);
}
__host__ __device__ inline int shift_blocks(int n, bool rotated) {
  return rotated ? (n + kMvRows - 1) / kMvRows : (n + 255) / 256;
}
__device__ __forceinline__ void shift_body(int b, const ShiftArgs& a) {
  auto u = [&](int j) { return shift_of(a, j); };
  if (a.R) {
    const double v = matvec_rows(b * kMvRows, a.n, a.R, a.ldr, u);
    const int i = b * kMvRows + threadIdx.x;
    if (threadIdx.x < kMvRows && i < a.n) a.d[i] = v;
  } else {
    const int i = b * 256 + threadIdx.x;
    if (i < a.n) a.d[i] = u(i);
  }
}

}  // namespace cmx

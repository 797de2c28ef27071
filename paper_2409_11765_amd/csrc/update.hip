// Ranking, recombination and the float64 vector updates of one generation
// (Alg. 1 'update' line, Sec. 2.1), plus the stopping tests (Sec. 2.2).
//
// Readings shared with the oracle (no formula is printed in the paper):
// tutorial default rates, positive weights w_1..w_mu summing to one, the
// cumulative step-size path p_sigma built from C^{-1/2} y_w = B z_w, the
// h_sigma stall of p_c, sigma <- sigma exp((cs/ds)(||p_sigma||/chi_n - 1)).
// All reductions use a fixed order (no floating-point atomics), so a run is
// bitwise reproducible.
#include "internal.h"
#include "vector.h"

namespace cmx {

namespace {

__device__ __forceinline__ double rank_key(double v) { return v != v ? __builtin_inf() : v; }

// ---- ranking by chunk sort and merge: the keys (f, index), NaN counted as
// +inf, are cut into chunks of kSortChunk; each chunk is sorted by a bitonic
// network (k_sort); the rank of a key is its position in its own chunk plus, for
// every other chunk, the number of that chunk's keys below it, found by binary
// search (k_merge, chunks taken kMergeGroup at a time from LDS); with more than
// kMergeGroup chunks the counts of several groups are summed by k_scatter.
// The keys are distinct, so the ranks form the stable ascending permutation
// exactly; the counts are integers.  The first kernel also sums up f from the
// fitness tiles, and the last one writes order[rank] = index and the best point:
// one launch up to lambda = 256 and two up to 2048, where the fitness sum, the
// sort, the counts, their scatter and the best point took four or five of 4-7 us.
constexpr int kSortChunk = 256, kMergeGroup = 8;

__device__ __forceinline__ bool key_less(double ka, int ia, double kb, int ib) {
  return ka < kb || (ka == kb && ia < ib);
}

// Best-so-far point and the f-history ring, before m and sigma move: called by
// every thread of a workgroup with its key's rank (negative: none), index and value.
template <typename T>
struct BestArgs {
  int n, lam;
  const T* Y;
  int ldy;
  const double* m;
  double *x_best, *hist;
  int hist_len;
  DevScalars* sc;
  int32_t* order;
};
template <typename T>
__device__ __forceinline__ void place(const BestArgs<T>& a, int rank, int i, double key) {
  __shared__ int first;
  if (threadIdx.x == 0) first = -1;
  __syncthreads();
  if (rank >= 0) {
    a.order[rank] = i;
    if (rank == a.lam - 1) a.sc->f_gen_max = key;
    if (rank == 0) first = threadIdx.x;
  }
  __syncthreads();
  if (first < 0) return;  // (uniform)
  __shared__ double f0s;
  __shared__ int i0s;
  if (static_cast<int>(threadIdx.x) == first) {
    f0s = key;
    i0s = i;
  }
  __syncthreads();
  const double f0 = f0s;
  const bool better = f0 < a.sc->f_best;
  if (better) {
    const double sigma = a.sc->sigma;
    const T* y = a.Y + static_cast<int64_t>(i0s) * a.ldy;
    for (int q = threadIdx.x; q < a.n; q += blockDim.x) a.x_best[q] = a.m[q] + sigma * static_cast<double>(y[q]);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a.hist[a.sc->hist_count % a.hist_len] = f0;
    a.sc->hist_count += 1;
    a.sc->f_gen_min = f0;
    if (better) a.sc->f_best = f0;
  }
}

// chunk c: f from `tiles` partial sums a point (tiles = 0: f is given), sorted; a
// padding key (+inf, INT_MAX) is above every real one.  Partners in a wave
// exchange by shuffles, and the network is no wider than the chunk's keys.  The only
// chunk is the order itself; the sorted chunks go to skey and sidx otherwise.
template <typename T>
__device__ __forceinline__ void sort_body(int c, int nchunks, const T* __restrict__ partial, int tiles,
                                          double* __restrict__ f, double* __restrict__ skey, int* __restrict__ sidx,
                                          const BestArgs<T>& a) {
  __shared__ double ks[kSortChunk];
  __shared__ int is[kSortChunk];
  const int t = threadIdx.x, i = c * kSortChunk + t, lam = a.lam;
  double k = __builtin_inf();
  int ix = 0x7fffffff;
  if (i < lam) {
    double v;
    if (tiles > 0) {
      v = sum_strided(partial + i, lam, tiles);
      v += 0.0;
      f[i] = v;
    } else {
      v = f[i];
    }
    k = rank_key(v);
    ix = i;
  }
  const int keys = min(kSortChunk, lam - c * kSortChunk);
  for (int size = 2; size < 2 * keys; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      double pk;
      int pi;
      if (stride >= 64) {
        __syncthreads();
        ks[t] = k;
        is[t] = ix;
        __syncthreads();
        pk = ks[t ^ stride];
        pi = is[t ^ stride];
      } else {
        pk = __shfl_xor(k, stride);
        pi = __shfl_xor(ix, stride);
      }
      const bool up = (t & size) == 0, low = (t & stride) == 0;
      const bool less = low ? key_less(pk, pi, k, ix) : key_less(k, ix, pk, pi);
      if (less == up) {
        k = pk;
        ix = pi;
      }
    }
  if (nchunks == 1) {
    place(a, ix < lam ? t : -1, ix, k);
  } else {
    skey[i] = k;
    sidx[i] = ix;
  }
}

// workgroup (c, g): the keys of chunk c counted against chunks
// [g kMergeGroup, (g + 1) kMergeGroup) other than c; the ranks, if these are
// all chunks
template <typename T>
__device__ __forceinline__ void merge_body(int c, int g, int nchunks, const double* __restrict__ skey,
                                           const int* __restrict__ sidx, int32_t* __restrict__ part,
                                           const BestArgs<T>& a) {
  __shared__ double ok[kSortChunk];
  __shared__ int oi[kSortChunk];
  const int t = threadIdx.x, lam = a.lam;
  const double kt = skey[c * kSortChunk + t];
  const int it = sidx[c * kSortChunk + t];
  int cnt = 0;
  const int c1 = min(nchunks, (g + 1) * kMergeGroup);
  for (int o = g * kMergeGroup; o < c1; ++o) {
    if (o == c) continue;  // uniform over the workgroup
    __syncthreads();
    ok[t] = skey[o * kSortChunk + t];
    oi[t] = sidx[o * kSortChunk + t];
    __syncthreads();
    int lo = 0, hi = kSortChunk;  // the first entry not below (kt, it)
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (key_less(ok[mid], oi[mid], kt, it))
        lo = mid + 1;
      else
        hi = mid;
    }
    cnt += lo;
  }
  if (nchunks <= kMergeGroup)
    place(a, it < lam ? t + cnt : -1, it, kt);
  else if (it < lam)
    part[static_cast<int64_t>(g) * lam + it] = cnt;
}

template <typename T>
__device__ __forceinline__ void scatter_body(int c, int ngroups, const double* __restrict__ skey,
                                             const int* __restrict__ sidx, const int32_t* __restrict__ part,
                                             const BestArgs<T>& a) {
  const int t = threadIdx.x;
  const int i = sidx[c * kSortChunk + t];
  int rank = -1;
  if (i < a.lam) {
    rank = t;
    for (int g = 0; g < ngroups; ++g) rank += part[static_cast<int64_t>(g) * a.lam + i];
  }
  place(a, rank, i, skey[c * kSortChunk + t]);
}

template <typename T>
__global__ void __launch_bounds__(256) k_sort(const T* __restrict__ partial, int tiles, double* __restrict__ f,
                                              double* __restrict__ skey, int* __restrict__ sidx, BestArgs<T> a) {
  sort_body<T>(blockIdx.x, gridDim.x, partial, tiles, f, skey, sidx, a);
}

template <typename T>
__global__ void __launch_bounds__(256) k_merge(const double* __restrict__ skey, const int* __restrict__ sidx,
                                               int32_t* __restrict__ part, BestArgs<T> a) {
  merge_body<T>(blockIdx.x, blockIdx.y, gridDim.x, skey, sidx, part, a);
}

template <typename T>
__global__ void __launch_bounds__(256) k_scatter(int ngroups, const double* __restrict__ skey,
                                                 const int* __restrict__ sidx, const int32_t* __restrict__ part,
                                                 BestArgs<T> a) {
  scatter_body<T>(blockIdx.x, ngroups, skey, sidx, part, a);
}

// y_w = sum_{r<mu} w_r y_{order[r]}, z_w likewise (float64 accumulation), and
// Yhat[:, r] = sqrt(w_r) y_{order[r]} for the rank-mu SYRK.  Grid: 32 rows x
// chunks of 64 ranks; each chunk writes its own partial sums, in rank order.
// All of a tile's loads are under way at once, eight ranks to a thread, and the
// sums read LDS: with a thread for a row's 64 ranks the kernel waited on a chain
// of loads (n = 333, lambda = 1030 float64 15.7 us, now 5.4; n = 1000, lambda = 6144
// 22.4 to 21).
constexpr int kRecRows = 32, kRecRanks = 64;
template <typename T>
__device__ __forceinline__ void recombine_body(int bx, int by, int n, int mu, const T* __restrict__ Y,
                                               const T* __restrict__ Z, int ld, const int32_t* __restrict__ order,
                                               const double* __restrict__ w, const double* __restrict__ sqrtw,
                                               T* __restrict__ Ysel, int ldsel, double* __restrict__ part_yw,
                                               double* __restrict__ part_zw) {
  constexpr int PER = kRecRanks * kRecRows / 256;
  __shared__ T ys[kRecRanks][kRecRows], zs[kRecRanks][kRecRows];
  __shared__ double ws[kRecRanks];
  const int t = threadIdx.x, r = t & (kRecRows - 1), g = t / kRecRows;
  const int i = min(bx * kRecRows + r, n - 1), r0 = by * kRecRanks, cnt = min(kRecRanks, mu - r0);
  const bool mine = bx * kRecRows + r < n;
  T y[PER], z[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int64_t c = static_cast<int64_t>(order[r0 + min(g * PER + q, cnt - 1)]) * ld;
    y[q] = Y[c + i];
    z[q] = Z[c + i];
  }
  if (t < cnt) ws[t] = w[r0 + t];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int k = g * PER + q;
    ys[k][r] = y[q];
    zs[k][r] = z[q];
    if (mine && k < cnt)
      Ysel[static_cast<int64_t>(r0 + k) * ldsel + i] = static_cast<T>(sqrtw[r0 + k] * static_cast<double>(y[q]));
  }
  __syncthreads();
  // the first wave sums y, the second z
  if (mine && ((t & 63) < kRecRows) && t < 128) {
    const T(*v)[kRecRows] = t < 64 ? ys : zs;
    double a = 0.0;
#pragma unroll 16
    for (int k = 0; k < cnt; ++k) a += ws[k] * static_cast<double>(v[k][r]);
    (t < 64 ? part_yw : part_zw)[static_cast<int64_t>(by) * n + i] = a;
  }
}

template <typename T>
__global__ void __launch_bounds__(256) k_recombine(int n, int mu, const T* __restrict__ Y,
                                                   const T* __restrict__ Z, int ld,
                                                   const int32_t* __restrict__ order,
                                                   const double* __restrict__ w,
                                                   const double* __restrict__ sqrtw, T* __restrict__ Ysel,
                                                   int ldsel, double* __restrict__ part_yw,
                                                   double* __restrict__ part_zw) {
  recombine_body<T>(blockIdx.x, blockIdx.y, n, mu, Y, Z, ld, order, w, sqrtw, Ysel, ldsel, part_yw, part_zw);
}

// y_w and z_w from their chunks' sums, in order
__device__ __forceinline__ void reduce_yz_body(int bx, int n, int nchunks, const double* __restrict__ py,
                                               const double* __restrict__ pz, double* __restrict__ yw,
                                               double* __restrict__ zw) {
  const int i = bx * blockDim.x + threadIdx.x;
  if (i >= n) return;
  yw[i] = sum_strided(py + i, n, nchunks);
  zw[i] = sum_strided(pz + i, n, nchunks);
}

__global__ void k_reduce_yz(int n, int nchunks, const double* __restrict__ py, const double* __restrict__ pz,
                            double* __restrict__ yw, double* __restrict__ zw) {
  reduce_yz_body(blockIdx.x, n, nchunks, py, pz, yw, zw);
}

// part[c][i] = sum over the columns j of chunk c of M(i, j) (x_j - x0_j) (x0 null:
// x_j)
__global__ void __launch_bounds__(256) k_matvec(int n, const double* __restrict__ M, int ld,
                                                const double* __restrict__ x, const double* __restrict__ x0,
                                                double* __restrict__ part) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int j0 = blockIdx.y * 64, j1 = min(n, j0 + 64);
  double s = 0.0;
#pragma unroll 16
  for (int j = j0; j < j1; ++j) s += M[static_cast<int64_t>(j) * ld + i] * (x[j] - (x0 ? x0[j] : 0.0));
  part[static_cast<int64_t>(blockIdx.y) * n + i] = s;
}

// bz = B z_w; with nchunks > 0 y_w and z_w are summed up on the way, z_w by each
// workgroup for itself (worth a launch of 4 us while that is at most kSumHere
// loads a workgroup: n = 512 with 16 chunks; beyond it k_reduce_yz sums once)
constexpr int kSumHere = 8192;
__device__ __forceinline__ void bz_body(int b, int n, const double* __restrict__ B, int ldb, int nchunks,
                                        const double* __restrict__ py, const double* __restrict__ pz,
                                        const double* __restrict__ zw, double* __restrict__ yw,
                                        double* __restrict__ bz) {
  const int t = threadIdx.x;
  const double v = matvec_rows(b * kMvRows, n, B, ldb,
                               [&](int j) { return nchunks > 0 ? sum_strided(pz + j, n, nchunks) : zw[j]; });
  const int i = b * kMvRows + (t & 31);
  if (i >= n) return;
  if (t < kMvRows)
    bz[i] = v;
  else if (nchunks > 0 && t >= 64 && t < 64 + kMvRows)
    yw[i] = sum_strided(py + i, n, nchunks);
}

__global__ void __launch_bounds__(256) k_bz(int n, const double* __restrict__ B, int ldb, int nchunks,
                                            const double* __restrict__ py, const double* __restrict__ pz,
                                            const double* __restrict__ zw, double* __restrict__ yw,
                                            double* __restrict__ bz) {
  bz_body(blockIdx.x, n, B, ldb, nchunks, py, pz, zw, yw, bz);
}

// sum over NT threads as a tree of halves (thread t adds t + s, s = NT / 2 .. 1),
// the last six levels by shuffles; the result in every thread
template <int NT>
__device__ double block_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
#pragma unroll
  for (int s = NT / 2; s >= 64; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = v = v + red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x < 64) {
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v += __shfl_down(v, s);
    if (threadIdx.x == 0) red[0] = v;
  }
  __syncthreads();
  return red[0];
}

// p_sigma, h_sigma, p_c, m, sigma and the covariance coefficient a, from B z_w as
// bz_chunks partial sums.  (NT threads;
// the sum does not depend on how many of 1024 or fewer hold no element.)
template <int NT>
__device__ __forceinline__ void vec_update_body(const KParams& kp, const double* __restrict__ bz, int bz_chunks,
                                                const double* __restrict__ yw, double* __restrict__ m,
                                                double* __restrict__ ps, double* __restrict__ pc,
                                                DevScalars* __restrict__ sc) {
  __shared__ double red[NT];
  const int n = kp.n;
  const double sigma = sc->sigma;
  const int64_t g = sc->gen;
  const double fps = sqrt(kp.cs * (2.0 - kp.cs) * kp.mueff);
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += NT) {
    const double v = (1.0 - kp.cs) * ps[i] + fps * sum_strided(bz + i, n, bz_chunks);
    ps[i] = v;
    acc += v * v;
  }
  const double denom = sqrt(1.0 - pow(1.0 - kp.cs, 2.0 * static_cast<double>(g + 1)));
  const double nps = sqrt(block_sum<NT>(acc, red));
  const double hsig = (nps / denom < (1.4 + 2.0 / (n + 1.0)) * kp.chin) ? 1.0 : 0.0;
  const double fpc = hsig * sqrt(kp.cc * (2.0 - kp.cc) * kp.mueff);
  for (int i = threadIdx.x; i < n; i += NT) {
    pc[i] = (1.0 - kp.cc) * pc[i] + fpc * yw[i];
    m[i] = m[i] + sigma * yw[i];
  }
  if (threadIdx.x == 0) {
    sc->ps_norm = nps;
    sc->hsig = hsig;
    sc->c_coef = 1.0 - kp.c1 - kp.cmu * kp.sumw + (1.0 - hsig) * kp.c1 * kp.cc * (2.0 - kp.cc);
    sc->sigma = sigma * exp((kp.cs / kp.ds) * (nps / kp.chin - 1.0));
    sc->gen = g + 1;
    sc->evals += kp.lam;
  }
}

template <int NT>
__global__ void __launch_bounds__(NT) k_vec_update(KParams kp, const double* __restrict__ bz, int bz_chunks,
                                                   const double* __restrict__ yw, double* __restrict__ m,
                                                   double* __restrict__ ps, double* __restrict__ pc,
                                                   DevScalars* __restrict__ sc) {
  vec_update_body<NT>(kp, bz, bz_chunks, yw, m, ps, pc, sc);
}

// largest of four values each over 256 threads, and the or of their flags, in
// every thread
__device__ __forceinline__ void block_max4_or(double (&v)[4], int& flags) {
  __shared__ double red[4][4];
  __shared__ int fl[4];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = fmax(v[q], __shfl_xor(v[q], m));
    flags |= __shfl_xor(flags, m);
  }
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) red[threadIdx.x >> 6][q] = v[q];
    fl[threadIdx.x >> 6] = flags;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = fmax(v[q], red[w][q]);
    flags |= fl[w];
  }
  __syncthreads();
}

// Stopping tests evaluated after the update (reading of Sec. 2.2; thresholds
// of the original IPOP-CMA-ES paper).
__device__ __forceinline__ void stop_body(const KParams& kp, const StopParams& sp, const double* __restrict__ m,
                                          const double* __restrict__ C, int ldc, const double* __restrict__ B,
                                          int ldb, const double* __restrict__ D, const double* __restrict__ pc,
                                          const double* __restrict__ hist, DevScalars* __restrict__ sc,
                                          uint32_t* __restrict__ hstop) {
  const int n = kp.n;
  const double sigma = sc->sigma;
  const int64_t g = sc->gen;
  const int ax = static_cast<int>(g % n);
  enum { AXIS_MOVES = 1, COORD_STUCK = 2, NONFINITE = 4 };
  // largest sd, |p_c|, D and -D; of the f history largest f and -f
  double v[4] = {0.0, 0.0, 0.0, -__builtin_inf()};
  double hv[4] = {-__builtin_inf(), -__builtin_inf(), 0.0, 0.0};
  int flags = 0, none = 0;
  for (int i = threadIdx.x; i < n; i += 256) {
    const double cii = C[static_cast<int64_t>(i) * ldc + i];
    const double sd = sqrt(cii);
    v[0] = fmax(v[0], sd);
    v[1] = fmax(v[1], fabs(pc[i]));
    v[2] = fmax(v[2], D[i]);
    v[3] = fmax(v[3], -D[i]);
    const double mi = m[i];
    if (mi + 0.1 * sigma * D[ax] * B[static_cast<int64_t>(ax) * ldb + i] != mi) flags |= AXIS_MOVES;
    if (mi + 0.2 * sigma * sd == mi) flags |= COORD_STUCK;
    if (!isfinite(mi) || !isfinite(cii) || !isfinite(pc[i]) || !isfinite(D[i])) flags |= NONFINITE;
  }
  // (a full ring: the last hist_len generations are all of it)
  const bool full = sc->hist_count >= sp.hist_len;
  if (full)
    for (int q = threadIdx.x; q < sp.hist_len; q += 256) {
      hv[0] = fmax(hv[0], hist[q]);
      hv[1] = fmax(hv[1], -hist[q]);
    }
  block_max4_or(v, flags);
  block_max4_or(hv, none);
  if (threadIdx.x != 0) return;
  const double maxsd = v[0], maxpc = v[1], dmax = v[2], dmin = -v[3];
  const bool axis_moves = flags & AXIS_MOVES, coord_stuck = flags & COORD_STUCK, nonfinite = flags & NONFINITE;
  uint32_t bits = 0;
  if (full) {
    const double hmax = hv[0], hmin = -hv[1];
    if (hmax - hmin < sp.tol_hist_fun) bits |= 1u << 0;
    if (fmax(hmax, sc->f_gen_max) - fmin(hmin, sc->f_gen_min) < sp.tol_fun) bits |= 1u << 1;
  }
  if (sigma * maxsd < sp.tolx && sigma * maxpc < sp.tolx) bits |= 1u << 2;
  if (!axis_moves) bits |= 1u << 3;
  if (coord_stuck) bits |= 1u << 4;
  if (!sc->eig_ok || !(dmin > 0.0) || (dmax / dmin) * (dmax / dmin) > sp.max_condition) bits |= 1u << 5;
  if (sc->f_best < sp.f_target) bits |= 1u << 6;
  if (sp.max_gens > 0 && g >= sp.max_gens) bits |= 1u << 7;
  if (sp.max_evals > 0 && sc->evals >= sp.max_evals) bits |= 1u << 8;
  if (nonfinite || !isfinite(sigma)) bits |= 1u << 9;
  sc->stop = bits;
  // the host's copy of the bits and of f_best (pinned, mapped host memory:
  // the bits at hstop[0], f_best at hstop[2..3]): system-scope stores, read
  // by the host after the end of this kernel
  if (hstop) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(hstop + 2),
                       static_cast<unsigned long long>(__double_as_longlong(sc->f_best)), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(hstop, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

__global__ void __launch_bounds__(256) k_stop(KParams kp, StopParams sp, const double* __restrict__ m,
                                              const double* __restrict__ C, int ldc,
                                              const double* __restrict__ B, int ldb,
                                              const double* __restrict__ D, const double* __restrict__ pc,
                                              const double* __restrict__ hist, DevScalars* __restrict__ sc,
                                              uint32_t* __restrict__ hstop) {
  stop_body(kp, sp, m, C, ldc, B, ldb, D, pc, hist, sc, hstop);
}

__global__ void __launch_bounds__(256) k_shift(ShiftArgs a) { shift_body(blockIdx.x, a); }

// out[i] = sum over the chunks of 64 columns, in order
__global__ void __launch_bounds__(256) k_reduce_vec(int n, int nchunks, const double* __restrict__ part,
                                                    double* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = sum_strided(part + i, n, nchunks);
}

__global__ void k_set_identity(double* A, int n, int ld) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(n) * ld) return;
  const int col = static_cast<int>(idx / ld), row = static_cast<int>(idx % ld);
  A[idx] = (row == col) ? 1.0 : 0.0;
}

template <typename T>
__global__ void k_convert(const double* __restrict__ s, int lds, T* __restrict__ d, int ldd, int rows,
                          int cols) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(rows) * cols) return;
  const int c = static_cast<int>(idx / rows), r = static_cast<int>(idx % rows);
  d[static_cast<int64_t>(c) * ldd + r] = static_cast<T>(s[static_cast<int64_t>(c) * lds + r]);
}

// word i of the block belongs to the array whose run of words holds it
__device__ __forceinline__ uint32_t* xfer_word(const XferArgs& a, int i) {
  for (int k = 0; k < a.count; ++k) {
    if (i < a.words[k]) return static_cast<uint32_t*>(const_cast<void*>(a.dev[k])) + i;
    i -= a.words[k];
  }
  return nullptr;
}
__global__ void __launch_bounds__(256) k_xfer_out(XferArgs a, uint32_t* __restrict__ block) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t* p = xfer_word(a, i);
  if (p) block[i] = *p;
}
__global__ void __launch_bounds__(256) k_xfer_in(XferArgs a, const uint32_t* __restrict__ block,
                                                 DevScalars* __restrict__ sc, double sigma, int64_t gen) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t* p = xfer_word(a, i);
  if (p) *p = block[i];
  if (i == 0) {
    sc->sigma = sigma;
    sc->gen = gen;
    sc->stop = 0;
    sc->hist_count = 0;
    sc->eig_ok = 1;
  }
}

template <typename T>
__global__ void __launch_bounds__(256) k_scale_columns(int n, const double* __restrict__ B, int ldb,
                                                       const double* __restrict__ D, T* __restrict__ out, int ldo) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x, c = blockIdx.y;
  if (r < n) out[static_cast<int64_t>(c) * ldo + r] = static_cast<T>(B[static_cast<int64_t>(c) * ldb + r] * D[c]);
}

}  // namespace

namespace {
int xfer_blocks(const XferArgs& a) {
  int total = 1;
  for (int k = 0; k < a.count; ++k) total += a.words[k];
  return ceil_div(total, 256);
}
}  // namespace

hipError_t launch_xfer_out(hipStream_t st, const XferArgs& a, uint32_t* block) {
  k_xfer_out<<<xfer_blocks(a), 256, 0, st>>>(a, block);
  return hipGetLastError();
}

hipError_t launch_xfer_in(hipStream_t st, const XferArgs& a, const uint32_t* block, DevScalars* sc, double sigma,
                          int64_t gen) {
  k_xfer_in<<<xfer_blocks(a), 256, 0, st>>>(a, block, sc, sigma, gen);
  return hipGetLastError();
}

hipError_t launch_scale_columns(hipStream_t st, bool fp64, int n, const double* B, int ldb, const double* D, void* out,
                                int ldo) {
  const dim3 grid(ceil_div(n, 256), n);
  if (fp64)
    k_scale_columns<double><<<grid, 256, 0, st>>>(n, B, ldb, D, static_cast<double*>(out), ldo);
  else
    k_scale_columns<float><<<grid, 256, 0, st>>>(n, B, ldb, D, static_cast<float*>(out), ldo);
  return hipGetLastError();
}

// the rank work area (int32 elements): sorted keys (double, 2 words each),
// their indices, then the per-group counts
struct RankWork {
  double* skey;
  int* sidx;
  int32_t* part;
  int nchunks, ngroups;
};
__host__ __device__ inline RankWork rank_work_of(int32_t* work, int lam) {
  RankWork w;
  w.nchunks = (lam + kSortChunk - 1) / kSortChunk;
  w.ngroups = (w.nchunks + kMergeGroup - 1) / kMergeGroup;
  w.skey = reinterpret_cast<double*>(work);
  w.sidx = work + 2 * w.nchunks * kSortChunk;
  w.part = w.sidx + w.nchunks * kSortChunk;
  return w;
}

namespace {
template <typename T>
hipError_t rank(hipStream_t st, const RankArgs& r) {
  const BestArgs<T> a{r.n,   r.lam,  static_cast<const T*>(r.Y), r.ldy,  r.m, r.x_best,
                      r.hist, r.hist_len, r.sc, r.order};
  const RankWork w = rank_work_of(r.work, r.lam);
  k_sort<T><<<w.nchunks, 256, 0, st>>>(static_cast<const T*>(r.partial), r.tiles, r.f, w.skey, w.sidx, a);
  if (w.nchunks > 1) k_merge<T><<<dim3(w.nchunks, w.ngroups), 256, 0, st>>>(w.skey, w.sidx, w.part, a);
  if (w.ngroups > 1) k_scatter<T><<<w.nchunks, 256, 0, st>>>(w.ngroups, w.skey, w.sidx, w.part, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_rank(hipStream_t st, bool fp64, const RankArgs& r) {
  return fp64 ? rank<double>(st, r) : rank<float>(st, r);
}

size_t rank_work_elems(int lam) {
  const size_t nchunks = ceil_div(lam, kSortChunk), ngroups = ceil_div(static_cast<int>(nchunks), kMergeGroup);
  return 3 * nchunks * kSortChunk + ngroups * static_cast<size_t>(lam) + 2;
}

hipError_t launch_recombine(hipStream_t st, bool fp64, int n, int lam, int mu, const void* Y, const void* Z,
                            int ld, const int32_t* order, const double* w, const double* sqrtw, void* Ysel,
                            int ldsel, double* part_yw, double* part_zw, int* nchunks) {
  (void)lam;
  *nchunks = ceil_div(mu, kRecRanks);
  dim3 grid(ceil_div(n, kRecRows), *nchunks);
  if (fp64)
    k_recombine<double><<<grid, 256, 0, st>>>(n, mu, static_cast<const double*>(Y),
                                              static_cast<const double*>(Z), ld, order, w, sqrtw,
                                              static_cast<double*>(Ysel), ldsel, part_yw, part_zw);
  else
    k_recombine<float><<<grid, 256, 0, st>>>(n, mu, static_cast<const float*>(Y), static_cast<const float*>(Z),
                                             ld, order, w, sqrtw, static_cast<float*>(Ysel), ldsel, part_yw,
                                             part_zw);
  return hipGetLastError();
}

hipError_t launch_bz(hipStream_t st, int n, const double* B, int ldb, int nchunks, const double* part_yw,
                     const double* part_zw, double* yw, double* zw, double* bz, int* bz_chunks) {
  const bool here = n <= kMvOneMax && nchunks * n <= kSumHere;
  if (!here) k_reduce_yz<<<ceil_div(n, 256), 256, 0, st>>>(n, nchunks, part_yw, part_zw, yw, zw);
  if (n <= kMvOneMax) {
    k_bz<<<ceil_div(n, kMvRows), 256, 0, st>>>(n, B, ldb, here ? nchunks : 0, part_yw, part_zw, zw, yw, bz);
    *bz_chunks = 1;
  } else {
    *bz_chunks = ceil_div(n, 64);
    k_matvec<<<dim3(ceil_div(n, 256), *bz_chunks), 256, 0, st>>>(n, B, ldb, zw, nullptr, bz);
  }
  return hipGetLastError();
}

hipError_t launch_vec_update(hipStream_t st, const KParams& kp, const double* bz, int bz_chunks, const double* yw, double* m,
                             double* ps, double* pc, DevScalars* sc) {
  if (kp.n <= 64)
    k_vec_update<64><<<1, 64, 0, st>>>(kp, bz, bz_chunks, yw, m, ps, pc, sc);
  else if (kp.n <= 256)
    k_vec_update<256><<<1, 256, 0, st>>>(kp, bz, bz_chunks, yw, m, ps, pc, sc);
  else
    k_vec_update<1024><<<1, 1024, 0, st>>>(kp, bz, bz_chunks, yw, m, ps, pc, sc);
  return hipGetLastError();
}

hipError_t launch_stop(hipStream_t st, const KParams& kp, const StopParams& sp, const double* m,
                       const double* C, int ldc, const double* B, int ldb, const double* D,
                       const double* pc, const double* hist, DevScalars* sc, uint32_t* hstop) {
  k_stop<<<1, 256, 0, st>>>(kp, sp, m, C, ldc, B, ldb, D, pc, hist, sc, hstop);
  return hipGetLastError();
}

hipError_t launch_shift(hipStream_t st, const ShiftArgs& a) {
  if (!a.R || a.n <= kMvOneMax) {
    k_shift<<<shift_blocks(a.n, a.R != nullptr), 256, 0, st>>>(a);
    return hipGetLastError();
  }
  const int nch = ceil_div(a.n, 64), rows = ceil_div(a.n, 256);
  k_matvec<<<dim3(rows, nch), 256, 0, st>>>(a.n, a.R, a.ldr, a.m, a.xstar, a.part);
  k_reduce_vec<<<rows, 256, 0, st>>>(a.n, nch, a.part, a.d);
  return hipGetLastError();
}

// B <- (3 B - B (B^T B)) / 2 from T = B (B^T B): one Newton-Schulz step
// towards the orthogonal polar factor of B (rows < n only)
__device__ __forceinline__ void polar_body(int bx, int n, double* __restrict__ B, int ldb, const double* __restrict__ T,
                                           int ldt) {
  const int64_t idx = static_cast<int64_t>(bx) * blockDim.x + threadIdx.x;
  const int64_t total = static_cast<int64_t>(n) * n;
  if (idx >= total) return;
  const int col = static_cast<int>(idx / n), row = static_cast<int>(idx % n);
  double& b = B[static_cast<int64_t>(col) * ldb + row];
  b = 1.5 * b - 0.5 * T[static_cast<int64_t>(col) * ldt + row];
}

__global__ void k_polar_step(int n, double* __restrict__ B, int ldb, const double* __restrict__ T, int ldt) {
  polar_body(blockIdx.x, n, B, ldb, T, ldt);
}

// ---- variants

// active covariance update: one workgroup per rank r; ranks beyond mu get the
// negative weight scaled by n / ||C^{-1/2} y||^2 = n / ||z||^2 (y = B D z with
// orthonormal B), the norm summed in float64 in a fixed order
template <typename T>
__global__ void __launch_bounds__(256) k_active_cols(int n, int mu, const T* __restrict__ Y, const T* __restrict__ Z,
                                                     int ld, const int32_t* __restrict__ order,
                                                     const double* __restrict__ w_all, T* __restrict__ Ysel,
                                                     T* __restrict__ Ysig, int ldsel) {
  __shared__ double red[256];
  const int r = blockIdx.x;
  T* ys = Ysel + static_cast<int64_t>(r) * ldsel;
  T* yg = Ysig + static_cast<int64_t>(r) * ldsel;
  if (r < mu) {  // the positive columns, as the recombination wrote them
    for (int i = threadIdx.x; i < n; i += 256) yg[i] = ys[i];
    return;
  }
  const int64_t c = static_cast<int64_t>(order[r]) * ld;
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) {
    const double z = static_cast<double>(Z[c + i]);
    acc += z * z;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  const double wr = w_all[r], z2 = red[0];
  const double sc = (wr < 0.0 && z2 > 0.0) ? sqrt(-wr * n / z2) : 0.0;
  for (int i = threadIdx.x; i < n; i += 256) {
    const double v = sc * static_cast<double>(Y[c + i]);
    ys[i] = static_cast<T>(v);
    yg[i] = static_cast<T>(-v);
  }
}

// separable sampling: y = D z
template <typename T>
__global__ void __launch_bounds__(256) k_sep_sample(int n, int lam, const double* __restrict__ D,
                                                    const T* __restrict__ Z, int ldz, T* __restrict__ Y, int ldy) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(n) * lam) return;
  const int k = static_cast<int>(idx / n), i = static_cast<int>(idx % n);
  Y[static_cast<int64_t>(k) * ldy + i] = static_cast<T>(D[i] * static_cast<double>(Z[static_cast<int64_t>(k) * ldz + i]));
}

// separable covariance update: the diagonal of the rank-one plus rank-mu update
template <typename T>
__global__ void __launch_bounds__(256) k_sep_cov(int n, int mu, const T* __restrict__ Y, int ldy,
                                                 const int32_t* __restrict__ order, const double* __restrict__ w,
                                                 const double* __restrict__ pc, double c1, double cmu,
                                                 double* __restrict__ C, int ldc, const DevScalars* __restrict__ sc) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double acc = 0.0;
  for (int r = 0; r < mu; ++r) {
    const double y = static_cast<double>(Y[static_cast<int64_t>(order[r]) * ldy + i]);
    acc += w[r] * y * y;
  }
  double& cii = C[static_cast<int64_t>(i) * ldc + i];
  cii = sc->c_coef * cii + c1 * pc[i] * pc[i] + cmu * acc;
}

// separable "decomposition": D = sqrt(diag C), B D = diag(D); eig_ok when the
// diagonal is positive (a one-workgroup kernel)
template <typename T>
__global__ void __launch_bounds__(256) k_sep_eigen(int n, const double* __restrict__ C, int ldc,
                                                   double* __restrict__ D, T* __restrict__ BD, int ldbd,
                                                   DevScalars* __restrict__ sc) {
  __shared__ int bad;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += 256) {
    const double cii = C[static_cast<int64_t>(i) * ldc + i];
    if (!(cii > 0.0)) atomicOr(&bad, 1);
    const double d = sqrt(fmax(cii, 0.0));
    D[i] = d;
    BD[static_cast<int64_t>(i) * ldbd + i] = static_cast<T>(d);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    sc->eig_ok = bad ? 0 : 1;
    sc->jac_sweeps = 0;
    sc->jac_corr = 0;
  }
}

__device__ __forceinline__ BestArgs<float> best_args(const GFront& e) {
  return BestArgs<float>{e.n, e.lam, e.Y, e.ldn, e.m, e.x_best, e.hist, e.hist_len, e.sc, e.order};
}

// ---- the update steps of a grouped front (one launch per step for all
// descents; workgroup w of descent i is local block w - off[i], split into
// (bx, by) by the descent's own grid width)
__global__ void __launch_bounds__(256) kg_update256(int kind, const GFront* __restrict__ g, const int* __restrict__ off,
                                                    int count, GroupDueMask mask) {
  const int i = group_find(off, count, blockIdx.x);
  const GFront& e = g[i];
  const int w = blockIdx.x - off[i];
  switch (kind) {
    case GF_SHIFT: shift_body(w, ShiftArgs{e.n, e.Rd, e.ldn, e.m, e.xstar, e.d, nullptr}); break;
    case GF_SORT: {
      const RankWork rw = rank_work_of(e.rank_work, e.lam);
      sort_body<float>(w, rw.nchunks, e.partial, e.fit_tiles, e.f, rw.skey, rw.sidx, best_args(e));
      break;
    }
    case GF_MERGE: {
      const RankWork rw = rank_work_of(e.rank_work, e.lam);
      merge_body<float>(w % rw.nchunks, w / rw.nchunks, rw.nchunks, rw.skey, rw.sidx, rw.part, best_args(e));
      break;
    }
    case GF_SCATTER: {
      const RankWork rw = rank_work_of(e.rank_work, e.lam);
      scatter_body<float>(w, rw.ngroups, rw.skey, rw.sidx, rw.part, best_args(e));
      break;
    }
    case GF_RECOMB: {
      const int gx = (e.n + kRecRows - 1) / kRecRows;
      recombine_body<float>(w % gx, w / gx, e.n, e.mu, e.Y, e.Z, e.ldn, e.order, e.w, e.sqrtw, e.Ysel, e.ldn,
                            e.part_yw, e.part_zw);
      break;
    }
    case GF_REDYZ:
      reduce_yz_body(w, e.n, (e.mu + kRecRanks - 1) / kRecRanks, e.part_yw, e.part_zw, e.yw, e.zw);
      break;
    case GF_BZ: {
      const int nch = (e.mu + kRecRanks - 1) / kRecRanks;
      bz_body(w, e.n, e.B, e.ldn, static_cast<int64_t>(nch) * e.n <= kSumHere ? nch : 0, e.part_yw, e.part_zw, e.zw,
              e.yw, e.bz);
      break;
    }
    case GF_POLAR:
      if (due_mask_bit(mask, i)) polar_body(w, e.n, e.B, e.ldn, e.T, e.ldn);
      break;
    case GF_STOP: stop_body(e.kp, e.sp, e.m, e.C, e.ldn, e.B, e.ldn, e.D, e.pc, e.hist, e.sc, e.hstop); break;
    default: break;
  }
}

__global__ void __launch_bounds__(1024) kg_vec_update(const GFront* __restrict__ g, const int* __restrict__ off,
                                                      int count) {
  const int i = group_find(off, count, blockIdx.x);
  const GFront& e = g[i];
  vec_update_body<1024>(e.kp, e.bz, 1, e.yw, e.m, e.ps, e.pc, e.sc);
}

hipError_t launch_group_update(hipStream_t st, int kind, const GFront* g, const int* off, int count, int wgs,
                               const GroupDueMask* mask) {
  if (wgs == 0) return hipSuccess;
  if (kind == GF_VECUPD) {
    kg_vec_update<<<wgs, 1024, 0, st>>>(g, off, count);
  } else {
    GroupDueMask m{};
    if (mask) m = *mask;
    kg_update256<<<wgs, 256, 0, st>>>(kind, g, off, count, m);
  }
  return hipGetLastError();
}

int rank_chunks(int lam) { return ceil_div(lam, kSortChunk); }
int rank_merge_wgs(int lam) {
  const int nch = ceil_div(lam, kSortChunk);
  return nch > 1 ? nch * ceil_div(nch, kMergeGroup) : 0;
}
int rank_scatter_wgs(int lam) { return rank_chunks(lam) > kMergeGroup ? rank_chunks(lam) : 0; }
int recombine_wgs(int n, int mu) { return ceil_div(n, kRecRows) * ceil_div(mu, kRecRanks); }
int reduce_yz_wgs(int n, int mu) {
  return static_cast<int64_t>(ceil_div(mu, kRecRanks)) * n <= kSumHere ? 0 : ceil_div(n, 256);
}

hipError_t launch_active_cols(hipStream_t st, bool fp64, int n, int lam, int mu, const void* Y, const void* Z, int ld,
                              const int32_t* order, const double* w_all, void* Ysel, void* Ysig, int ldsel) {
  if (fp64)
    k_active_cols<double><<<lam, 256, 0, st>>>(n, mu, static_cast<const double*>(Y), static_cast<const double*>(Z), ld,
                                               order, w_all, static_cast<double*>(Ysel), static_cast<double*>(Ysig),
                                               ldsel);
  else
    k_active_cols<float><<<lam, 256, 0, st>>>(n, mu, static_cast<const float*>(Y), static_cast<const float*>(Z), ld,
                                              order, w_all, static_cast<float*>(Ysel), static_cast<float*>(Ysig),
                                              ldsel);
  return hipGetLastError();
}

hipError_t launch_sep_sample(hipStream_t st, bool fp64, int n, int lam, const double* D, const void* Z, int ldz,
                             void* Y, int ldy) {
  const int64_t total = static_cast<int64_t>(n) * lam;
  const int blocks = static_cast<int>((total + 255) / 256);
  if (fp64)
    k_sep_sample<double><<<blocks, 256, 0, st>>>(n, lam, D, static_cast<const double*>(Z), ldz,
                                                 static_cast<double*>(Y), ldy);
  else
    k_sep_sample<float><<<blocks, 256, 0, st>>>(n, lam, D, static_cast<const float*>(Z), ldz, static_cast<float*>(Y),
                                                ldy);
  return hipGetLastError();
}

hipError_t launch_sep_cov(hipStream_t st, bool fp64, int n, int mu, const void* Y, int ldy, const int32_t* order,
                          const double* w, const double* pc, double c1, double cmu, double* C, int ldc,
                          const DevScalars* sc) {
  if (fp64)
    k_sep_cov<double><<<ceil_div(n, 256), 256, 0, st>>>(n, mu, static_cast<const double*>(Y), ldy, order, w, pc, c1,
                                                        cmu, C, ldc, sc);
  else
    k_sep_cov<float><<<ceil_div(n, 256), 256, 0, st>>>(n, mu, static_cast<const float*>(Y), ldy, order, w, pc, c1,
                                                       cmu, C, ldc, sc);
  return hipGetLastError();
}

hipError_t launch_sep_eigen(hipStream_t st, bool fp64, int n, const double* C, int ldc, double* D, void* BD, int ldbd,
                            DevScalars* sc) {
  if (fp64)
    k_sep_eigen<double><<<1, 256, 0, st>>>(n, C, ldc, D, static_cast<double*>(BD), ldbd, sc);
  else
    k_sep_eigen<float><<<1, 256, 0, st>>>(n, C, ldc, D, static_cast<float*>(BD), ldbd, sc);
  return hipGetLastError();
}

hipError_t launch_polar_step(hipStream_t st, int n, double* B, int ldb, const double* T, int ldt) {
  const int64_t total = static_cast<int64_t>(n) * n;
  k_polar_step<<<static_cast<int>((total + 255) / 256), 256, 0, st>>>(n, B, ldb, T, ldt);
  return hipGetLastError();
}

hipError_t launch_set_identity(hipStream_t st, double* A, int n, int ld) {
  const int64_t total = static_cast<int64_t>(n) * ld;
  k_set_identity<<<static_cast<int>((total + 255) / 256), 256, 0, st>>>(A, n, ld);
  return hipGetLastError();
}

hipError_t launch_to_precision(hipStream_t st, bool fp64, const double* src, int ld_src, void* dst, int ld_dst,
                               int rows, int cols) {
  const int64_t total = static_cast<int64_t>(rows) * cols;
  const int blocks = static_cast<int>((total + 255) / 256);
  if (blocks == 0) return hipSuccess;
  if (fp64)
    k_convert<double><<<blocks, 256, 0, st>>>(src, ld_src, static_cast<double*>(dst), ld_dst, rows, cols);
  else
    k_convert<float><<<blocks, 256, 0, st>>>(src, ld_src, static_cast<float*>(dst), ld_dst, rows, cols);
  return hipGetLastError();
}

}  // namespace cmx

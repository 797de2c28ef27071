// Refinement of the eigendecomposition C = B D^2 B^T (Sec. 2.1) by products.
//
// A warm-started solve begins with eigenvectors V of the previous covariance,
// so S = V^T C V is nearly diagonal.  One step rotates every index pair at
// once: with R = I - V^T V (V's distance from orthogonality) and d_i =
// S_ii / (V^T V)_ii, the angle of the pair (i, j) is that of its own 2 x 2
// problem in the basis made orthogonal to first order,
//   s_ij = S_ij + R_ij (d_i + d_j) / 2,   theta_ij = atan(2 s_ij / (d_j - d_i)) / 2,
// clipped at kClip, and
//   V <- V X,   X = I + Theta + R / 2 + Theta^2 / 2 + Theta^3 / 6
// (Theta antisymmetric).  To first order this is the refinement of Ogita and
// Aishima ("Iterative refinement for symmetric eigenvalue decomposition",
// Japan J. Indust. Appl. Math. 35, 2018): it converges quadratically in both
// the off-diagonal part and the orthogonality, and since every step starts
// again from C, neither the rounding of the steps before it nor a drift of B
// from one solve to the next stays in the result.  The second and third order
// terms, Jacobi's angle in place of the quotient, the clip and a bound on the
// length of Theta's rows let it start from angles that are not small
// (||Theta||_F^2 up to kThLimit n).
//
// A step takes five float64 products (two of them, and the two powers of
// Theta, of lower tiles only); a block-Jacobi sweep reduces off(A) about as
// far in N/16 - 1 dependent rounds.  At n = 1000 a step takes a quarter of a
// sweep's time.
//
// Whether a step is applied, and whether it was the last, is decided on the
// device by every workgroup alike from the same partial sums, so several
// steps can be queued behind one another; the host reads the outcome once.
//
// Measured at n = 1000 (us): C V 40.1, S and G 48.0, Theta 10.4 (its long rows
// 7.2 more), Theta^2 (with X where Theta^3 does not count) 29.7, Theta^3 and X 32 where it
// does, V X 39.0, so about 190 a step against 730 a sweep of 63 rounds; 50 TFLOP/s in the
// whole products (a library's 1000^3 product takes 37.1), bound by the float64
// matrix cores and, at one or two tiles per CU, by the start of each tile's loads
// and the sum over the waves.  At n = 200: 4.1, 4.3, 5.7, 5.9, 5.2 and 4.1, bound by
// latency; a sweep of 13 rounds takes 150.
#include "dtile.h"
#include "internal.h"
#include "refine.h"

namespace cmx {

namespace {

using TinyTile = Tile<1, 4>;
using SmallTile = Tile<2, 8>;
using LargeTile = Tile<3, 4>;

__device__ __forceinline__ void lower_tile(int t, int& tm, int& tn) {
  tm = static_cast<int>((sqrtf(8.0f * t + 1.0f) - 1.0f) * 0.5f);
  while ((tm + 1) * (tm + 2) / 2 <= t) ++tm;
  while (tm * (tm + 1) / 2 > t) --tm;
  tn = t - tm * (tm + 1) / 2;
}

// out = op(A) B over all tiles; the first workgroup clears `count` words of `clear`
template <class TL, bool TA, bool CLAMP>
__global__ void __launch_bounds__(TL::THREADS, 2) k_ref_full(const double* __restrict__ A, int lda,
                                                             const double* __restrict__ B, int N, int n,
                                                             double* __restrict__ out, int rmax, int kmax,
                                                             const int* __restrict__ word, int mask, int want,
                                                             unsigned* __restrict__ clear, int count) {
  __shared__ double lds[TL::LDS];
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < count; i += TL::THREADS) clear[i] = 0;
  const bool go = word == nullptr || (*word & mask) == want;
  const int side = (n + TL::T - 1) / TL::T;
  const int t = xcd_order(blockIdx.x, gridDim.x);
  const int m0 = (t % side) * TL::T, n0 = (t / side) * TL::T;
  if (!TL::template product<TA, CLAMP>(lds, A, lda, B, N, (n + 15) / 16, m0, n0, rmax, N, kmax, go)) return;
#pragma unroll
  for (int e = 0; e < TL::PER; ++e) {
    const int idx = threadIdx.x + TL::THREADS * e, r = idx % TL::T, c = idx / TL::T;
    if (m0 + r < N && n0 + c < N) out[static_cast<int64_t>(n0 + c) * N + m0 + r] = TL::get(lds, r, c);
  }
}

// lower tiles of S = V^T T (MIRROR: both triangles) and, with twice the
// workgroups, of G = V^T V
template <class TL, bool MIRROR>
__global__ void __launch_bounds__(TL::THREADS, 2) k_ref_sg(const double* __restrict__ V, const double* __restrict__ Tm,
                                                           int N, int n, int ntl, double* __restrict__ S,
                                                           double* __restrict__ G, const int* __restrict__ word) {
  __shared__ double lds[TL::LDS];
  const bool go = word == nullptr || *word == 0;
  int t = xcd_order(blockIdx.x, gridDim.x);
  const bool second = t >= ntl;
  if (second) t -= ntl;
  int tm, tn;
  lower_tile(t, tm, tn);
  const int m0 = tm * TL::T, n0 = tn * TL::T;
  if (!TL::template product<true, false>(lds, V, N, second ? V : Tm, N, (n + 15) / 16, m0, n0, N, N, N, go)) return;
  double* out = second ? G : S;
  double v[TL::PER];
#pragma unroll
  for (int e = 0; e < TL::PER; ++e) {
    const int idx = threadIdx.x + TL::THREADS * e, r = idx % TL::T, c = idx / TL::T;
    v[e] = MIRROR && tm == tn && r < c ? TL::get(lds, c, r) : TL::get(lds, r, c);
    if (MIRROR && (m0 + r >= n || n0 + c >= n)) v[e] = 0.0;  // the sweeps need zero padding
    if (m0 + r < N && n0 + c < N) out[static_cast<int64_t>(n0 + c) * N + m0 + r] = v[e];
  }
  if (MIRROR && tm != tn) TL::store_mirror(lds, v, out, N, m0, n0);
}

// sums of four values over the workgroup, in a fixed order, and the largest of a fifth
template <int NW, int M>
__device__ __forceinline__ void block_reduce(double (&v)[M], double (*red)[M]) {
  static_assert(M == 4 || M == 5, "four sums, then one maximum");
  auto join = [](int q, double a, double b) { return q < 4 ? a + b : fmax(a, b); };
#pragma unroll
  for (int q = 0; q < M; ++q)
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v[q] = join(q, v[q], __shfl_xor(v[q], m));
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int q = 0; q < M; ++q) red[threadIdx.x >> 6][q] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < M; ++q) {
    v[q] = red[0][q];
#pragma unroll
    for (int w = 1; w < NW; ++w) v[q] = join(q, v[q], red[w][q]);
  }
}

// Theta from the lower tiles of S and G (null: R = 0), 32 x 32 tiles; both
// triangles of Theta; per tile the squared norms of Theta, R, s and d (tiles
// of padding are zero); the first-order eigenvalues d, and per tile and row the sums over
// the tile's columns of theta_ji s_ij, which is what rotating by Theta adds to d_i, and
// of theta_ij^2.  Of the latter a tile's longest row is added to reach, for each 32 rows
// of Theta, which bounds their squared lengths: in units of 2^-16, since a sum of whole
// numbers does not depend on which tile comes first, rounded down, so that most tiles
// of the last steps add nothing, and k_ref_square counts one more for each tile.
// (0.4 us at n = 1000, nothing at n = 333; added up in k_ref_square from an array it took
// 1.4 us there, and the number of tiles times the largest part of any of them, which
// costs nothing, is so coarse a bound that nearly every step was damped in vain.)
constexpr int kCT = 32;
constexpr double kReachUnit = 1.0 / 65536.0;
__global__ void __launch_bounds__(256) k_ref_theta(const double* __restrict__ S, const double* __restrict__ G, int N,
                                                   int n, const double* __restrict__ scale, double* __restrict__ Th,
                                                   double* __restrict__ part, double* __restrict__ dsum,
                                                   double* __restrict__ rsum, unsigned* __restrict__ reach,
                                                   double* __restrict__ dv, const int* __restrict__ word) {
  __shared__ double tl[kCT][kCT + 1], ts[kCT][kCT + 1];
  __shared__ double dr[kCT], dc[kCT];
  __shared__ double red[4][4];
  if (word && *word != 0) return;
  int bi, bj;
  lower_tile(blockIdx.x, bi, bj);
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5;
  const int r0 = bi * kCT, c0 = bj * kCT;
  double sv[kCT / 8], gv[kCT / 8];
#pragma unroll
  for (int q = 0; q < kCT / 8; ++q) {
    const int64_t at = static_cast<int64_t>(c0 + ty + 8 * q) * N + r0 + tx;
    sv[q] = S[at];
    gv[q] = G ? G[at] : 0.0;
  }
  if (t < 2 * kCT) {
    const int i = (t < kCT ? r0 : c0) + (t & 31);
    const int64_t at = static_cast<int64_t>(i) * N + i;
    double v = 0.0;
    if (i < n) v = G ? S[at] / G[at] : S[at];
    (t < kCT ? dr : dc)[t & 31] = v;
    if (bi == bj && t < kCT && i < n) dv[i] = v;
  }
  __syncthreads();
  const double eps = 2.2e-16 * scale[0], unit = unit_scale(scale[0]), noise = unit * noise_level(n, eps);
  double th2 = 0.0, r2 = 0.0, off2 = 0.0, tot2 = 0.0;
#pragma unroll
  for (int q = 0; q < kCT / 8; ++q) {
    const int k = ty + 8 * q, r = r0 + tx, c = c0 + k;
    double th = 0.0, w = 0.0;
    if (r < n && c < n && r > c) {
      const double rij = -gv[q];
      const double a = sv[q] + 0.5 * rij * (dr[tx] + dc[k]);
      const double g = dr[tx] - dc[k];  // d_r - d_c: the rotation of the pair (c, r), c < r
      bool counts;
      const double h = refine_angle(unit * a, unit * g, noise, counts);
      th = -h;  // Theta(r, c) = -Theta(c, r)
      w = h * a;  // theta_cr s: added to d_r, taken from d_c
      if (counts) th2 = fma(2.0 * h, h, th2);
      r2 = fma(2.0 * rij, rij, r2) + (a - a);  // (a - a): NaN when a is not finite
      off2 = fma(2.0 * a, a, off2);
    } else if (r < n && r == c) {
      const double rii = G ? 1.0 - gv[q] : 0.0;
      r2 = fma(rii, rii, r2);
      tot2 = fma(dr[tx], dr[tx], tot2);
    }
    tl[tx][k] = th;
    ts[tx][k] = w;
  }
  double sums[4] = {th2, r2, off2, tot2};
  block_reduce<4>(sums, red);  // (its barrier also covers tl and ts)
  if (t < 4) part[4 * blockIdx.x + t] = t == 0 ? sums[0] : t == 1 ? sums[1] : t == 2 ? sums[2] : sums[3];
#pragma unroll
  for (int q = 0; q < kCT / 8; ++q) {
    const int k = ty + 8 * q;
    if (bi != bj) {
      Th[static_cast<int64_t>(c0 + k) * N + r0 + tx] = tl[tx][k];
      Th[static_cast<int64_t>(r0 + k) * N + c0 + tx] = -tl[k][tx];
    } else {
      Th[static_cast<int64_t>(c0 + k) * N + r0 + tx] = tx >= k ? tl[tx][k] : -tl[k][tx];
    }
  }
  // rows: + sum over the tile's columns; columns: - sum over its rows (the
  // first wave; the second the same for theta^2, which has no sign)
  if (t < 128) {
    const int i = t & 31;
    const bool sq = t >= 64, cols = (t & 32) != 0, twice = cols && bi == bj;
    double (*m)[kCT + 1] = sq ? tl : ts;
    double s = 0.0, o = 0.0;
#pragma unroll
    for (int k = 0; k < kCT; ++k) {
      const double v = cols ? m[k][i] : m[i][k];
      s += sq ? v * v : v;
    }
    if (bi == bj)
#pragma unroll
      for (int k = 0; k < kCT; ++k) o += sq ? m[k][i] * m[k][i] : m[k][i];
    const double sum = sq ? s + o : (cols ? -s : s - o);
    if (!twice) (sq ? rsum : dsum)[static_cast<int64_t>(cols ? bi : bj) * N + (cols ? c0 : r0) + i] = sum;
    if (sq) {
      double most = sum;
#pragma unroll
      for (int m = 16; m >= 1; m >>= 1) most = fmax(most, __shfl_xor(most, m));
      const unsigned units = static_cast<unsigned>(most / kReachUnit);
      if (i == 0 && !twice && units > 0)
        __hip_atomic_fetch_add(&reach[cols ? bj : bi], units, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ---- control words of a solve's refinement.  Step j reads state[j & 1]
// (0: run) and writes state[(j + 1) & 1] and bits[j & 1], so no workgroup
// reads a word that its own launch writes.
enum { RC_STATE = 0, RC_BITS = 2, RC_APPLIED = 4, RC_SMALL = 5, RC_TH2 = 6, RC_LONG = 8, RC_CUBES = 9 };
enum { RB_APPLY = 1, RB_CUBE = 2 };

// Theta damped where a row of it is long: theta_ij times min(1, c / |row i|,
// c / |row j|), c = longest_row, 32 x 32 tiles as in k_ref_theta.  A tile whose
// rows and columns are all short, which is every tile in the last steps, is left
// alone.  ||Theta||_F^2 is summed as by the NW waves of k_ref_square, so that both
// see the same bits and with them the same bound.
template <int NW>
__global__ void __launch_bounds__(256) k_ref_damp(double* __restrict__ Th, int N, int n,
                                                  const double* __restrict__ part, const double* __restrict__ rsum,
                                                  const int* __restrict__ ctl, int par, int first) {
  __shared__ double f[2 * kCT];
  __shared__ double red[NW];
  if (!first && ctl[RC_STATE + par] != 0) return;
  const float before = first ? 0.0f : __int_as_float(ctl[RC_TH2 + par]);
#pragma unroll
  for (int q = 0; q < NW / 4; ++q) {
    double sum = 0.0;
    for (int i = threadIdx.x + 256 * q; i < gridDim.x; i += 64 * NW) sum += part[4 * i];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m);
    if ((threadIdx.x & 63) == 0) red[(threadIdx.x >> 6) + 4 * q] = sum;
  }
  __syncthreads();
  double th2 = red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) th2 += red[w];
  const double row = longest_row(th2, before, n);
  int bi, bj;
  lower_tile(blockIdx.x, bi, bj);
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5;
  const int r0 = bi * kCT, c0 = bj * kCT;
  bool damp = false;
  if (t < 2 * kCT) {
    const int i = (t < kCT ? r0 : c0) + tx;
    double s = 0.0;
#pragma unroll 8
    for (int k = 0; k < N / kCT; ++k) s += rsum[static_cast<int64_t>(k) * N + i];
    damp = s > row * row;
    f[t] = damp ? row / sqrt(s) : 1.0;
  }
  if (!__syncthreads_or(damp)) return;
#pragma unroll
  for (int q = 0; q < kCT / 8; ++q) {
    const int k = ty + 8 * q;
    Th[static_cast<int64_t>(c0 + k) * N + r0 + tx] *= fmin(f[tx], f[kCT + k]);
    if (bi != bj) Th[static_cast<int64_t>(r0 + k) * N + c0 + tx] *= fmin(f[kCT + tx], f[k]);
  }
}

// X of one lower tile and of its mirror, in place of G (X and G share a
// buffer; useg false: R = 0; plain: Theta = 0): lower(r, c) and its transpose
// from the symmetric and antisymmetric parts.  sq(e, at): Theta^2 of element e, cube(r, c): Theta^3.
// The workgroups of the diagonal tiles also sum up the eigenvalues.
template <class TL, class Square, class Cube>
__device__ __forceinline__ void make_x(double* lds, const double* __restrict__ Th, int N, int n, int tm, int tn,
                                       bool useg, bool plain, double* __restrict__ X, const double* __restrict__ dsum,
                                       const double* __restrict__ dv, double* __restrict__ evals, Square sq,
                                       Cube cube) {
  const int m0 = tm * TL::T, n0 = tn * TL::T;
  double v[TL::PER];
#pragma unroll
  for (int e = 0; e < TL::PER; ++e) {
    const int idx = threadIdx.x + TL::THREADS * e, r = idx % TL::T, c = idx / TL::T;
    const int gr = m0 + r, gc = n0 + c;
    v[e] = 0.0;
    if (gr >= N || gc >= N) continue;
    const int64_t at = static_cast<int64_t>(gc) * N + gr;
    double lower = 0.0;
    if (gr < n && gc < n) {
      const double id = gr == gc ? 1.0 : 0.0;
      double sym = id + (plain ? 0.0 : 0.5 * sq(e, at));
      const double anti = plain ? 0.0 : Th[at] + cube(r, c) * (1.0 / 6.0);
      if (useg) sym += 0.5 * (id - X[at]);
      lower = sym + anti;
      v[e] = sym - anti;
    }
    X[at] = lower;
  }
  if (tm != tn) {
    TL::store_mirror(lds, v, X, N, m0, n0);
  } else if (threadIdx.x < TL::T) {
    const int i = m0 + threadIdx.x;
    if (i < n) {
      double s = dv[i];
      const int terms = plain ? 0 : N / kCT;
#pragma unroll 8
      for (int k = 0; k < terms; ++k) s += dsum[static_cast<int64_t>(k) * N + i];
      evals[i] = s;
    }
  }
}

// Decision on the step whose Theta is in place, by every workgroup alike, and
// the lower tiles of Theta^2.  While Theta^3 counts, both triangles of Theta^2
// are stored and k_ref_cube forms X; else X is formed here.  A step that may have
// long rows without k_ref_damp queued before it, or needs Theta^3 without k_ref_cube
// behind it, is held: the host queues it again from here on, with both (its row
// counts are cleared by then: the held step has entered it among those with long rows).
// So what a step computes does not depend on what was queued.
template <class TL>
__global__ void __launch_bounds__(TL::THREADS, 2) k_ref_square(const double* __restrict__ Th, int N, int n,
                                                               double* __restrict__ S2,
                                                               const double* __restrict__ part, int count,
                                                               const unsigned* __restrict__ reach, int first,
                                                               double thmax, int damped, int cube, int again,
                                                               int par,
                                                               int* __restrict__ ctl,
                                                               int* __restrict__ flags, double* __restrict__ X,
                                                               const double* __restrict__ dsum,
                                                               const double* __restrict__ dv,
                                                               double* __restrict__ evals) {
  __shared__ double lds[TL::LDS];
  __shared__ double red[TL::NW][5];
  const int before = first ? 0 : ctl[RC_STATE + par];
  const float th2_before = first ? 0.0f : __int_as_float(ctl[RC_TH2 + par]);
  const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
  double sums[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < count; i += TL::THREADS)
#pragma unroll
    for (int q = 0; q < 4; ++q) sums[q] += part[4 * i + q];
  for (int i = threadIdx.x; i < N / kCT; i += TL::THREADS) sums[4] = fmax(sums[4], kReachUnit * (reach[i] + N / kCT));
  int tm, tn;
  lower_tile(xcd_order(blockIdx.x, gridDim.x), tm, tn);
  const int m0 = tm * TL::T, n0 = tn * TL::T;
  // Theta^T Theta = -Theta^2
  if (!TL::template product<true, false>(lds, Th, N, Th, N, (n + 15) / 16, m0, n0, N, N, N, before == 0)) {
    if (lead) {  // nothing to do, nor for the steps behind this one
      ctl[RC_STATE + (par ^ 1)] = before;
      ctl[RC_BITS + par] = 0;
    }
    return;
  }
  block_reduce<TL::NW>(sums, red);
  const double th2 = sums[0], r2 = sums[1];
  const bool small_th = th2 <= kDone * kDone;
  // rounding is left as it is, whatever its angles are: the step only takes out R
  const bool plain = !small_th && !first && th2 > kStall * th2_before && sums[2] <= kOffDone * kOffDone * sums[3];
  const bool last = (small_th || plain) && r2 <= kDoneR * kDoneR;
  const bool apply = isfinite(th2) && isfinite(r2) && (!first || th2 <= thmax) && r2 <= kRLimit * n;
  const double row = longest_row(th2, th2_before, n);
  const bool rows = !plain && 1.001 * sums[4] > row * row;
  const bool third = !plain && th2 > kCubeFrom * kCubeFrom;
  const bool hold = apply && ((rows && !damped) || (third && !cube));
  const int bits = !apply || hold ? 0 : RB_APPLY | (third ? RB_CUBE : 0);
  if (lead) {
    const int state = !apply ? (first ? RS_REJECTED : RS_DIVERGED) : hold ? RS_HELD : last ? RS_DONE : RS_ACTIVE;
    const int applied = (first ? 0 : ctl[RC_APPLIED]) + (apply && !hold ? 1 : 0);
    const int small = (first ? 0 : ctl[RC_SMALL]) + (apply && !hold && th2 <= 4e-6 ? 1 : 0);
    ctl[RC_STATE + (par ^ 1)] = state;
    ctl[RC_BITS + par] = bits;
    ctl[RC_APPLIED] = applied;
    ctl[RC_TH2 + (par ^ 1)] = __float_as_int(static_cast<float>(th2));
    ctl[RC_SMALL] = small;
    __hip_atomic_store(&flags[RF_STATE], state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&flags[RF_APPLIED], applied, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const int longs = rows ? applied + (hold ? 1 : 0) : first && !again ? 0 : ctl[RC_LONG];
    ctl[RC_LONG] = longs;
    const int cubes = third ? applied : first ? 0 : ctl[RC_CUBES];
    ctl[RC_CUBES] = cubes;
    __hip_atomic_store(&flags[RF_CUBE], cubes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&flags[RF_LONG], longs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&flags[RF_SMALL], small, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if (!apply || hold) return;
  double v[TL::PER];
#pragma unroll
  for (int e = 0; e < TL::PER; ++e) {
    const int idx = threadIdx.x + TL::THREADS * e, r = idx % TL::T, c = idx / TL::T;
    v[e] = -TL::get(lds, r, c);
  }
  if (!(bits & RB_CUBE)) {
    make_x<TL>(lds, Th, N, n, tm, tn, first == 0, plain, X, dsum, dv, evals, [&](int e, int64_t) { return v[e]; },
               [](int, int) { return 0.0; });
    return;
  }
#pragma unroll
  for (int e = 0; e < TL::PER; ++e) {
    const int idx = threadIdx.x + TL::THREADS * e, r = idx % TL::T, c = idx / TL::T;
    if (m0 + r < N && n0 + c < N) S2[static_cast<int64_t>(n0 + c) * N + m0 + r] = v[e];
  }
  if (tm != tn) TL::store_mirror(lds, v, S2, N, m0, n0);
}

// X where Theta^3 counts: the lower tiles of Theta Theta^2, then make_x
template <class TL>
__global__ void __launch_bounds__(TL::THREADS, 2) k_ref_cube(const double* __restrict__ Th,
                                                             const double* __restrict__ S2, int N, int n, int useg,
                                                             double* __restrict__ X, const double* __restrict__ dsum,
                                                             const double* __restrict__ dv,
                                                             double* __restrict__ evals,
                                                             const int* __restrict__ word) {
  __shared__ double lds[TL::LDS];
  const bool go = (*word & RB_CUBE) != 0;
  int tm, tn;
  lower_tile(xcd_order(blockIdx.x, gridDim.x), tm, tn);
  // Theta^T Theta^2 = -Theta^3
  if (!TL::template product<true, false>(lds, Th, N, S2, N, (n + 15) / 16, tm * TL::T, tn * TL::T, N, N, N, go)) return;
  make_x<TL>(lds, Th, N, n, tm, tn, useg != 0, false, X, dsum, dv, evals, [&](int, int64_t at) { return S2[at]; },
             [&](int r, int c) { return -TL::get(lds, r, c); });
}

// the state that a held step reads, as it was before it
__global__ void k_ref_again(int* __restrict__ state) { *state = RS_ACTIVE; }

template <class TL>
hipError_t queue_start(hipStream_t st, const RefineStep& a, KTimer* kt) {
  const int side = ceil_div(a.n, TL::T), low = side * (side + 1) / 2;
  timed_launch(kt, KID_EIG_GEMM, k_ref_full<TL, true, true>, side * side, TL::THREADS, st, a.C, a.ldc, a.V, a.N, a.n,
               a.T, a.n, a.ldc, nullptr, 0, 0, nullptr, 0);
  timed_launch(kt, KID_EIG_GEMM, k_ref_sg<TL, true>, low, TL::THREADS, st, a.V, a.T, a.N, a.n, low, a.S, nullptr,
               nullptr);
  return hipGetLastError();
}

template <class TL>
hipError_t queue_step(hipStream_t st, const RefineStep& a, KTimer* kt) {
  const int N = a.N, side = ceil_div(a.n, TL::T), full = side * side, low = side * (side + 1) / 2;
  const int nt = N / kCT, tiles = nt * (nt + 1) / 2;
  int* state = a.ctl + RC_STATE + a.par;
  int* bits = a.ctl + RC_BITS + a.par;
  if (!a.first && !a.again) {
    timed_launch(kt, KID_EIG_GEMM, k_ref_full<TL, true, true>, full, TL::THREADS, st, a.C, a.ldc, a.V, N, a.n, a.T,
                 a.n, a.ldc, state, ~0, 0, nullptr, 0);  // C V (C is symmetric)
    timed_launch(kt, KID_EIG_GEMM, k_ref_sg<TL, false>, 2 * low, TL::THREADS, st, a.V, a.T, N, a.n, low, a.S, a.X,
                 state);
  }
  if (a.again && !a.first) k_ref_again<<<1, 1, 0, st>>>(state);
  if (!a.again)
    k_ref_theta<<<tiles, 256, 0, st>>>(a.S, a.first ? nullptr : a.X, N, a.n, a.scale, a.Th, a.part, a.dsum, a.rsum, a.reach,
                                     a.dv, a.first ? nullptr : state);
  if (a.damp)
    k_ref_damp<TL::NW><<<tiles, 256, 0, st>>>(a.Th, N, a.n, a.part, a.rsum, a.ctl, a.par, a.first ? 1 : 0);
  timed_launch(kt, KID_EIG_GEMM, k_ref_square<TL>, low, TL::THREADS, st, a.Th, N, a.n, a.T, a.part, tiles, a.reach,
               a.first ? 1 : 0, a.thmax, a.damp ? 1 : 0, a.cube ? 1 : 0, a.again ? 1 : 0, a.par, a.ctl, a.flags, a.X,
               a.dsum, a.dv, a.evals);
  if (a.cube)
    timed_launch(kt, KID_EIG_GEMM, k_ref_cube<TL>, low, TL::THREADS, st, a.Th, a.T, N, a.n, a.first ? 0 : 1, a.X, a.dsum,
                 a.dv, a.evals, bits);
  timed_launch(kt, KID_EIG_GEMM, k_ref_full<TL, false, false>, full, TL::THREADS, st, a.V, N, a.X, N, a.n, a.Vn, N, N,
               bits, static_cast<int>(RB_APPLY), static_cast<int>(RB_APPLY), a.reach, nt);
  return hipGetLastError();
}

}  // namespace

constexpr int kSmallFrom = 384, kLargeFrom = 640;

hipError_t launch_refine_start(hipStream_t st, const RefineStep& a, KTimer* kt) {
  if (a.n >= kLargeFrom) return queue_start<LargeTile>(st, a, kt);
  return a.n >= kSmallFrom ? queue_start<SmallTile>(st, a, kt) : queue_start<TinyTile>(st, a, kt);
}

hipError_t launch_refine_step(hipStream_t st, const RefineStep& a, KTimer* kt) {
  if (a.n >= kLargeFrom) return queue_step<LargeTile>(st, a, kt);
  return a.n >= kSmallFrom ? queue_step<SmallTile>(st, a, kt) : queue_step<TinyTile>(st, a, kt);
}

}  // namespace cmx

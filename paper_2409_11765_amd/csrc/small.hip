// Whole eigensolve C = B D^2 B^T (Sec. 2.1) of a descent with n <= 64 in one
// workgroup, from the covariance to the canonical B, D and B D; the descents of
// a group side by side, one workgroup each.
//
// The steps are those of the refinement by products (refine.hip): with V the
// eigenvectors so far (B_old at first), S = V^T C V and R = I - V^T V give every
// pair's angle, V <- V (I + Theta + R / 2 + Theta^2 / 2 + Theta^3 / 6).  All
// matrices stay in LDS and C in the registers of the waves that multiply by
// it; every wave forms one 16 x 16 block of a product on the float64 matrix
// cores, so a step is a handful of barriers.  While the angles are too large
// for that, a sweep of disjoint Jacobi rotations (n / 2 at a time, a round-robin
// over the n indices) makes them smaller first.  Angles can grow again: a close
// pair comes to light once what hid it has been turned away.  V, orthogonal
// only to some order after a step, is then made so (steps with Theta = 0)
// before the next sweep.
//
// Bound by one CU: at n = 64 a step takes 17 us, of which its six products
// occupy the matrix cores for 10 (64 cycles for each of 4096 / 16 instructions a
// product), and a sweep of 63 rounds, two barriers each, about 35.  A warm
// solve takes 5-9 steps: 17-34 us at n = 10, 133 us at n = 64.  Against block
// sweeps of 13 launches each with a host check between them, a whole generation
// went by this solve alone from 116 to 88 us at n = 10 (lambda = 10), 315 to 167
// at n = 40 (lambda = 15) and 343 to 233 at n = 64 (lambda = 16); the first twelve
// from C = I at n = 64, lambda = 16 took longer (532 against 497 us on average).
#include "internal.h"
#include "refine.h"

namespace cmx {

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

// a product's 16 x 16 block (bi, bj) over kb k-blocks of 16: X(m, k) =
// xs[m * LD + k], or with XT xs[k * LD + m]; Y(k, c) = ys[k * LD + c].  The
// result holds (row, column) = (l >> 4) + 4 r, l & 15 of the block in acc[r].
template <int LD, bool XT>
__device__ __forceinline__ doublex4 block_product(const double* xs, const double* ys, int kb, int bi, int bj) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  doublex4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int kk = 0; kk < kb; ++kk)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = 16 * kk + 4 * s + lk;
      const double a = XT ? xs[k * LD + 16 * bi + li] : xs[(16 * bi + li) * LD + k];
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, ys[k * LD + 16 * bj + li], acc, 0, 0, 0);
    }
  return acc;
}

// round-robin pairing of ne (even) players, round r, pair x
__device__ __forceinline__ void player_pair(int ne, int r, int x, int& a, int& b) {
  if (x == 0) {
    a = r;
    b = ne - 1;
  } else {
    a = r + x;
    a = a >= ne - 1 ? a - (ne - 1) : a;
    b = r - x;
    b = b < 0 ? b + (ne - 1) : b;
  }
}

// One sweep of rotations of A (n x n, the lower triangle of a symmetric matrix)
// in LDS, accumulated in V.  A round has two phases: the first wave forms the
// rotations of the n / 2 pairs while every wave turns V by the round before;
// then the thread of the pairs (x, y), x >= y, turns the four entries of A that
// the two share, in place.  With n odd the player past the end is a zero row
// and column, which nothing turns.
template <int NB, int LD>
__device__ void rotation_sweep(double* A, double* V, double2 (*rot)[8 * NB], int n, double thr, double inv) {
  constexpr int H = 8 * NB;
  const int ne = n + (n & 1), h = ne / 2;
  const int t = threadIdx.x, vx = t % H, vy = t / H;
  int ux = static_cast<int>((sqrtf(8.0f * t + 1.0f) - 1.0f) * 0.5f);
  while ((ux + 1) * (ux + 2) / 2 <= t) ++ux;
  while (ux * (ux + 1) / 2 > t) --ux;
  const int uy = t - ux * (ux + 1) / 2;
  auto at = [](int a, int b) { return max(a, b) * LD + min(a, b); };
  for (int r = 0; r < ne; ++r) {
    const bool turn = r < ne - 1;
    if (turn && t < h) {
      int a, b;
      player_pair(ne, r, t, a, b);
      double c, s;
      jacobi_rotation(A[a * LD + a], A[b * LD + b], A[at(a, b)], thr, inv, c, s);
      rot[r & 1][t] = make_double2(c, s);
    }
    if (r > 0 && vx < h && vy < h) {
      int a, b;
      player_pair(ne, r - 1, vx, a, b);
      const double2 cs = rot[(r - 1) & 1][vx];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        double* row = V + (2 * vy + q) * LD;
        const double va = row[a], vb = row[b];
        row[a] = cs.x * va - cs.y * vb;
        row[b] = cs.y * va + cs.x * vb;
      }
    }
    __syncthreads();
    if (turn && ux < h) {
      int ax, bx, ay, by;
      player_pair(ne, r, ux, ax, bx);
      player_pair(ne, r, uy, ay, by);
      const double2 x = rot[r & 1][ux], y = rot[r & 1][uy];
      const int i00 = at(ax, ay), i01 = at(ax, by), i10 = at(bx, ay), i11 = at(bx, by);
      const double m00 = A[i00], m01 = A[i01], m10 = A[i10], m11 = A[i11];
      const double p00 = m00 * y.x - m01 * y.y, p01 = m00 * y.y + m01 * y.x;
      const double p10 = m10 * y.x - m11 * y.y, p11 = m10 * y.y + m11 * y.x;
      A[i00] = x.x * p00 - x.y * p10;
      A[i01] = x.x * p01 - x.y * p11;
      A[i10] = x.y * p00 + x.x * p10;
      A[i11] = x.y * p01 + x.x * p11;
    }
    __syncthreads();
  }
}

// largest ||Theta||_F^2 / n of a step: a sweep of n - 1 rounds costs two steps
// here, so less is left to the steps than in refine.hip (generations at n = 64,
// lambda = 16, the first twelve / the next: 0.12 575 / 320 us, 0.25 532 / 297, 0.5
// 602 / 283, 1.0 606 / 312)
constexpr double kThLimitSmall = 0.25;
constexpr double kThLimitAgain = 0.02;  // when a solve starts over
constexpr double kRLimitSmall = 0.5;    // of ||R||_F^2; a solve starts over beyond it
constexpr double kRSweep = 1e-20;       // ||R||_F^2 a sweep can start from
constexpr int kMaxSmallSteps = 80;

template <int NB>
__global__ void __launch_bounds__(64 * NB * NB) kg_whole(const GEigDesc* __restrict__ g, int count, GroupDueMask due,
                                                         int max_sweeps, int* __restrict__ hsweeps) {
  constexpr int S = 16 * NB, LD = S + 1, NW = NB * NB, NT = 64 * NW;
  __shared__ double Vl[S * LD], Tl[S * LD], Sl[S * LD], Gl[S * LD];
  __shared__ double ev[S], dg[S], sgn[S];
  __shared__ double red[2][NW];
  __shared__ double2 rot[2][S / 2];
  __shared__ int perm[S];
  const int i = blockIdx.x;
  if (i >= count) return;
  const GEigDesc& e = g[i];
  if (e.N != S) return;
  int* ctl = e.ctl;
  const int n = e.n, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int li = lane & 15, lk = lane >> 4, bi = w % NB, bj = w / NB;
  if (t == 0) ctl[GC_DUE] = 0;  // nothing for the block sweeps to do
  if (!due_mask_bit(due, i)) return;
  const int nb = (n + 15) / 16;
  const bool mine = bi < nb && bj < nb;
  // this wave's rows of C (C is symmetric: read along its columns)
  double creg[4 * NB];
#pragma unroll
  for (int s = 0; s < 4 * NB; ++s) {
    const int m = 16 * bi + li, k = 4 * s + lk;
    creg[s] = m < n && k < n ? e.C[static_cast<int64_t>(m) * e.ldc + k] : 0.0;
  }
  auto load_v = [&](bool identity) {
    for (int idx = t; idx < S * S; idx += NT) {
      const int r = idx % S, c = idx / S;
      const double v = identity ? (r == c ? 1.0 : 0.0) : r < n && c < n ? e.B[static_cast<int64_t>(c) * e.ldb + r] : 0.0;
      Vl[r * LD + c] = r < n && c < n ? v : 0.0;
    }
  };
  load_v(false);
  __syncthreads();
  auto put = [&](double* m, const doublex4& acc) {
#pragma unroll
    for (int r = 0; r < 4; ++r) m[(16 * bi + lk + 4 * r) * LD + 16 * bj + li] = acc[r];
  };
  // the sums of two values over the workgroup
  auto add_up = [&](double& x, double& y) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      x += __shfl_xor(x, m);
      y += __shfl_xor(y, m);
    }
    if (lane == 0) {
      red[0][w] = x;
      red[1][w] = y;
    }
    __syncthreads();
    x = red[0][lane % NW];
    y = red[1][lane % NW];
#pragma unroll
    for (int m = NW / 2; m >= 1; m >>= 1) {
      x += __shfl_xor(x, m);
      y += __shfl_xor(y, m);
    }
  };
  int sweeps = 0, steps = 0, tries = 0, code = 0;
  double limit = kThLimitSmall;
  while (code == 0) {
    // T = C V, G = V^T V
    if (mine) {
      doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4 * NB; ++s)
        if (s < 4 * nb)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(creg[s], Vl[(4 * s + lk) * LD + 16 * bj + li], acc, 0, 0, 0);
      const doublex4 gg = block_product<LD, true>(Vl, Vl, nb, bi, bj);
      put(Tl, acc);
      put(Gl, gg);
    }
    __syncthreads();
    if (mine) put(Sl, block_product<LD, true>(Vl, Tl, nb, bi, bj));  // S = V^T T
    __syncthreads();
    if (t < S) dg[t] = t < n ? Sl[t * LD + t] / Gl[t * LD + t] : 0.0;
    __syncthreads();
    // Theta into T, and above S's diagonal what the rotation of a pair adds to
    // its eigenvalues; norms.  The pairs of rows i and ne - 1 - i together are
    // one row of ne - 1 threads.
    double dmax = fabs(dg[lane % S]);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, m));
    const double eps = 2.2e-16 * dmax, unit = unit_scale(dmax), noise = unit * noise_level(n, eps);
    double th2 = 0.0, r2 = 0.0, all2 = 0.0;
    const int ne = n + (n & 1);
    for (int idx = t; idx < ne / 2 * (ne - 1); idx += NT) {
      const int i = idx / (ne - 1), j = idx - i * (ne - 1);
      const int hi = j >= i ? j + 1 : ne - 1 - j, lo = j >= i ? i : ne - 1 - i;
      if (hi >= n) continue;
      const double rij = -Gl[hi * LD + lo];
      const double a = Sl[hi * LD + lo] + 0.5 * rij * (dg[hi] + dg[lo]);
      bool counts;
      const double h = refine_angle(unit * a, unit * (dg[hi] - dg[lo]), noise, counts);
      Tl[lo * LD + hi] = h;
      Tl[hi * LD + lo] = -h;
      Sl[lo * LD + hi] = h * a;
      if (counts) th2 = fma(2.0 * h, h, th2);
      r2 = fma(2.0 * rij, rij, r2);
      all2 = fma(2.0 * a, a, all2);
    }
    if (t < n) {
      const double rii = 1.0 - Gl[t * LD + t];
      r2 = fma(rii, rii, r2);
      all2 = fma(dg[t], dg[t], all2);
      Tl[t * LD + t] = 0.0;
    }
    // C is refused if it is not finite, or so large that the sum of its squares is
    // not (as by the sweeps' test): that sum is formed only where a thread's part of
    // it is near the end of the range, which a NaN in th2 tells all of them
    const double part = th2;
    if (!(all2 < 1e300)) th2 = __builtin_nan("");
    add_up(th2, r2);
    if (th2 != th2) {
      th2 = part;
      __syncthreads();
      add_up(th2, all2);
      if (!isfinite(all2)) r2 = all2;
    }
    bool square = true;
    if (!isfinite(th2) || !(r2 <= kRLimitSmall)) {
      // the steps went astray, B_old is not orthogonal, or C is not finite:
      // once more from B_old, then from the identity
      if (++tries == 3) {
        code = isfinite(th2) && isfinite(r2) ? 2 : 3;
        break;
      }
      if (steps == 0) tries = 2;
      limit = kThLimitAgain;
      load_v(tries == 2);
      __syncthreads();
      continue;
    }
    if (th2 > limit * n) {
      if (r2 <= kRSweep) {
        if (sweeps >= max_sweeps) {
          code = 2;
          break;
        }
        rotation_sweep<NB, LD>(Sl, Vl, rot, n, eps, dmax > 0.0 ? 1.0 / dmax : 0.0);
        ++sweeps;
        continue;
      }
      square = false;  // Theta = 0: only V's orthogonality
    }
    if (steps >= kMaxSmallSteps) {
      code = 2;
      break;
    }
    const bool last = square && th2 <= kDone * kDone && r2 <= kDoneR * kDoneR;
    if (last) {
      if (t < n) {
        double e = dg[t];
        for (int k = 0; k < t; ++k) e += Sl[k * LD + t];
        for (int k = t + 1; k < n; ++k) e -= Sl[t * LD + k];
        ev[t] = e;
      }
      __syncthreads();
    }
    // Theta^2 into S, X into G, V <- V X
    if (mine && square) {
      const doublex4 sq = block_product<LD, true>(Tl, Tl, nb, bi, bj);
      put(Sl, -sq);
    }
    __syncthreads();
    const bool cube = square && th2 > kCubeFrom * kCubeFrom;
    if (mine) {
      doublex4 p = {0.0, 0.0, 0.0, 0.0};
      if (cube) p = block_product<LD, true>(Tl, Sl, nb, bi, bj);  // -Theta^3
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * bi + lk + 4 * r, col = 16 * bj + li, at = row * LD + col;
        const double id = row == col ? 1.0 : 0.0;
        Gl[at] = row < n && col < n
                     ? id + 0.5 * (id - Gl[at]) + (square ? 0.5 * Sl[at] + Tl[at] - p[r] * (1.0 / 6.0) : 0.0)
                     : 0.0;
      }
    }
    __syncthreads();
    doublex4 nv = {0.0, 0.0, 0.0, 0.0};
    if (mine) nv = block_product<LD, false>(Vl, Gl, nb, bi, bj);
    __syncthreads();
    if (mine) put(Vl, nv);
    __syncthreads();
    ++steps;
    if (last) code = 1;
  }
  if (code != 1 && t < n) ev[t] = dg[t];
  __syncthreads();
  if (t == 0) {
    int* st = e.status;
    st[0] = code;
    st[1] = sweeps + steps;
    st[2] = 0;
    ctl[GC_LAST] = sweeps + steps;
    __hip_atomic_store(&hsweeps[i], sweeps + steps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&hsweeps[kGroupMax + i], code, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  // ascending eigenvalues (ties by index), each column's largest-magnitude
  // entry (first on ties) positive, then B, D and B D in that order
  if (t < S) perm[t] = t;  // (non-finite eigenvalues can leave ranks unassigned)
  __syncthreads();
  if (t < n) {
    const double vi = ev[t];
    int cnt = 0;
    for (int j = 0; j < n; ++j) cnt += (ev[j] < vi) || (ev[j] == vi && j < t);
    perm[cnt] = t;
    e.perm[cnt] = t;
    e.evals[t] = vi;
    double best = -1.0;
    int arg = 0;
    for (int r = 0; r < n; ++r) {
      const double v = fabs(Vl[r * LD + t]);
      if (v > best) {
        best = v;
        arg = r;
      }
    }
    sgn[t] = Vl[arg * LD + t] < 0.0 ? -1.0 : 1.0;
    e.sign[t] = sgn[t];
    if (cnt == 0) {
      e.sc->eig_ok = (vi > 0.0 && code == 1) ? 1 : 0;
      e.sc->jac_sweeps = sweeps + steps;
      e.sc->jac_corr = 0;
    }
  }
  __syncthreads();
  for (int idx = t; idx < n * n; idx += NT) {
    const int r = idx / n, row = idx - r * n;  // output column r, row
    const int cc = min(max(perm[r], 0), n - 1);
    const double d = sqrt(fmax(ev[cc], 0.0));
    const double v = sgn[cc] * Vl[row * LD + cc];
    if (row == 0) e.D[r] = d;
    e.B[static_cast<int64_t>(r) * e.ldb + row] = v;
    if (e.bd64)
      static_cast<double*>(e.BD)[static_cast<int64_t>(r) * e.ldbd + row] = v * d;
    else
      static_cast<float*>(e.BD)[static_cast<int64_t>(r) * e.ldbd + row] = static_cast<float>(v * d);
  }
}

}  // namespace

hipError_t launch_group_whole(hipStream_t st, const GEigDesc* g, int count, const GroupDueMask& due, int max_sweeps,
                              int* hsweeps, bool any32, bool any64) {
  static_assert(kWholeSolveN == 64, "the two sizes below");
  if (any32) kg_whole<2><<<count, 256, 0, st>>>(g, count, due, max_sweeps, hsweeps);
  if (any64) kg_whole<4><<<count, 1024, 0, st>>>(g, count, due, max_sweeps, hsweeps);
  return hipGetLastError();
}

}  // namespace cmx

// What the eigensolve's parts share: block-Jacobi sweeps (eigen.hip), the
// refinement by products over the whole GPU (refine.hip) and the whole solve in
// one workgroup (small.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace cmx {

// Largest ||Theta||_F^2 / n of a solve's first step (the sweep that comes first
// beyond it lowers a large one faster than the three to four steps of its time do;
// below it the steps are faster), and of the first step after steps that went
// astray; largest ||R||_F^2 / n of any step.
constexpr double kThLimit = 4.0;
constexpr double kThCareful = 0.05;
constexpr double kRLimit = 0.01;
// Longest row of Theta; the entries of longer ones are scaled down.  The angles
// of a row are right one by one, but in a cluster of eigenvalues they act on the
// same few dimensions and together overshoot.  The shorter the rows, the more
// clusters converge, and the slower all else does, so the length follows how
// much ||Theta||_F^2 fell in the step before (before = 0: the first step).
// Without it steps went astray from ||Theta||_F^2 = 0.7 n on and left 6-14 sweeps to
// the first generations of a search.
__device__ __forceinline__ double longest_row(double th2, double before, int n) {
  if (before == 0.0) return th2 > 2.0 * n ? 0.5 : 0.75;
  return th2 > 0.9 * before ? 0.4 : th2 > 0.8 * before ? 0.55 : 0.75;
}
constexpr double kClip = 0.35;
// a step is the last one once ||Theta||_F and ||R||_F are below these (what it
// leaves of each is of the order of ||R||_F times either), or once the angles
// no longer shrink (||Theta||_F^2 by less than kStall a step) and the off-diagonal
// norm would end a solve by sweeps, kOffDone of the whole: rounding against
// rounding inside a close cluster of eigenvalues
constexpr double kDone = 2e-7;
constexpr double kDoneR = 1e-7;
constexpr double kOffDone = 1e-13;
constexpr double kStall = 0.1;
// Theta^3 / 6 is left out once ||Theta||_F is below this
constexpr double kCubeFrom = 1e-3;
// Entries at the level of the products' rounding (0.7 sqrt(n) eps each, eps =
// 2.2e-16 max d, as measured for V far from the identity at n = 1000; up to 4
// sqrt(n) eps here) are as small as they can get: they do not count, and turn
// nothing by more than kNoiseAngle (inside a multiple eigenvalue their angles
// are arbitrary, and X is orthogonal only while they are small).  Between
// separated eigenvalues they are turned, however small: left at eps, as the
// sweeps leave them, B was off by 2.8e-13 at n = 333 and a condition of 100.
constexpr double kNoiseAngle = 1e-6;
__device__ __forceinline__ double noise_level(int n, double eps) { return fmax(16.0, 4.0 * sqrt(static_cast<double>(n))) * eps; }

// the power of two that takes v to [1/2, 1): angles are formed from values scaled by
// it, whose squares then neither overflow nor vanish, and are the same bits
__device__ __forceinline__ double unit_scale(double v) { return ldexp(1.0, min(-__builtin_amdgcn_frexp_exp(v), 1000)); }

// angle of the rotation of a pair with off-diagonal entry a and eigenvalue
// difference g (scaled, as the noise); counts: whether it is above the noise
__device__ __forceinline__ double refine_angle(double a, double g, double noise, bool& counts) {
  counts = fabs(a) > noise;
  if (!(fabs(a) > 0.0)) return 0.0;
  const double t = 2.0 * a / (fabs(g) + sqrt(fma(g, g, 4.0 * a * a)));
  double h = t / fma(0.28, t * t, 1.0);  // atan(t) to 0.005, exact to first order
  h = g < 0.0 ? -h : h;
  if (!counts && fabs(h) > kNoiseAngle) h = 0.0;
  return fmin(fmax(h, -kClip), kClip);
}

// Jacobi rotation J = [[c, s], [-s, c]] on (a, b) that annihilates (J^T S J)_ab
// up to the accuracy of t (Golub & Van Loan, sym.schur2): t = sign(delta) 2 d /
// (|delta| + sqrt(delta^2 + 4 d^2)) with delta = S_bb - S_aa, d = S_ab;
// c = 1/sqrt(1 + t^2), s = t c; the identity when |d| <= thr.
// t only decides how far the entry is reduced, so it is formed in float32 from
// the entries scaled by inv = 1/max|a_ii| (relative error ~1e-7: the entry
// drops to ~1e-7 of itself and later rotations remove the rest).  c is then
// refined to float64 precision from that t by two Newton steps, because
// c^2 (1 + t^2) = 1 is what keeps each rotation, and so Q, orthogonal.
// Branch free, so the callers' loads issue up front and two rotations
// interleave.
__device__ __forceinline__ void jacobi_rotation(double saa, double sbb, double d, double thr, double inv, double& c,
                                                double& s) {
  const double dd = fabs(d) > thr ? d : 0.0;
  const float df = static_cast<float>(dd * inv);
  const float delta = static_cast<float>((sbb - saa) * inv);
  const float h = __builtin_amdgcn_sqrtf(fmaf(delta, delta, 4.0f * df * df));
  // |delta| + h >= 2 |df| > 0 whenever df != 0; the floor only guards 0 / 0
  const float tf = (delta >= 0.0f ? 2.0f : -2.0f) * df * __builtin_amdgcn_rcpf(fmaxf(fabsf(delta) + h, 1e-30f));
  const double t = static_cast<double>(tf);
  const double x = fma(t, t, 1.0);
  double y = static_cast<double>(__builtin_amdgcn_rsqf(fmaf(tf, tf, 1.0f)));
  y = y * fma(-0.5 * x * y, y, 1.5);
  c = y * fma(-0.5 * x * y, y, 1.5);
  s = t * c;
}

}  // namespace cmx

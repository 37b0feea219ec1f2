// Device helpers of the ADG library: delay draw, AT weights, one-step
// reactive-Euler physics and the numerical fluxes.
#pragma once

#include "adg_internal.hpp"

namespace adg {

// SplitMix64 output function (Steele, Lea & Flood 2014).
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long x) {
  unsigned long long z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Cross-lane moves by the data-parallel-primitive (DPP) modifier, without the LDS
// crossbar.  dpp_move<CTRL>(x) returns the x of the lane that CTRL selects (a lane
// with no source keeps its own x): quad permutations, row mirrors and the
// wavefront shifts.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
  const unsigned long long v = (unsigned long long)__double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp((int)(unsigned)v, (int)(unsigned)v, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(unsigned)(v >> 32), (int)(unsigned)(v >> 32), CTRL, 0xF, 0xF,
                                             false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
template <int CTRL>
__device__ __forceinline__ int dpp_move(int x) {
  return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
}
constexpr int kDppFromNext = 0x130;   // lane l takes lane l+1's value (wavefront shift)
constexpr int kDppFromPrev = 0x138;   // lane l takes lane l-1's value
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane l takes lane 7-l of its group of 8
constexpr int kDppMirror = 0x140;     // lane l takes lane 15-l of its group of 16

// n mod d for a step count n >= 0 and 0 < d: in 32-bit arithmetic while n fits
// (a 64-bit remainder by a run-time divisor is a long instruction sequence).
__device__ __forceinline__ int step_mod(long long n, int d) {
  return n >= 0 && n <= 0x7fffffffll ? (int)((unsigned)n % (unsigned)d) : (int)(n % d);
}

// Delay at PE interface i for time step n (Sec. 4), clamped so that all q
// levels n-k .. n-k-q+1 exist.  BRANCH_FREE: the SAA bin is counted over all
// kMaxL - 1 bin edges with the loads of every edge issued together (the
// detailed-chemistry load phase, where the draw sits between the loads and the
// barrier); otherwise the bins are searched in order (the one-step kernels,
// where most draws end at the first edges).  Both give the same bin: the first
// j with u < cum[j] (cum is non-decreasing), at most L - 1.
template <bool BRANCH_FREE = false>
__device__ __forceinline__ int eff_delay(const DelayParams &d, long long n, int i) {
  int k = 0;
  if (d.mode == 1) {
    k = step_mod(n, d.L);
  } else if (d.mode == 2) {
    unsigned long long ctr = (unsigned long long)n * (unsigned long long)d.nif + (unsigned long long)i;
    unsigned long long z = splitmix64(d.seed ^ (ctr * 0x9E3779B97F4A7C15ull));
    double u = (double)(z >> 11) * 0x1.0p-53;
    if constexpr (BRANCH_FREE) {
#pragma unroll
      for (int j = 0; j < kMaxL - 1; ++j) k += (j < d.L - 1 && u >= d.cum[j]) ? 1 : 0;
    } else {
      k = d.L - 1;
      for (int j = 0; j < d.L; ++j)
        if (u < d.cum[j]) { k = j; break; }
    }
  } else if (d.mode == 3) {
    k = d.sched[(long long)step_mod(n, d.sched_steps) * d.nif + i];
  }
  if (k <= 0) return 0;
  long long lim = n - d.q + 1;
  if (lim < 0) lim = 0;
  return k > lim ? (int)lim : k;
}

// Weight of level n-k-j in the AT combination of Eq. (7): the Lagrange
// extrapolation weight prod_{m != j} (k+m)/(m-j), which is the solution of
// Eq. (8).  Numerator and denominator are integers below 2^53 (k < 8, q <= 6), so
// their products are exact in FP64; one rounding, in the quotient.
__device__ __forceinline__ double at_weight(int q, int k, int j) {
  double num = 1.0, den = 1.0;
  for (int m = 0; m < q; ++m) {
    if (m == j) continue;
    num *= (double)(k + m);
    den *= (double)(m - j);
  }
  return num / den;
}

// Weight of level n-k-l for Legendre mode j of a buffer element (Eq. (11)): the temporal
// stencil uses all q levels for every mode; the hybrid spatio-temporal one extrapolates mode j,
// which carries the factor dx^j, from q_j = max(1, q - j) levels with the weights of that order
// (0 for the levels it does not use).
__device__ __forceinline__ double buffer_weight(const DelayParams &d, int k, int j, int l) {
  const int qj = d.hybrid ? max(1, d.q - j) : d.q;
  return l < qj ? at_weight(qj, k, l) : 0.0;
}
__device__ __forceinline__ int buffer_levels(const DelayParams &d, int j) { return d.hybrid ? max(1, d.q - j) : d.q; }

// End of time step n in the step's last launch (parity par): the next step's
// count goes to the other parity's counter.  Every launch of step n reads
// step[par] only, so one workgroup's plain store needs no atomic, no barrier and
// no wait; the next step's launches read it after this launch has ended.
__device__ __forceinline__ void advance_step(long long *step, int par, long long n, bool first_workgroup) {
  if (first_workgroup && threadIdx.x == 0) step[par ^ 1] = n + 1;
}

// ---------------------------------------------------------------- elementary functions
// The errors stated are the largest of 4 million arguments drawn from each range, against 64-bit-mantissa
// arithmetic.
// ln 2 to 42 bits (its product with an exponent is exact) and the rest.
constexpr double kLn2Hi = 0x1.62e42fefa3800p-1, kLn2Lo = 0x1.ef35793c76730p-45, kInvLn2 = 1.4426950408889634;

// exp(x): k = rint(x / ln 2), r = x - k ln 2 in two parts, the Taylor polynomial of degree 13 in
// |r| <= ln(2)/2 (its remainder is below 2^-57 of the result), 2^k by ldexp, which saturates to 0
// and infinity.  For arguments of a size below 2^30; 0.89 ulp on |x| <= 700.
__device__ __forceinline__ double exp_taylor(double x) {
  const double k = __builtin_rint(x * kInvLn2);
  double r = fma(k, -kLn2Hi, x);
  r = fma(k, -kLn2Lo, r);
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return __builtin_amdgcn_ldexp(p, (int)k);
}

// exp_taylor with its polynomial split by powers of r^2, r^4 and r^8: two more multiplications, and half
// of the dependent chain, for where one wavefront waits for one value.  1.73 ulp on |x| <= 700.
__device__ __forceinline__ double exp_short(double x) {
  const double k = __builtin_rint(x * kInvLn2);
  double r = fma(k, -kLn2Hi, x);
  r = fma(k, -kLn2Lo, r);
  const double r2 = r * r, r4 = r2 * r2, r8 = r4 * r4;
  const double a = fma(r2, fma(r, 1.0 / 6.0, 0.5), 1.0 + r);
  const double b = fma(r2, fma(r, 1.0 / 5040.0, 1.0 / 720.0), fma(r, 1.0 / 120.0, 1.0 / 24.0));
  const double c = fma(r2, fma(r, 1.0 / 39916800.0, 1.0 / 3628800.0), fma(r, 1.0 / 362880.0, 1.0 / 40320.0));
  const double d = fma(r, 1.0 / 6227020800.0, 1.0 / 479001600.0);
  return __builtin_amdgcn_ldexp(fma(r4, fma(r8, d, fma(r4, c, b)), a), (int)k);
}

// 1/x by the hardware estimate and two Newton steps, for x away from the ends of the range: correctly
// rounded but for rare last bits (0.500 ulp on 1e-300 .. 1e300).
__device__ __forceinline__ double recip(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

// log(x) of a normal positive x: x = 2^k m with sqrt(1/2) <= m < sqrt(2), s = (m-1)/(m+1), and
// log m = 2 artanh s by its series up to s^19 (|s| < 0.172: the rest is below 2^-55 of log m),
// split like exp_short's polynomial.  An infinite or NaN x gives NaN.  0.63 ulp on 200 .. 6000 (the
// temperatures it is used for), up to 2.5 ulp around 1, where log x is small.
__device__ __forceinline__ double log_short(double x) {
  double m = __builtin_amdgcn_frexp_mant(x);
  int k = __builtin_amdgcn_frexp_exp(x);
  const bool low = m < 0.70710678118654752;
  m = low ? m + m : m;
  k = low ? k - 1 : k;
  const double s = (m - 1.0) * recip(m + 1.0), z = s * s, z2 = z * z, z4 = z2 * z2;
  const double a = fma(z2, fma(z, 1.0 / 9.0, 1.0 / 7.0), fma(z, 1.0 / 5.0, 1.0 / 3.0));
  const double b = fma(z2, fma(z, 1.0 / 17.0, 1.0 / 15.0), fma(z, 1.0 / 13.0, 1.0 / 11.0));
  const double p = fma(z4, fma(z4, 1.0 / 19.0, b), a), s2 = s + s;
  return fma((double)k, kLn2Hi, s2 + fma(s2 * z, p, (double)k * kLn2Lo));
}

// Square root of a positive x from the hardware's estimate of 1/sqrt(x): one coupled step for the root g
// and half its reciprocal h (Goldschmidt's iteration), then the remainder x - g^2 folded in twice.  0.500
// ulp on 1e-290 .. 1e290.
__device__ __forceinline__ double root(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  r = fma(-g, g, x);
  g = fma(r, h, g);
  r = fma(-g, g, x);
  return fma(r, h, g);
}

// ---------------------------------------------------------------- one-step model
struct Prim1 {
  double rho, u, p, T, a;
};

// rho E = rho u^2/2 + p/(gamma-1) + q rho Y_R;  T = p/rho (R = 1).
__device__ __forceinline__ bool prim1(const OneStep &ph, const double *w, Prim1 &pr) {
  pr.rho = w[0];
  const double rinv = recip(pr.rho);
  pr.u = w[1] * rinv;
  pr.p = (ph.gamma - 1.0) * (w[2] - 0.5 * w[1] * pr.u - ph.q_heat * w[3]);
  pr.T = pr.p * rinv;
  pr.a = root(ph.gamma * pr.T);
  return pr.rho > 0.0 && pr.p > 0.0 && isfinite(pr.p) && isfinite(pr.rho);
}

__device__ __forceinline__ void flux1(const double *w, const Prim1 &pr, double *f) {
  f[0] = w[1];
  f[1] = w[1] * pr.u + pr.p;
  f[2] = pr.u * (w[2] + pr.p);
  f[3] = w[3] * pr.u;
  f[4] = w[4] * pr.u;
}

// Local Lax-Friedrichs flux of Sec. 3.1.
__device__ __forceinline__ bool rusanov1(const OneStep &ph, const double *wm, const double *wp, double *f) {
  Prim1 pm, pp;
  bool ok = prim1(ph, wm, pm);
  ok = prim1(ph, wp, pp) && ok;
  double fm[5], fp[5];
  flux1(wm, pm, fm);
  flux1(wp, pp, fp);
  double lm = fabs(pm.u) + pm.a, lp = fabs(pp.u) + pp.a;
  double lam = lm > lp ? lm : lp;
#pragma unroll
  for (int v = 0; v < 5; ++v) f[v] = 0.5 * (fm[v] + fp[v] - lam * (wp[v] - wm[v]));
  return ok;
}

// HLLC (Toro, Spruce & Speares 1994) with Davis wave-speed bounds.
__device__ __forceinline__ bool hllc1(const OneStep &ph, const double *wm, const double *wp, double *f) {
  Prim1 pm, pp;
  bool ok = prim1(ph, wm, pm);
  ok = prim1(ph, wp, pp) && ok;
  double SL = fmin(pm.u - pm.a, pp.u - pp.a);
  double SR = fmax(pm.u + pm.a, pp.u + pp.a);
  if (SL >= 0.0) { flux1(wm, pm, f); return ok; }
  if (SR <= 0.0) { flux1(wp, pp, f); return ok; }
  double num = pp.p - pm.p + pm.rho * pm.u * (SL - pm.u) - pp.rho * pp.u * (SR - pp.u);
  double den = pm.rho * (SL - pm.u) - pp.rho * (SR - pp.u);
  double Ss = num * recip(den);
  const bool left = Ss >= 0.0;
  const double *wk = left ? wm : wp;
  const Prim1 &pk = left ? pm : pp;
  const double Sk = left ? SL : SR;
  double fk[5];
  flux1(wk, pk, fk);
  // w* = c (rho, rho Ss, E + (Ss - u)(rho Ss + p/(Sk - u)), rho Y), c = (Sk - u)/(Sk - Ss)
  const double du = Sk - pk.u, c = du * recip(Sk - Ss);
  double ws[5];
  ws[0] = c * pk.rho;
  ws[1] = ws[0] * Ss;
  ws[2] = c * (wk[2] + (Ss - pk.u) * (pk.rho * Ss + pk.p * recip(du)));
  ws[3] = c * wk[3];
  ws[4] = c * wk[4];
#pragma unroll
  for (int v = 0; v < 5; ++v) f[v] = fk[v] + Sk * (ws[v] - wk[v]);
  return ok;
}

template <int FLUX>
__device__ __forceinline__ bool numflux1(const OneStep &ph, const double *wm, const double *wp, double *f) {
  if constexpr (FLUX == 1) return hllc1(ph, wm, wp, f);
  else return rusanov1(ph, wm, wp, f);
}

}  // namespace adg

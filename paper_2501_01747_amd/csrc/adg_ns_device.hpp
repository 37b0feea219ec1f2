// Device functions shared by the detailed-chemistry stage kernels.
#pragma once

#include "adg_device.hpp"
#include "adg_ns.hpp"

namespace adg {

// Temperature from the internal energy e* by Newton's method from the fixed
// start T_guess, at most 50 iterations.  The mixture energy sum_i Y_i e_i(T) is
// linear in the species, so it is one quintic
// e(T) = T (c0 + T (c1 + T (c2 + T (c3 + T c4)))) + c5; returns cv(T) too.
// Newton converges quadratically here (cv > 0 varies slowly with T): once a
// correction is below 1e-8 T the iterate it produces is within about 1e-16 T of
// the root, so the loop stops there, one iteration before a correction below
// 1e-12 T would show it.
__device__ __forceinline__ bool newton_T(const double (&c)[6], double T0, double estar, double &T, double &cv) {
  const double d1 = 2.0 * c[1], d2 = 3.0 * c[2], d3 = 4.0 * c[3], d4 = 5.0 * c[4];
  T = T0;
  bool conv = false;
  for (int it = 0; it < 50; ++it) {
    const double T2 = T * T;   // by powers of T^2: the shorter dependent chain
    const double e = fma(T2, fma(T2, fma(T, c[4], c[3]), fma(T, c[2], c[1])), fma(T, c[0], c[5]));
    const double cvi = fma(T2, fma(T2, d4, fma(T, d3, d2)), fma(T, d1, c[0]));
    const double dT = (e - estar) * __builtin_amdgcn_rcp(cvi);   // the correction needs no IEEE quotient
    T -= dT;
    if (!(T > 0.0) || !isfinite(T)) break;
    if (fabs(dT) <= 1e-8 * T) { conv = true; break; }
  }
  const double T2 = T * T;
  cv = fma(T2, fma(T2, d4, fma(T, d3, d2)), fma(T, d1, c[0]));
  return conv;
}

// x within [0, E) by whole periods; x lies in [-span, E + span).
__device__ __forceinline__ int wrap(int x, int E, int span) {
  if (E < span) return (x % E + E) % E;   // meshes shorter than a tile
  return x < 0 ? x + E : x >= E ? x - E : x;
}

// AT combination (Eq. (7)) of the central trace and the flux of variable v at interface i from
// the levels n-k .. n-k-q+1 of stage st: levels 0..3 given (w, f; a level past q holds level
// n-k and has weight 0), later ones (q > 4) read here one at a time.  The carried and the
// in-launch combinations both come from here, so they round alike.
__device__ __forceinline__ void at_combine(const NsArgs &a, int q, int k, int nmod, int st, int i, int v,
                                           const double (&w)[4], const double (&f)[4], double &acw, double &acf) {
  acw = 0.0;
  acf = 0.0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double c = j < q ? at_weight(q, k, j) : 0.0;
    acw += c * w[j];
    acf += c * f[j];
  }
  for (int j = 4; j < q; ++j) {
    const double c = at_weight(q, k, j);
    const double *rec = ring_at(a.ring, ring_slot(nmod, k + j, a.ring.D), st, a.dl.nif, i);
    acw += c * rec[a.ring.off_Wc + v];
    acf += c * rec[a.ring.off_F + v];
  }
}

// The next launch's AT combinations at the PE interfaces that a tile of TE elements from e0 owns
// (faces e0 .. e0+nloc-1): stage + 1 of this step, or stage 0 of the next; their levels all precede
// what this launch writes.  sI[fo + 1]: interface of face e0 + fo.  One lane (of nl, lane l) per
// (variable, face).
template <int V>
__device__ __forceinline__ void carry_at(const NsArgs &a, int stage, long long n, int e0, int nloc, int TE,
                                         const int *sI, int l, int nl) {
  const int Vg = 3 + a.ns, q_at = a.dl.q;
  for (int idx = l; idx < V * TE; idx += nl) {
    const int v = idx / TE, fo = idx % TE;
    const int i = sI[fo + 1];
    if (v < Vg && fo < nloc && i >= 0) {
      const bool last = stage == a.nst - 1;
      const long long n2 = n + (last ? 1 : 0);
      const int s2 = last ? 0 : stage + 1;
      const int k2 = eff_delay<true>(a.dl, n2, i);
      const size_t base = (size_t)(e0 + fo) * (2 * Vg + 1);
      if (v == 0) a.at_out[base + 2 * Vg] = (double)k2;
      if (k2 > 0) {
        const int nm2 = step_mod(n2, a.ring.D);
        double w[4], f[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double *rec = ring_at(a.ring, ring_slot(nm2, k2 + (j < q_at ? j : 0), a.ring.D), s2, a.dl.nif, i);
          w[j] = rec[a.ring.off_Wc + v];
          f[j] = rec[a.ring.off_F + v];
        }
        double acw, acf;
        at_combine(a, q_at, k2, nm2, s2, i, v, w, f, acw, acf);
        a.at_out[base + v] = acw;
        a.at_out[base + Vg + v] = acf;
      }
    }
  }
}

}  // namespace adg

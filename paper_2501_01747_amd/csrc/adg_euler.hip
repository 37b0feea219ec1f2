// Step kernel of the one-step reactive Euler model: a whole time step per launch, with the
// troubled-cell indicator and the characteristic (AT-)WENO limiter of every stage's output in the
// same kernel for a limited problem.
//
// Stage (Sec. 3.1 Eq. (5), Sec. 3.2 Eq. (7)): one thread per element; each
// wavefront owns consecutive elements and holds neighbours on each side.  Every lane loads its
// element's modal DoFs from the component planes (coalesced) and forms both face traces;
// one numerical flux per face is computed and passed to the neighbouring lane by
// a lane shift; at PE-interface faces the synchronous flux of this level is written
// to the history ring and replaced by the AT combination of past levels.  The
// volume integral, the source projection, the lift and the RK combination then
// run in registers.
//
// Limiter (Sec. 3.3, Eq. (9)-(11)): with a second halo lane per stage, every limited
// element's two neighbours have their unlimited stage outputs inside the
// same wavefront, so the indicator and the WENO reconstruction read them from
// LDS (every stencil sees unlimited data, the simultaneous application of the limiter).
#include "adg_device.hpp"

namespace adg {

template <int M>
__device__ __forceinline__ void traces(const double (&u)[5][M], double *wl, double *wr) {
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    double sm = 0.0, sp = 0.0;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      sp += u[v][j];
      sm += (j & 1) ? -u[v][j] : u[v][j];
    }
    wl[v] = sm;
    wr[v] = sp;
  }
}

template <int M>
__device__ __forceinline__ void load_elem(const double *__restrict__ w, int E, int e, double (&u)[5][M]) {
  const double *we = w + sidx(e, 0, 5 * M);
#pragma unroll
  for (int v = 0; v < 5; ++v)
#pragma unroll
    for (int j = 0; j < M; ++j) u[v][j] = we[(v * M + j) * kLayoutBlock];
}

// The AT flux of Eq. (7) at PE interface i with delay k > 0: the past levels' synchronous
// fluxes of this stage combined with the Eq. (8) weights.  Levels 0..3 are loaded together
// (a level past q reads level n-k with weight 0), later ones (q > 4) one at a time.
__device__ __forceinline__ void at_flux(const EulerArgs &a, int nmod, int stage, int i, int k, double (&acc)[5]) {
#pragma unroll
  for (int v = 0; v < 5; ++v) acc[v] = 0.0;
  const int q = a.dl.q;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool in = j < q;
    const double c = in ? at_weight(q, k, j) : 0.0;
    const double *h = ring_at(a.ring, ring_slot(nmod, k + (in ? j : 0), a.ring.D), stage, a.dl.nif, i) + a.ring.off_F;
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[v] += c * h[v];
  }
  for (int j = 4; j < q; ++j) {
    const double c = at_weight(q, k, j);
    const double *h = ring_at(a.ring, ring_slot(nmod, k + j, a.ring.D), stage, a.dl.nif, i) + a.ring.off_F;
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[v] += c * h[v];
  }
}

// ------------------------------------------------------------------- limiter

// Characteristic left and right eigenvectors at the mean state (one-step model).
// Rows of L (linear forms in the conserved variables):
//   (dp - rho a du)/(2a^2), drho - dp/a^2, d(rho Y_R) - Y_R drho,
//   d(rho Y_R + rho Y_P - rho), (dp + rho a du)/(2a^2),
// with dp and du the differentials of p and u.  R = L^-1 in closed form: column k
// is the conserved perturbation whose characteristic variables are e_k, built from
// the primitive perturbations (drho, du, dp, dY_R) that L maps to e_k.  L involves
// Y_R only, so the product entry of the columns with drho = 1 is 1 - Y_R (not the
// mean state's Y_P): R is then the exact inverse for any state, and the limiter
// keeps rho Y_R + rho Y_P - rho at round-off instead of feeding its round-off back.
// Field c only: row c of L into lr, column c of R into rc.
__device__ __forceinline__ bool char_row_col(const OneStep &ph, const double *wb, int c, double (&lr)[5],
                                             double (&rc)[5]) {
  Prim1 pr;
  const bool ok = prim1(ph, wb, pr);
  const double rho = pr.rho, u = pr.u, a = pr.a, g1 = ph.gamma - 1.0, q = ph.q_heat;
  const double irho = 1.0 / rho;
  const double dp[5] = {g1 * 0.5 * u * u, -g1 * u, g1, -g1 * q, 0.0};
  const double du[5] = {-u * irho, irho, 0.0, 0.0, 0.0};
  const double a2 = a * a, ia2 = 1.0 / a2;
  const double YR = wb[3] * irho, YP = 1.0 - YR;
  const double l2[5] = {-YR, 0.0, 0.0, 1.0, 0.0};
  const double l3[5] = {-1.0, 0.0, 0.0, 1.0, 1.0};
  // the acoustic rows carry the sign of their wave speed u -+ a
  const double sa = c == 0 ? -1.0 : 1.0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const double drho = k == 0 ? 1.0 : 0.0;
    const double ac = (dp[k] + sa * rho * a * du[k]) * (0.5 * ia2);
    lr[k] = (c == 0 || c == 4) ? ac : c == 1 ? drho - dp[k] * ia2 : c == 2 ? l2[k] : l3[k];
  }
  // columns: acoustic -, entropy, reactant, species sum, acoustic +
  const double hk = 0.5 * u * u + q * YR;   // d(rho E)/d rho at fixed u, p, Y
  const double ha = a2 / g1;
  if (c == 0 || c == 4) {
    rc[0] = 1.0; rc[1] = u + sa * a; rc[2] = ha + hk + sa * u * a; rc[3] = YR; rc[4] = YP;
  } else if (c == 1) {
    rc[0] = 1.0; rc[1] = u; rc[2] = hk; rc[3] = YR; rc[4] = YP;
  } else if (c == 2) {
    rc[0] = 0.0; rc[1] = 0.0; rc[2] = q; rc[3] = 1.0; rc[4] = -1.0;
  } else {
    rc[0] = 0.0; rc[1] = 0.0; rc[2] = 0.0; rc[3] = 0.0; rc[4] = 1.0;
  }
  return ok && a > 0.0;
}

// minmod of three numbers: the one of least magnitude if all share a sign, else 0
__device__ __forceinline__ double minmod3(double x, double y, double z) {
  if (x > 0.0 && y > 0.0 && z > 0.0) return fmin(x, fmin(y, z));
  if (x < 0.0 && y < 0.0 && z < 0.0) return fmax(x, fmax(y, z));
  return 0.0;
}

template <int M>
__device__ __forceinline__ double trace_at(const double (&c)[M], int side) {
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < M; ++j) s += (side == 0 && (j & 1)) ? -c[j] : c[j];
  return s;
}

// Where the limiter of an owned element takes the neighbour across one face from:
// LDS at base + v sv + j sj.  Either the neighbouring lane's unlimited output, or one
// of the wavefront's slots holding, at a transmissive end (ghost), the constant equal
// to the element's own mean, or at a PE interface i with effective delay k > 0 the
// Eq. (11) AT combination of the unlimited outputs that past levels published to the
// history ring, formed once per stage.
struct NbSide {
  int base, sv, sj, i, k, ghost;
};

// LDS per wavefront of the limiter: the unlimited outputs [5M][64], per stage kNbSlots neighbours
// [5M] (two per lane for kSlotLanes lanes at a time), and per stage the AT fluxes of kSlotLanes faces.
constexpr int kSlotLanes = 4;
constexpr int kNbSlots = 2 * kSlotLanes;
template <int M, int S>
constexpr int lds_wave_doubles() { return 5 * M * 64 + S * kNbSlots * 5 * M + S * kSlotLanes * 5; }

// Modes of variable v of the neighbour across one face.  ls is the wavefront's LDS area.
template <int M>
__device__ __forceinline__ void nb_var(const NbSide &sd, int v, const double *ls, double (&c)[M]) {
#pragma unroll
  for (int j = 0; j < M; ++j) c[j] = ls[sd.base + v * sd.sv + j * sd.sj];
}

// Troubled-cell indicator (KXRCF or TVB minmod) of the element in lane `lane`, its own unlimited modes
// and its neighbours' in the wavefront's LDS area ls, variable by variable (few registers: the
// element's modes stay in registers beside it).
template <int M>
__device__ __forceinline__ bool troubled(const EulerArgs &a, const LimiterArgs &l, const NbSide (&sd)[2],
                                         const double *ls, int lane) {
  const bool ghostL = sd[0].ghost, ghostR = sd[1].ghost;
  auto own = [&](int v, double (&c)[M]) {
#pragma unroll
    for (int j = 0; j < M; ++j) c[j] = ls[(v * M + j) * 64 + lane];
  };
  bool flag = false;
  if (l.indicator == 2) {
    flag = true;   // every cell limited (the accuracy-test setting of the WENO limiter)
  } else if (l.indicator == 1) {
    // TVB minmod: the face deviations from the mean against the mean differences, every
    // variable; differences within 1e-10 of the largest |mean| of any variable in the
    // stencil count as equal (round-off in a constant state is not a slope)
    double scale = 0.0;
#pragma unroll
    for (int v = 0; v < 5; ++v)
      scale = fmax(scale, fmax(fabs(ls[(v * M) * 64 + lane]),
                               fmax(fabs(ls[sd[0].base + v * sd[0].sv]), fabs(ls[sd[1].base + v * sd[1].sv]))));
    const double tol = 1e-10 * scale;
#pragma unroll 1
    for (int v = 0; v < 5; ++v) {
      double c[M];
      own(v, c);
      const double m = c[0];
      const double dp = trace_at<M>(c, 1) - m, dm = m - trace_at<M>(c, 0);
      const double Dp = ls[sd[1].base + v * sd[1].sv] - m, Dm = m - ls[sd[0].base + v * sd[0].sv];
      const double mp = fabs(dp) <= l.tvb_mh2 ? dp : minmod3(dp, Dp, Dm);
      const double mm = fabs(dm) <= l.tvb_mh2 ? dm : minmod3(dm, Dp, Dm);
      if (fabs(mp - dp) > tol || fabs(mm - dm) > tol) flag = true;
    }
  } else {
    // KXRCF: jumps at inflow faces against h^((N_p+1)/2) max_q |w(xi_q)|, on rho and rho E;
    // tL/tR: the neighbours' traces at the shared faces of rho, rho u, rho E; eL/eR the element's own
    double tL[3], tR[3], eL[3], eR[3];
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      double c[M];
      nb_var<M>(sd[0], v, ls, c);
      tL[v] = trace_at<M>(c, 1);
      nb_var<M>(sd[1], v, ls, c);
      tR[v] = trace_at<M>(c, 0);
      own(v, c);
      eL[v] = trace_at<M>(c, 0);
      eR[v] = trace_at<M>(c, 1);
    }
    const double uL_e = eL[1] / eL[0], uR_e = eR[1] / eR[0];
    const double uL_n = ghostL ? uL_e : tL[1] / tL[0];
    const double uR_n = ghostR ? uR_e : tR[1] / tR[0];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int v = t == 0 ? 0 : 2;
      double jump = 0.0;
      if (0.5 * (uL_e + uL_n) > 0.0 && !ghostL) jump += eL[v] - tL[v];
      if (0.5 * (uR_e + uR_n) < 0.0 && !ghostR) jump += eR[v] - tR[v];
      double c[M], norm = 0.0;
      own(v, c);
#pragma unroll
      for (int q = 0; q < M; ++q) {
        double val = 0.0;
#pragma unroll
        for (int j = 0; j < M; ++j) val += c[j] * a.tb.B[q][j];
        norm = fmax(norm, fabs(val));
      }
      if (fabs(jump) / (l.kx_h * norm) > 1.0) flag = true;
    }
  }
  return flag;
}

// The simple WENO reconstruction of Eq. (9)-(10) of one characteristic field with
// modes vc in the cell and vL, vR in its neighbours: the limited modes vl.
template <int M>
__device__ __forceinline__ void weno_field(const LimiterArgs &l, const double (&vc)[M], const double (&vL)[M],
                                           const double (&vR)[M], double (&vl)[M]) {
  // re-expand the neighbours in the cell's coordinate and reset their mean
  double tL[M], tR[M];
#pragma unroll
  for (int k2 = 0; k2 < M; ++k2) {
    double sl = 0.0, sr = 0.0;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      sl += l.Tl[k2][j] * vL[j];
      sr += l.Tr[k2][j] * vR[j];
    }
    tL[k2] = sl; tR[k2] = sr;
  }
  tL[0] = vc[0];
  tR[0] = vc[0];
  double beta[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int p = 0; p < M; ++p)
#pragma unroll
    for (int r = 0; r < M; ++r) {
      beta[0] += tL[p] * l.Bm[p][r] * tL[r];
      beta[1] += vc[p] * l.Bm[p][r] * vc[r];
      beta[2] += tR[p] * l.Bm[p][r] * tR[r];
    }
  double wbar[3], sum = 0.0;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const double d = l.eps + beta[s];
    wbar[s] = l.gam[s] / (d * d);
    sum += wbar[s];
  }
  const double isum = 1.0 / sum;
  const double om0 = wbar[0] * isum, om1 = wbar[1] * isum, om2 = wbar[2] * isum;
#pragma unroll
  for (int j = 0; j < M; ++j) vl[j] = om0 * tL[j] + om1 * vc[j] + om2 * tR[j];
}

// Characteristic WENO of the troubled element whose unlimited modes sit in lane cl of the wavefront's
// LDS area, by a group of 8 lanes: lane c < 5 limits characteristic field c (lanes 5..7 repeat field 4
// and contribute nothing); w_lim[v] = sum_c R[v][c] v_c^lim is summed across the group in a fixed
// butterfly order, after which every lane of the group holds it, and a lane with take >= 0 receives
// the result of group `take` in u.  Every lane of the wavefront takes part.  Returns false if the
// mean state has no valid characteristic decomposition.
template <int M>
__device__ __forceinline__ bool weno_group(const EulerArgs &a, const LimiterArgs &l, const NbSide (&sd)[2],
                                           const double *ls, int cl, int c, int take, double (&u)[5][M]) {
  double wb[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) wb[v] = ls[(v * M) * 64 + cl];
  double lr[5], rc[5];
  const bool ok = char_row_col(a.ph, wb, c < 5 ? c : 4, lr, rc);
  double vc[M], vL[M], vR[M];
#pragma unroll
  for (int j = 0; j < M; ++j) {
    vc[j] = 0.0; vL[j] = 0.0; vR[j] = 0.0;
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    double cl_[M], cr_[M];
    nb_var<M>(sd[0], v, ls, cl_);
    nb_var<M>(sd[1], v, ls, cr_);
#pragma unroll
    for (int j = 0; j < M; ++j) {
      vc[j] += lr[v] * ls[(v * M + j) * 64 + cl];
      vL[j] += lr[v] * cl_[j];
      vR[j] += lr[v] * cr_[j];
    }
    // one variable's reads at a time: keeps the kernel's register budget
    __builtin_amdgcn_sched_barrier(0);
  }
  double vl[M];
  weno_field<M>(l, vc, vL, vR, vl);
  const int from = take >= 0 ? 8 * take : 0;
#pragma unroll
  for (int v = 0; v < 5; ++v)
#pragma unroll
    for (int j = 0; j < M; ++j) {
      double part = c < 5 ? rc[v] * vl[j] : 0.0;
      part += dpp_move<kDppXor1>(part);
      part += dpp_move<kDppXor2>(part);
      part += dpp_move<kDppHalfMirror>(part);   // the same sum as from lane ^ 4
      const double got = __shfl(part, from);
      if (take >= 0) u[v][j] = got;
    }
  return ok;
}

// The order of a wavefront's LDS accesses: its lanes run in lockstep and the LDS serves a wavefront's
// accesses in order, so only the compiler has to keep them.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Source points of a round's elements in stage s (kSlotLanes elements, two slots each: slot 2r + side
// belongs to the r-th): a face that needs a slot (transmissive end or delayed PE interface) points at
// it, and a ghost's slot is filled with the element's own mean; AT slots are gathered beforehand.
template <int M>
__device__ __forceinline__ void point_slots(int s, NbSide (&sd)[2], int rank, double *ls, int lane) {
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    if (!sd[side].ghost && sd[side].k <= 0) continue;
    const int slot = s * kNbSlots + 2 * (rank % kSlotLanes) + side;
    double *sl = ls + 5 * M * 64 + slot * 5 * M;
    if (sd[side].ghost) {
#pragma unroll
      for (int v = 0; v < 5; ++v)
#pragma unroll
        for (int j = 0; j < M; ++j) sl[v * M + j] = j == 0 ? ls[(v * M) * 64 + lane] : 0.0;
    }
    sd[side].base = 5 * M * 64 + slot * 5 * M;
    sd[side].sv = M;
    sd[side].sj = 1;
  }
}

// The n-th lowest set bit of m (-1: none).
__device__ __forceinline__ int nth_bit(unsigned long long m, int n) {
  for (int j = 0; j < n && m; ++j) m &= m - 1;
  return m ? __ffsll((long long)m) - 1 : -1;
}

// The AT neighbours of a round's slots in the stages s0 .. s0 + NS - 1: the Eq. (11) combination of the
// unlimited boundary-element outputs that past levels published, gathered by all lanes of the
// wavefront at once, one lane per component with its q levels in flight together (two levels per
// component and round trip, one owner per element, took three times the registers).  nball: the lanes
// that need a slot, less the earlier rounds'.  Ghost slots are left to their owners.
template <int M, int NS>
__device__ __forceinline__ void gather_slots(const EulerArgs &a, int nmod, int s0, const NbSide (&sd)[2],
                                             unsigned long long nball, double *ls, int lane) {
  constexpr int C = 5 * M, T = NS * kNbSlots * C;
#pragma unroll 1
  for (int q0 = 0; q0 < T; q0 += 64) {
    const int pair = q0 + lane;
    const int ds = min(pair / (kNbSlots * C), NS - 1), sc = pair % (kNbSlots * C);
    const int sl = sc / C, comp = sc % C, side = sl & 1, s = s0 + ds;
    const int src = nth_bit(nball, sl >> 1);
    const int i0 = __shfl(sd[0].i, max(src, 0)), i1 = __shfl(sd[1].i, max(src, 0));
    const int k0 = __shfl(sd[0].k, max(src, 0)), k1 = __shfl(sd[1].k, max(src, 0));
    const int i = side ? i1 : i0, k = side ? k1 : k0;   // a ghost side has i = -1, k = 0
    if (pair < T && src >= 0 && i >= 0 && k > 0) {
      const int off = a.ring.off_U + (side == 0 ? 0 : C) + comp;
      const int mode = comp % M;
      const int qm = buffer_levels(a.dl, mode);   // levels this mode uses (q, or max(1, q - mode))
      double acc = 0.0;
      // levels past qm read level n-k (no further load) with weight 0
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool in = j < qm;
        const double w = in ? buffer_weight(a.dl, k, mode, j) : 0.0;
        acc += w * ring_at(a.ring, ring_slot(nmod, k + (in ? j : 0), a.ring.D), s, a.dl.nif, i)[off];
      }
      for (int j = 4; j < qm; ++j)
        acc += buffer_weight(a.dl, k, mode, j) *
               ring_at(a.ring, ring_slot(nmod, k + j, a.ring.D), s, a.dl.nif, i)[off];
      ls[5 * M * 64 + (s * kNbSlots + sl) * C + comp] = acc;
    }
  }
}

// ---------------------------------------------------------------- step kernel

// LDS doubles of a wavefront without the limiter: the AT fluxes of the lanes' faces for every stage.
template <int S>
constexpr int fat_wave_doubles() { return S * 5 * 64; }

// The AT fluxes of the first kSlotLanes delayed faces of a wavefront in every stage, one lane per
// component, each the same combination at_flux forms.  fball: the lanes whose right face is delayed.
template <int S>
__device__ __forceinline__ void gather_fluxes(const EulerArgs &a, int nmod, unsigned long long fball, int iface, int kf,
                                              double *fs, int lane) {
  constexpr int T = S * kSlotLanes * 5;
  static_assert(T <= 128, "two rounds");
#pragma unroll 1
  for (int q0 = 0; q0 < T; q0 += 64) {
    const int pair = q0 + lane;
    const int s = min(pair / (kSlotLanes * 5), S - 1), r = pair / 5 % kSlotLanes, v = pair % 5;
    const int src = nth_bit(fball, r);
    const int i = __shfl(iface, max(src, 0)), k = __shfl(kf, max(src, 0));
    if (pair < T && src >= 0) {
      const int q = a.dl.q;
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool in = j < q;
        const double c = in ? at_weight(q, k, j) : 0.0;
        acc += c * ring_at(a.ring, ring_slot(nmod, k + (in ? j : 0), a.ring.D), s, a.dl.nif, i)[a.ring.off_F + v];
      }
      for (int j = 4; j < q; ++j)
        acc += at_weight(q, k, j) * ring_at(a.ring, ring_slot(nmod, k + j, a.ring.D), s, a.dl.nif, i)[a.ring.off_F + v];
      fs[pair] = acc;
    }
  }
}

// Elements a wavefront owns: its lanes less a halo of one lane per stage on each side, two per stage
// with the limiter.
template <int S, bool LIM>
constexpr int owned_lanes() { return 64 - 2 * S * (LIM ? 2 : 1); }

// One whole time step (S stages).  Lane l of a wavefront holds element base + l - H (base = (64 - 2H) *
// wavefront index; H = S, 2S with the limiter): the lanes H .. 63-H own their element, the H lanes on
// each side hold neighbours.  A stage needs one neighbour on each side for the fluxes, and one more for
// the limiter, so stage s forms the outputs of the lanes w s + 1 .. 62 - w s (w = H / S), which is what
// the stages after it need: the state is read once and written once per step (16 B per scalar DOF,
// where one launch per stage moves 64 B for SSP-RK3) and a small problem pays one launch and one
// memory latency per step instead of S.  The halo lanes repeat their owners' arithmetic bit for bit (6
// of 64 lanes for SSP-RK3, 12 with the limiter).  Past levels' fluxes and boundary-element outputs are
// all that a delayed face reads from the ring, and those precede the step, so they are gathered for
// every stage at the start, beside the state loads, and kept in LDS.
//   Without the limiter, N_p = 2, against one launch per stage: 9.6 us per step against 21.7 at
// E = 512 (launch and latency bound), 0.27 ms against 0.78 at E = 2^22 in a steady run (was bound by HBM at
// 5.2 TB/s; now by the FP64 issue rate, 3.7 TB/s of the one read and one write).  Instructions decide both, so
// the Legendre values that are 0 or 1 are left out, the factors of dt L are folded into one per mode,
// and recip, root and exp_taylor stand for the general division, square root and exponential (0.33 ms
// and 11.1 us without that).
//   With it the wavefront stages its unlimited outputs in LDS, and the lanes w s + 2 .. 61 - w s run the
// indicator and, if troubled, the WENO reconstruction from them; their limited values return to
// registers.  No other wavefront's data is needed, so wavefronts never wait for each other.  Against one
// launch per stage: 25 us per step against 52 at E = 8192, N_p = 3 (latency bound), 147 against 240 at
// E = 10^6, N_p = 2 (HBM bound before; now by the VALU issue slots).  Registers decide the latter:
// with w^n held through the limiter 160 bytes per lane went to scratch, three times the step's own
// writes, and the step took 275 us.
template <int M, int FLUX, int S, bool LIM>
__device__ __forceinline__ void euler_step_body(const EulerArgs &a, const LimiterArgs &l, const double *win, double *wout,
                                                double *lds, int wave, long long n, int par) {
  constexpr int V = 5, Q = M, W = LIM ? 2 : 1, H = W * S, WE = owned_lanes<S, LIM>();
  constexpr int RK = S == 3 ? 0 : S == 2 ? 1 : 2;
  const int lane = threadIdx.x & 63;
  const int base = wave * WE;
  const int E = a.E;
  if (base < E) {
    const int xu = base + lane - H;                       // element index before periodic wrap
    const bool periodic = a.periodic != 0;
    // an element of the mesh, or its periodic image within the halo
    const bool inside = periodic ? xu <= E - 1 + H : (xu >= 0 && xu < E);
    const bool own = lane >= H && lane < 64 - H && xu < E;
    const bool ghost_l = !periodic && xu == -1;           // transmissive ends: ghost = interior trace
    const bool ghost_r = !periodic && xu == E;
    // face xu + 1, right of the lane's element
    const bool face_lane = lane <= 62 && (periodic ? xu + 1 <= E - 1 + H : (xu >= -1 && xu < E));
    int x = xu, fidx = xu + 1;
    if (periodic) {   // within a few periods of [0, E)
      while (x < 0) x += E;
      while (x >= E) x -= E;
      fidx = x + 1;   // face E is face 0
    }
    const int iface = face_lane ? a.face_if[fidx] : -1;
    const int nmod = step_mod(n, a.ring.D);
    double u[V][M], wn[V][M];
    if (inside) {
      load_elem<M>(win, E, x, u);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v)
#pragma unroll
        for (int j = 0; j < M; ++j) u[v][j] = 0.0;
    }
    // (the limiter kernel draws with the branch-free count, the other with the ordered search: measured)
    const int kf = iface >= 0 ? eff_delay<LIM>(a.dl, n, iface) : 0;
    const int if_left = LIM ? dpp_move<kDppFromPrev>(iface) : -1;
    double *ls = nullptr, *fat = nullptr;
    NbSide sd[2];
    unsigned long long nball = 0, fball = 0;
    int rank = 0, frank = 0;
    bool needs = false;
    if constexpr (LIM) {
      ls = lds;
      fat = ls + 5 * M * 64 + S * kNbSlots * 5 * M;
      // the neighbours of a limited element across a transmissive end or a delayed PE interface need
      // a slot: kSlotLanes such elements per round, two slots each
      const bool limits = lane >= 2 && lane <= 61 && (periodic ? xu <= E + H - 3 : inside);
      const int k_left = dpp_move<kDppFromPrev>(kf);
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        const bool ghost = limits && !periodic && (side == 0 ? x == 0 : x == E - 1);
        const int i = (limits && !ghost) ? (side == 0 ? if_left : iface) : -1;
        const int k = i >= 0 ? (side == 0 ? k_left : kf) : 0;
        sd[side].i = i;
        sd[side].k = k;
        sd[side].ghost = ghost;
        needs = needs || ghost || k > 0;
      }
      nball = __ballot(needs);
      fball = __ballot(kf > 0);
      const unsigned long long below = (1ull << lane) - 1ull;
      rank = __popcll(nball & below);
      frank = __popcll(fball & below);
      if (fball) gather_fluxes<S>(a, nmod, fball, iface, kf, fat, lane);
      if (fball) gather_slots<M, S>(a, nmod, 0, sd, nball, ls, lane);
      wave_lds_fence();
    } else {
      fat = lds + lane;
      if (kf > 0) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
          double F[V];
          at_flux(a, nmod, s, iface, kf, F);
#pragma unroll
          for (int v = 0; v < V; ++v) fat[(s * V + v) * 64] = F[v];
        }
      }
    }
    // the second operand of the RK combination: w^n, or the 2N register.  With the limiter w^n is read
    // again (from L2) in each stage that uses it, so that it takes no registers during the limiter.
    constexpr bool kReload = LIM && RK == 0;
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (int j = 0; j < M; ++j) wn[v][j] = RK == 0 && !kReload ? u[v][j] : 0.0;
    bool ok = true;
#pragma unroll 1
    for (int s = 0; s < S; ++s) {
      const RkStage rk = rk_stage(RK, s);
      const double ca = rk.ca, cb = rk.cb;
      // the lanes whose output a later stage or the store needs
      const bool calc = lane > W * s && lane < 63 - W * s && (periodic ? xu <= E + H - 2 - W * s : inside);
      double wl[V], wr[V], F[V], Fl[V];
      traces<M>(u, wl, wr);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const double next_l = dpp_move<kDppFromNext>(wl[v]);
        const double prev_r = dpp_move<kDppFromPrev>(wr[v]);
        if (ghost_l) wr[v] = next_l;
        if (ghost_r) wl[v] = prev_r;
      }
      double wp[V];
#pragma unroll
      for (int v = 0; v < V; ++v) wp[v] = dpp_move<kDppFromNext>(wl[v]);
      const bool fok = numflux1<FLUX>(a.ph, wr, wp, F);
      // faces that an owned element has
      if (face_lane && lane >= H - 1 && lane < 64 - H && xu < E) ok = fok && ok;
      if (iface >= 0) {
        if (own) {   // the face's owner publishes the synchronous flux of this level
          double *rec = ring_at(a.ring, nmod, s, a.dl.nif, iface) + a.ring.off_F;
#pragma unroll
          for (int v = 0; v < V; ++v) rec[v] = F[v];
        }
        if (kf > 0) {
          if constexpr (LIM) {
            if (frank < kSlotLanes) {
#pragma unroll
              for (int v = 0; v < V; ++v) F[v] = fat[(s * kSlotLanes + frank) * 5 + v];
            } else {
              at_flux(a, nmod, s, iface, kf, F);
            }
          } else {
#pragma unroll
            for (int v = 0; v < V; ++v) F[v] = fat[(s * V + v) * 64];
          }
        }
      }
#pragma unroll
      for (int v = 0; v < V; ++v) Fl[v] = dpp_move<kDppFromPrev>(F[v]);
      if (calc) {
        // b_j = sum_q w_q P_j'(xi_q) f_q - F_{e+1} P_j(1) + F_e P_j(-1); the face terms go in first
        double vol[V][M], srcR[M];
#pragma unroll
        for (int j = 0; j < M; ++j) {
          srcR[j] = 0.0;
#pragma unroll
          for (int v = 0; v < V; ++v) vol[v][j] = -F[v] + ((j & 1) ? -Fl[v] : Fl[v]);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          double wq[V];
#pragma unroll
          for (int v = 0; v < V; ++v) {
            double acc = u[v][0];   // P_0 = 1
#pragma unroll
            for (int j = 1; j < M; ++j) acc += u[v][j] * a.tb.B[q][j];
            wq[v] = acc;
          }
          Prim1 pr;
          ok = prim1(a.ph, wq, pr) && ok;
          double f[V];
          flux1(wq, pr, f);
          // (the exponent held to where exp is 0 or infinite in FP64)
          const double rate = a.ph.k_pre * wq[3] * exp_taylor(fmin(fmax(-a.ph.e_act * (pr.rho * recip(pr.p)), -800.0), 800.0));
#pragma unroll
          for (int j = 0; j < M; ++j) {
            if (j > 0) {   // P_0' = 0
              const double g = a.tb.WG[q][j];
#pragma unroll
              for (int v = 0; v < V; ++v) vol[v][j] += g * f[v];
            }
            srcR[j] -= a.tb.WB[q][j] * rate;
          }
        }
        double wr_[V][M];
        double (&wk)[V][M] = kReload ? wr_ : wn;
        if constexpr (kReload) {
          // an opaque index: the compiler would otherwise keep every component's address across the loop
          int xr = x;
          asm volatile("" : "+v"(xr));
          load_elem<M>(win, E, xr, wk);
        }
#pragma unroll
        for (int j = 0; j < M; ++j) {
          const double cb_j = a.dt_dx * (2 * j + 1), src = a.dt_2 * (2 * j + 1) * srcR[j];
#pragma unroll
          for (int v = 0; v < V; ++v) {
            // explicit fused multiply-adds: every kernel that runs this combination rounds alike.  In
            // the first stage ca is 0 (and cb 1, or the 2N register 0)
            if constexpr (RK == 0) {
              double y = fma(cb_j, vol[v][j], u[v][j]);
              if (v == 3) y += src;
              if (v == 4) y -= src;
              u[v][j] = fma(ca, wk[v][j], cb * y);
            } else {
              double dl = cb_j * vol[v][j];
              if (v == 3) dl += src;
              if (v == 4) dl -= src;
              wn[v][j] = fma(ca, wn[v][j], dl);
              u[v][j] = fma(cb, wn[v][j], u[v][j]);
            }
            if constexpr (LIM) ls[(v * M + j) * 64 + lane] = u[v][j];
          }
        }
        if constexpr (LIM) {
          if (own && a.store_U) {   // boundary-element outputs of this level, on both sides of an interface
            if (if_left >= 0) {
              double *rec = ring_at(a.ring, nmod, s, a.dl.nif, if_left) + a.ring.off_U + V * M;
#pragma unroll
              for (int c = 0; c < V * M; ++c) rec[c] = u[c / M][c % M];
            }
            if (iface >= 0) {
              double *rec = ring_at(a.ring, nmod, s, a.dl.nif, iface) + a.ring.off_U;
#pragma unroll
              for (int c = 0; c < V * M; ++c) rec[c] = u[c / M][c % M];
            }
          }
        }
      }
      if constexpr (LIM) {
        const bool limits = lane >= W * s + 2 && lane <= 61 - W * s && (periodic ? xu <= E + H - 3 - W * s : inside);
        const int my_round = needs ? rank / kSlotLanes : 0;
        const int nrounds = max(1, (__popcll(nball) + kSlotLanes - 1) / kSlotLanes);
#pragma unroll
        for (int side = 0; side < 2; ++side) {
          sd[side].base = lane + (side == 0 ? -1 : 1);
          sd[side].sv = M * 64;
          sd[side].sj = 64;
        }
        bool flagged = false;
        unsigned long long left = nball;
#pragma unroll 1
        for (int round = 0; round < nrounds; ++round) {
          wave_lds_fence();   // the outputs are in LDS; the previous round's slots have been read
          // (the first round's AT slots were gathered at the start)
          if (round > 0) gather_slots<M, 1>(a, nmod, s, sd, left, ls, lane);
          if (limits && needs && my_round == round) point_slots<M>(s, sd, rank, ls, lane);
          for (int g = 0; g < kSlotLanes && left; ++g) left &= left - 1;
          wave_lds_fence();   // the slots are read by other lanes of the wavefront below
          bool flag = false;
          if (limits && my_round == round) flag = troubled<M>(a, l, sd, ls, lane);
          flagged = flagged || flag;
          // troubled elements: eight at a time, one group of 8 lanes each (group g takes the
          // g-th lowest remaining troubled lane)
          unsigned long long rem = __ballot(flag);
          const int grp = lane >> 3, cf = lane & 7;
#pragma unroll 1
          while (rem) {
            const int cl = nth_bit(rem, grp);
            const int mine = (rem >> lane) & 1 ? __popcll(rem & ((1ull << lane) - 1ull)) : 8;
            for (int g = 0; g < 8 && rem; ++g) rem &= rem - 1;
            const int src = max(cl, 0);
            NbSide sc[2];
#pragma unroll
            for (int side = 0; side < 2; ++side) {
              sc[side].base = __shfl(sd[side].base, src);
              sc[side].sv = __shfl(sd[side].sv, src);
              sc[side].sj = __shfl(sd[side].sj, src);
            }
            const bool wok = weno_group<M>(a, l, sc, ls, src, cf, mine < 8 ? mine : -1, u);
            if (cl >= 0) ok = wok && ok;
          }
        }
        if (own && flagged) atomicAdd(l.flag_count, 1ull);
        if (own && s == S - 1) l.flags[x] = flagged ? 1 : 0;
        wave_lds_fence();   // the outputs have been read
      }
    }
    if (own) {
      double *dst = wout + sidx(x, 0, V * M);
#pragma unroll
      for (int v = 0; v < V; ++v)
#pragma unroll
        for (int j = 0; j < M; ++j) dst[(v * M + j) * kLayoutBlock] = u[v][j];
    }
    if (!ok) atomicOr(a.err, (int)kErrState);
  }
  advance_step(a.step, par, n, wave == 0);
}

// Wavefronts per workgroup (they share nothing): four without the limiter, one with it, whose LDS
// then packs a CU in steps of one wavefront.
template <bool LIM>
constexpr int kEulerWaves = LIM ? 1 : 4;
// Wavefronts per SIMD that the registers are held to.  Without a bound N_p = 4 takes 262 registers, one
// wavefront: 216 us per step at E = 2^20, 158 with two (15.6 and 16.0 at E = 4000, where there is one).
// With the limiter the 2N schemes hold a register beside the state and spill for it (104 bytes a lane at
// N_p = 2, 160 at N_p = 4); per step against one launch per stage, HLLC and KXRCF: RK2 at E = 500 000
// 62.8 us against 96.0 (N_p = 2) and 116 against 224 (N_p = 4), LSERK4 146 against 248 and 281 against 582;
// at E = 8192 19.9 against 30.8 (RK2, N_p = 2) and 66.5 against 137 (LSERK4, N_p = 4).
template <int M, bool LIM>
constexpr int kEulerMinWaves = LIM ? (M <= 3 ? 3 : 2) : M == 5 ? 2 : 1;
template <int M, int S, bool LIM>
constexpr int euler_wave_lds() { return LIM ? lds_wave_doubles<M, S>() : fat_wave_doubles<S>(); }

template <int M, int FLUX, int S>
__global__ __launch_bounds__(64 * kEulerWaves<false>, (kEulerMinWaves<M, false>)) void euler_step_kernel(EulerArgs a) {
  __shared__ double lds[kEulerWaves<false> * euler_wave_lds<M, S, false>()];
  const int w = threadIdx.x >> 6;
  euler_step_body<M, FLUX, S, false>(a, LimiterArgs{}, a.ws, a.wout, lds + w * euler_wave_lds<M, S, false>(),
                                     xcd_item(blockIdx.x, gridDim.x) * kEulerWaves<false> + w, a.step[a.par], a.par);
}

template <int M, int FLUX, int S>
__global__ __launch_bounds__(64 * kEulerWaves<true>, (kEulerMinWaves<M, true>)) void euler_lim_step_kernel(EulerArgs a, LimiterArgs l) {
  __shared__ double lds[kEulerWaves<true> * euler_wave_lds<M, S, true>()];
  const int w = threadIdx.x >> 6;
  euler_step_body<M, FLUX, S, true>(a, l, a.ws, a.wout, lds + w * euler_wave_lds<M, S, true>(),
                                    xcd_item(blockIdx.x, gridDim.x) * kEulerWaves<true> + w, a.step[a.par], a.par);
}

// Batched step: one workgroup per (instance, block) entry of the work list, for instances of one
// order, flux and limiter choice, all at step counter parity par; an instance whose step count has
// reached its target is skipped by all of its workgroups alike (its first one carries the count over
// to the other parity).  w^n of a step lives in W[n mod 2].  Batches run SSP-RK3.
template <int M, int FLUX, bool LIM>
__global__ __launch_bounds__(64 * kEulerWaves<LIM>, (kEulerMinWaves<M, LIM>)) void euler_batch_kernel(
    const EulerSet *__restrict__ sets, const int2 *__restrict__ tiles, int par) {
  __shared__ double lds[kEulerWaves<LIM> * euler_wave_lds<M, 3, LIM>()];
  const int2 tl = tiles[blockIdx.x];
  const EulerArgs &a = sets[tl.x].st;
  const long long n = a.step[par];
  if (n >= a.target) {
    if (tl.y == 0 && threadIdx.x == 0) a.step[par ^ 1] = n;
    return;
  }
  const int c = (int)(n & 1), w = threadIdx.x >> 6;
  euler_step_body<M, FLUX, 3, LIM>(a, sets[tl.x].lim, a.W[c], a.W[1 - c], lds + w * euler_wave_lds<M, 3, LIM>(),
                                   tl.y * kEulerWaves<LIM> + w, n, par);
}

// ---------------------------------------------------------------- launchers

int euler_blocks(int E, int stages, bool lim) {
  const int we = 64 - 2 * stages * (lim ? 2 : 1), waves = lim ? kEulerWaves<true> : kEulerWaves<false>;
  return ((E + we - 1) / we + waves - 1) / waves;
}

template <int M, int FLUX, int S>
static void step_MFS(const EulerArgs &a, const LimiterArgs *lim, hipStream_t s) {
  const dim3 grid(euler_blocks(a.E, S, lim != nullptr));
  if (lim) hipLaunchKernelGGL((euler_lim_step_kernel<M, FLUX, S>), grid, dim3(64 * kEulerWaves<true>), 0, s, a, *lim);
  else hipLaunchKernelGGL((euler_step_kernel<M, FLUX, S>), grid, dim3(64 * kEulerWaves<false>), 0, s, a);
}

template <int M, int FLUX>
static hipError_t step_MF(int stages, const EulerArgs &a, const LimiterArgs *lim, hipStream_t s) {
  if (stages == 3) step_MFS<M, FLUX, 3>(a, lim, s);
  else if (stages == 2) step_MFS<M, FLUX, 2>(a, lim, s);
  else if (stages == 5) step_MFS<M, FLUX, 5>(a, lim, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int M>
static hipError_t step_M(int flux, int stages, const EulerArgs &a, const LimiterArgs *lim, hipStream_t s) {
  return flux == 1 ? step_MF<M, 1>(stages, a, lim, s) : step_MF<M, 0>(stages, a, lim, s);
}

hipError_t launch_euler_step(int M, int flux, int stages, const EulerArgs &a, const LimiterArgs *lim, hipStream_t s) {
  switch (M) {
    case 2: return step_M<2>(flux, stages, a, lim, s);
    case 3: return step_M<3>(flux, stages, a, lim, s);
    case 4: return step_M<4>(flux, stages, a, lim, s);
    case 5: return step_M<5>(flux, stages, a, lim, s);
  }
  return hipErrorInvalidValue;
}

template <int M, int FLUX>
static hipError_t batch_MF(bool lim, const EulerSet *sets, const int2 *tiles, int ntiles, int par, hipStream_t s) {
  if (lim)
    hipLaunchKernelGGL((euler_batch_kernel<M, FLUX, true>), dim3(ntiles), dim3(64 * kEulerWaves<true>), 0, s, sets, tiles, par);
  else
    hipLaunchKernelGGL((euler_batch_kernel<M, FLUX, false>), dim3(ntiles), dim3(64 * kEulerWaves<false>), 0, s, sets, tiles, par);
  return hipGetLastError();
}

template <int M>
static hipError_t batch_M(int flux, bool lim, const EulerSet *sets, const int2 *tiles, int ntiles, int par, hipStream_t s) {
  return flux == 1 ? batch_MF<M, 1>(lim, sets, tiles, ntiles, par, s) : batch_MF<M, 0>(lim, sets, tiles, ntiles, par, s);
}

hipError_t launch_euler_batch(int M, int flux, bool lim, const EulerSet *sets, const int2 *tiles, int ntiles, int par,
                              hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  switch (M) {
    case 2: return batch_M<2>(flux, lim, sets, tiles, ntiles, par, s);
    case 3: return batch_M<3>(flux, lim, sets, tiles, ntiles, par, s);
    case 4: return batch_M<4>(flux, lim, sets, tiles, ntiles, par, s);
    case 5: return batch_M<5>(flux, lim, sets, tiles, ntiles, par, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace adg

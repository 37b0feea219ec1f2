// Detailed-chemistry Navier-Stokes stage with one lane per point (quadrature node or face trace):
// the form of the stage for sizes that fill the device, and for batches.  adg_ns.hip holds the form
// that spreads a point's species and reactions over lanes, for problems of about one tile per CU.
//
// A tile of TE elements takes one workgroup of NW wavefronts: lanes [0, TE Q) hold the nodes, the
// next 2 (TE + 1) the two traces of every tile face, the last four the traces that complete the
// central traces of the faces beyond (the gradients of the two halo elements need them).  Every lane
// reads its element's modes (the lanes of an element read the same addresses) and keeps its point's
// values and the volume part of its gradient in registers; only traces, face data and the nodal
// results of the volume integral pass through LDS.  Each species and reaction index is then the same
// in all lanes: the mechanism is read by scalar loads and enters the FP64 instructions as scalar
// operands, with no table in LDS and no index arithmetic per lane, and the species production is
// summed in registers.
//
// The stage is bound by the VALU issue rate (66 % of a stage of 4096 instances) and, at five tiles a CU, by
// the latency of the phases between its barriers; with few tiles, by that of one tile alone.  With the
// reactions and species spread over lanes a node took about 150 wavefront instructions, 27 % of them FP64
// arithmetic; here it takes 58, 62 % of them FP64.  Measured per stage (9 species, N_p = 3): E = 2^18 374 us
// in the best spread form, 149 here; E = 2^16 99 and 48; 1024 instances of 128..4096 elements, N_p = 2 and
// 3, 1713 and 565; but one instance of 200 elements 11.6 and 16.9.  The tile of three wavefronts beat a
// tile of one (no barriers, but a third of its lanes idle in the chemistry: 178 at E = 2^18).
#include "adg_ns_device.hpp"

namespace adg {

// Forms the values here: left to itself the compiler moves the arithmetic past the barriers to its
// uses and keeps all of its operands (four times the registers) alive until then.
template <int N>
__device__ __forceinline__ void pin(double (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
}

// exp_taylor of N arguments (of a size below 2^31), their dependent chains side by side.
template <int N>
__device__ __forceinline__ void exp_taylor_n(double (&x)[N]) {
  double k[N], r[N], p[N];
#pragma unroll
  for (int d = 0; d < N; ++d) k[d] = __builtin_rint(x[d] * kInvLn2);
#pragma unroll
  for (int d = 0; d < N; ++d) r[d] = fma(k[d], -kLn2Hi, x[d]);
#pragma unroll
  for (int d = 0; d < N; ++d) r[d] = fma(k[d], -kLn2Lo, r[d]);
  const double c[13] = {1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0, 1.0 / 362880.0, 1.0 / 40320.0,
                        1.0 / 5040.0, 1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.5, 1.0, 1.0};
#pragma unroll
  for (int d = 0; d < N; ++d) p[d] = 1.0 / 6227020800.0;
#pragma unroll
  for (int i = 0; i < 13; ++i)
#pragma unroll
    for (int d = 0; d < N; ++d) p[d] = fma(p[d], r[d], c[i]);
#pragma unroll
  for (int d = 0; d < N; ++d) x[d] = __builtin_amdgcn_ldexp(p[d], (int)k[d]);
}

// Bound of the exponents whose products (two factors and their reciprocals) stay in range.
constexpr double kMaxExponent = 250.0;

// Geometry of a tile of TE elements.
template <int M, int NS, int TE>
struct LaneTile {
  static constexpr int V = 3 + NS, Q = M;
  static constexpr int NF = TE + 3;                 // faces e0-1 .. e0+TE+1; local fl <-> face e0 - 1 + fl
  static constexpr int NN = TE * Q;                 // nodes; node p <-> element p / Q, node p % Q
  static constexpr int T0 = NN + (NN & 1);          // first trace lane: a face's two traces are lanes 2m, 2m + 1
  static constexpr int NP = T0 + 2 * (TE + 1);      // end of the traces of the faces e0 .. e0+TE
  static constexpr int NL = NP + 4;                 // end of the outer traces
  static constexpr int NW = (NL + 63) / 64, NTH = 64 * NW;
  static constexpr int NCW = (NN + 63) / 64;        // wavefronts that hold nodes
  static constexpr int NI = (V * TE + NTH - 1) / NTH;   // (variable, element) items of a lane in the last phase
};

// LDS of one tile.
template <int M, int NS, int TE>
struct LaneLds {
  using G = LaneTile<M, NS, TE>;
  static constexpr int V = G::V;
  double F[V][TE + 1];            // face fluxes
  union {
    // until the gradients are formed: traces of the faces e0-1 .. e0+TE+1, left (of the element left
    // of the face) and right; at a delayed PE interface, the AT central trace less the synchronous one
    struct {
      double tl[V][G::NF], tr[V][G::NF], dw[V][G::NF];
    } f;
    // then, per wavefront of nodes: the species' rate factors, and after them the fluxes and sources
    // at the nodes (each wavefront overwrites its own block only, after its own last read)
    union {
      struct {
        double z[NS + 1][64], ib[NS + 1][64];
      } c;
      double gs[V + NS][64];
    } nd[G::NCW];
  };
};

// The tile's faces: interface index (or -1) and effective delay; and the n faces that are interfaces.
template <int NF>
struct LanePe {
  int i[NF], k[NF], f[NF], n;
};

// AT combination (Eq. (7)) of the central trace and the flux of variable v at interface i from the
// levels n-k .. n-k-q+1: levels 0..3 loaded together (a level past q reads level n-k, weight 0).
__device__ __forceinline__ void at_levels(const NsArgs &a, int q, int k, int nm, int stage, int i, int v, double &w,
                                          double &f) {
  double hw[4], hf[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double *rec = ring_at(a.ring, ring_slot(nm, k + (j < q ? j : 0), a.ring.D), stage, a.dl.nif, i);
    hw[j] = rec[a.ring.off_Wc + v];
    hf[j] = rec[a.ring.off_F + v];
  }
  w = f = 0.0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double c = j < q ? at_weight(q, k, j) : 0.0;
    w += c * hw[j];
    f += c * hf[j];
  }
#pragma unroll 1
  for (int j = 4; j < q; ++j) {
    const double c = at_weight(q, k, j);
    const double *rec = ring_at(a.ring, ring_slot(nm, k + j, a.ring.D), stage, a.dl.nif, i);
    w += c * rec[a.ring.off_Wc + v];
    f += c * rec[a.ring.off_F + v];
  }
}

template <int M, int NS, int TE>
__device__ __forceinline__ void ns_lane_tile(const NsArgs &a, const double *__restrict__ ws, const double *prev,
                                             double *wout, int stage, int advance, const RkStage rk, double *kbuf,
                                             int e0, long long n, int par, LaneLds<M, NS, TE> &L,
                                             LanePe<TE + 3> &P) {
  using G = LaneTile<M, NS, TE>;
  constexpr int V = G::V, Q = M, NF = G::NF, NN = G::NN, T0 = G::T0, NP = G::NP, NTH = G::NTH, NI = G::NI;
  // constant address space: uniform reads become scalar loads whatever is stored in between
  const auto *mk = (const __attribute__((address_space(4))) NsMechT<NS> *)(uintptr_t)a.mech;
  constexpr int kLines = (int)((sizeof mk->sp + 24 * sizeof mk->rx[0]) / 64), kPre = (kLines + G::NW - 1) / G::NW;
  const int t = threadIdx.x;
  const int E = a.E, Vg = 3 + a.ns, VMg = Vg * M;
  const int nloc = min(TE, E - e0);
  const bool periodic = a.periodic != 0;
  const int nm = step_mod(n, a.ring.D);   // the current level's ring slot
  const int q_at = a.dl.q;

  // interface map of the tile's faces (the first wavefront holds them all)
  static_assert(NF <= 64, "the faces of a tile sit in one wavefront");
  int fi = -1;
  if (t < NF) {
    int f = e0 - 1 + t;
    if (periodic) f = wrap(f, E, TE + 4);
    if (f >= 0 && f <= E) fi = a.face_if[f];
  }

  // the lane's point: element el (relative to e0) and row r of the point tables (nodes r < Q, then
  // xi = +1, xi = -1); a trace lane belongs to face fl
  const bool node = t < NN, trace = t >= T0 && t < NP;
  int el, r, fl = 0, side = 0;
  if (node) {
    el = t / Q;
    r = t % Q;
  } else {
    // the faces fl = 1, 2, ..., then the outer faces fl = 0 and fl = TE + 2
    const int pp = min(max(t - T0, 0), 2 * (TE + 1) + 3);
    fl = pp < 2 * (TE + 1) ? (pp >> 1) + 1 : pp < 2 * (TE + 1) + 2 ? 0 : TE + 2;
    side = pp & 1;
    el = fl - 2 + side;
    r = Q + side;
  }
  bool valid = node || trace;
  int x = e0 + el;
  if (periodic) {
    x = wrap(x, E, TE + 4);
  } else {
    // at a transmissive end the ghost side of the face is evaluated at the interior element's trace;
    // points past it repeat the end element and are not used
    valid = valid && (node ? x < E : e0 + fl - 1 <= E);
    if (x < 0) { x = 0; el = -e0; r = Q + 1; }
    else if (x >= E) { x = E - 1; el = E - 1 - e0; r = Q; }
  }

  // The mechanism's records into the scalar cache: a wavefront of a small launch would miss on each in turn
  // (16 species, E = 2^16, N_p = 3: 100 -> 86 us a stage).  The loads go out before those of the modes, in
  // whose shadow they return; issued after them, the wait took 3800 of a tile's 41000 cycles, and the batched
  // kernel kept 24 bytes of scratch per lane (up to 150 tiles 55 -> 51.5 us a step, E = 2^18 153 -> 149 a
  // stage, 1024 instances 602 -> 565; a stage of 4096 instances 5.9 -> 4.9 GB of HBM traffic).
  int pre[kPre];
  {
    const auto *line = (const __attribute__((address_space(4))) int *)(uintptr_t)&static_cast<const NsMechT<NS> *>(a.mech)->sp[0];
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
#pragma unroll
    for (int i = 0; i < kPre; ++i) pre[i] = line[min(w + i * G::NW, kLines - 1) * 16];
    __builtin_amdgcn_sched_barrier(0);
  }

  // values at the point and the volume part of the gradient there, from the element's modes
  double X[V], D[V];
  {
    double bq[M], gd[M];
#pragma unroll
    for (int j = 0; j < M; ++j) {
      bq[j] = r < Q ? a.tb.B[min(r, Q - 1)][j] : (r == Q || !(j & 1)) ? 1.0 : -1.0;
      gd[j] = a.tb.GD[r][j];
    }
    const double *we = ws + sidx(x, 0, VMg);
    // all loads in flight at once: no branch per variable.  Padded species (past Vg) read variable
    // 0 again and are set to zero.
    auto values = [&](auto stored) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        double w[M];
#pragma unroll
        for (int j = 0; j < M; ++j) w[j] = we[(stored(v) * M + j) * kLayoutBlock];
        X[v] = bq[0] * w[0];
        D[v] = gd[0] * w[0];
#pragma unroll
        for (int j = 1; j < M; ++j) {
          X[v] = fma(bq[j], w[j], X[v]);
          D[v] = fma(gd[j], w[j], D[v]);
        }
      }
    };
    if (Vg == V) {
      values([](int v) { return v; });
    } else {
      values([&](int v) { return v < Vg ? v : 0; });
#pragma unroll
      for (int v = 4; v < V; ++v)
        if (v >= Vg) X[v] = D[v] = 0.0;
    }
    pin(X);
    pin(D);
#pragma unroll
    for (int i = 1; i < kPre; ++i) pre[0] ^= pre[i];
    asm volatile("" ::"s"(pre[0]));
  }
  if (t >= T0 && t < G::NL) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if (side == 0) L.f.tl[v][fl] = X[v];
      else L.f.tr[v][fl] = X[v];
    }
  }
  int kf = 0;
  if (t < 64) {
    kf = fi >= 0 ? eff_delay<true>(a.dl, n, fi) : 0;
    const unsigned long long pe_mask = __ballot(fi >= 0);
    if (t < NF) {
      P.i[t] = fi;
      P.k[t] = kf;
      if (fi >= 0) P.f[__popcll(pe_mask & ((1ull << t) - 1ull))] = t;
    }
    if (t == 0) P.n = __popcll(pe_mask);
  }
  __syncthreads();

  // gradients at the points, from the synchronous central traces
  const double ga = a.tb.GA[r], gb = a.tb.GB[r];
  const int fL = min(max(el + 1, 0), NF - 2);   // left face of the point's element (clamped: outer traces)
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const double wl = 0.5 * (L.f.tl[v][fL] + L.f.tr[v][fL]), wr = 0.5 * (L.f.tl[v][fL + 1] + L.f.tr[v][fL + 1]);
    D[v] = a.inv_dx * (ga * wr - gb * wl - D[v]);
  }
  pin(D);
  const int iface = trace ? P.i[fl] : -1;
  const int npe = __builtin_amdgcn_readfirstlane(P.n);
  if (npe) {
    // one lane per (interface, variable): the synchronous central trace of an owned interface is
    // published for this level; the AT combinations (Eq. (7)) of a delayed one's central trace and flux
    // are formed together, the flux goes to its place and the central trace corrects the gradients of the
    // two elements, but for the interface's own traces: their flux is the synchronous one, published.
    // Every wavefront takes pairs: with the first one alone, 9000 elements with a PE interface at every face
    // took 108 us a step at N_p = 2 and 142 with q = 6 levels, against 69 and 83 (tiles spread over lanes: 81
    // and 95); one face in 16, 63.7 and 60.2.
    for (int p = t; p < npe * V; p += NTH) {
      const int g = P.f[p / V], v = p % V, i = P.i[g], k = P.k[g];
      if (v < Vg) {
        const double wc = 0.5 * (L.f.tl[v][g] + L.f.tr[v][g]);
        if (g >= 1 && g <= nloc) ring_at(a.ring, nm, stage, a.dl.nif, i)[a.ring.off_Wc + v] = wc;
        if (k > 0) {
          double aw, af;
          at_levels(a, q_at, k, nm, stage, i, v, aw, af);
          if (g >= 1 && g <= TE + 1) L.F[v][g - 1] = af;
          L.f.dw[v][g] = aw - wc;
        }
      }
    }
    __syncthreads();
    if (iface < 0) {
      if (P.k[fL] > 0) {
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (v < Vg) D[v] -= a.inv_dx * gb * L.f.dw[v][fL];
      }
      if (P.k[fL + 1] > 0) {
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (v < Vg) D[v] += a.inv_dx * ga * L.f.dw[v][fL + 1];
      }
    }
  }
  // the second operand of the RK combination of this lane's (variable, element) items of the last
  // phase (w^n or the 2N register, from HBM): in flight during the point physics and the chemistry
  const bool use_prev = rk.two_n ? rk.ca != 0.0 : rk.ca != 0.0 || rk.cb != 1.0;
  auto item = [&](int m, int &v, int &e) -> size_t {
    const int idx = t + m * NTH;
    v = idx / TE;
    e = idx % TE;
    const bool in = idx < V * TE && e < nloc && v < Vg;
    if (!in) v = V;
    return in ? sidx(e0 + e, v * M, VMg) : sidx(e0, 0, VMg);
  };
  double pi[NI][M];
#pragma unroll
  for (int m = 0; m < NI; ++m)
#pragma unroll
    for (int j = 0; j < M; ++j) pi[m][j] = 0.0;
  if (use_prev) {
#pragma unroll
    for (int m = 0; m < NI; ++m) {
      int v, e;
      const double *src = prev + item(m, v, e);
#pragma unroll
      for (int j = 0; j < M; ++j) pi[m][j] = src[j * kLayoutBlock];
    }
  }
  __syncthreads();   // the face data has been read: its LDS is used again below

  // point physics
  bool ok = true;
  double lnT, invT;
  int fast;
  const int wv = min(t >> 6, G::NCW - 1), ln = t & 63;
  auto &nd = L.nd[wv];
  {
    const double rho = X[0], rho_inv = 1.0 / rho, u = X[1] * rho_inv, En = X[2] * rho_inv;
    const double estar = En - 0.5 * u * u;
    double c[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) c[q] = 0.0;
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int q = 0; q < 7; ++q) c[q] = fma(X[3 + i], mk->ek[i][q], c[q]);
    const double c6[6] = {c[0] * rho_inv, c[1] * rho_inv, c[2] * rho_inv, c[3] * rho_inv, c[4] * rho_inv, c[5] * rho_inv};
    const double Rmix = c[6] * rho_inv;
    double T, cv;
    const bool conv = newton_T(c6, mk->T_guess, estar, T, cv);
    lnT = log(T);
    invT = 1.0 / T;
    const double cp = cv + Rmix, p = rho * Rmix * T, rcv = 1.0 / cv;
    if (valid) ok = conv && p > 0.0 && isfinite(p) && rho > 0.0;
    double g1 = X[1] * u + p, g2 = u * (X[2] + p);
    double rhoD = 0.0, kc = 0.0;
    if (a.viscous) {
      // f^d of Eq. (2)-(3): tau = 4/3 mu u_x, heat flux -kappa T_x + sum_i h_i J_i with
      // T_x = (e_x - sum_i e_i dY_i/dx)/c_v, J_i = -rho D dY_i/dx (unit Lewis number, rho D = mu/Pr)
      const double mu = mk->mu_ref * exp_taylor(mk->mu_exp * (lnT - mk->ln_T_ref));
      rhoD = mu * mk->inv_prandtl;
      kc = rhoD * cp * rcv;
      const double u_x = (D[1] - u * D[0]) * rho_inv;
      const double e_x = (D[2] - En * D[0]) * rho_inv - u * u_x;
      const double tau = (4.0 / 3.0) * mu * u_x;
      g1 -= tau;
      g2 -= tau * u + kc * e_x;
    }
    // species: diffusive and enthalpy fluxes, and at the nodes the rate factors
    const double lnc0 = mk->ln_p_over_Ru - lnT;   // ln(p_ref / (Ru T))
    const double d0 = D[0] * rho_inv;
    double sum_eY = 0.0, sum_hY = 0.0, big = 0.0;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const auto &sp = mk->sp[i];
      const double y = X[3 + i];
      const double hR = fma(T, fma(T, fma(T, fma(T, fma(T, sp.h2[3], sp.h2[2]), sp.h2[1]), sp.h2[0]), sp.a0), sp.a5);
      double gy = y * u;
      if (a.viscous) {
        const double Yx = (D[3 + i] - y * d0) * rho_inv;
        const double RY = sp.Ri * Yx;
        sum_eY = fma(hR - T, RY, sum_eY);
        sum_hY = fma(hR, RY, sum_hY);
        gy = fma(-rhoD, Yx, gy);
      }
      D[3 + i] = gy;
      if (node) {
        const double sR = fma(sp.a0, lnT, fma(T, fma(T, fma(T, fma(T, sp.s2[2], sp.s2[1]), sp.s2[0]), sp.a1), sp.a6));
        // arg = -g_i/(Ru T) + ln(p_ref/(Ru T)); exp(arg) is the reciprocal of the species' factor in K_c
        const double arg = fma(-hR, invT, sR) + lnc0;
        big = fabs(arg) <= kMaxExponent ? big : 1.0;   // NaN included
        nd.c.ib[i][ln] = arg;
        nd.c.z[i][ln] = y * sp.invW;
      }
    }
    g2 += kc * sum_eY - rhoD * sum_hY;
    D[0] = X[1];
    D[1] = g1;
    D[2] = g2;
    // (a forward constant that underflows takes a reverse rate formed from it along, though that may be large)
    fast = __all(!(node && valid) || (big == 0.0 && invT <= mk->invT_factored));
    if (t >= (T0 & ~63)) {
      // Rusanov total flux f = (g- + g+)/2 - lambda (w+ - w-)/2, formed by the right lane of a
      // face's pair from its neighbour's values; at PE interfaces the synchronous flux is published
      // and the AT combination is used
      const double lam1 = fabs(u) + sqrt(cp * rcv * p * rho_inv);
      const double lam = fmax(lam1, dpp_move<kDppFromPrev>(lam1));
      const bool delayed = trace && P.k[fl] > 0;   // its AT flux is in place
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const double gl = dpp_move<kDppFromPrev>(D[v]), xl = dpp_move<kDppFromPrev>(X[v]);
        if (trace && side == 1) {
          const double F = 0.5 * (gl + D[v] - lam * (X[v] - xl));
          if (iface >= 0 && v < Vg && fl <= nloc) ring_at(a.ring, nm, stage, a.dl.nif, iface)[a.ring.off_F + v] = F;
          if (!delayed || v >= Vg) L.F[v][fl - 1] = F;
        }
      }
    }
  }

  // chemistry, by the wavefronts that hold nodes
  if (t < 64 * G::NCW) {
    double wd[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) wd[i] = 0.0;
    nd.c.z[NS][ln] = 1.0;
    if (fast) {
      // z_i = c_i / exp(arg_i): rate = kf [prod_reactants exp(arg)] (prod_reactants z - prod_products z)
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const double ib = exp_taylor(nd.c.ib[i][ln]);
        nd.c.z[i][ln] *= recip(ib);
        nd.c.ib[i][ln] = ib;
      }
      nd.c.ib[NS][ln] = 1.0;
      const int nr = mk->nr;
      // a few reactions side by side: their dependent chains overlap
      for (int q = 0; q < nr; q += kNsReactionGroup) {
        constexpr int R = kNsReactionGroup;
        double kf[R], rate[R];
#pragma unroll
        for (int d = 0; d < R; ++d) kf[d] = fma(mk->rx[q + d].b, lnT, fma(-mk->rx[q + d].EaR, invT, mk->rx[q + d].lnA));
        exp_taylor_n(kf);
#pragma unroll
        for (int d = 0; d < R; ++d) {
          const int r0 = mk->rx[q + d].sp[0], r1 = mk->rx[q + d].sp[1], p0 = mk->rx[q + d].sp[2], p1 = mk->rx[q + d].sp[3];
          const double zr = nd.c.z[r0][ln] * nd.c.z[r1][ln], zp = nd.c.z[p0][ln] * nd.c.z[p1][ln];
          rate[d] = kf[d] * (nd.c.ib[r0][ln] * nd.c.ib[r1][ln]) * (zr - zp);
        }
#pragma unroll
        for (int d = 0; d < R; ++d)
#pragma unroll
          for (int i = 0; i < NS; ++i) wd[i] = fma(mk->rx[q + d].nu[i], rate[d], wd[i]);
      }
    } else {
      // factors beyond the range of their products: the exponents are summed first
      nd.c.ib[NS][ln] = 0.0;
      const int nr = mk->nr;
#pragma unroll 1
      for (int q = 0; q < nr; ++q) {
        const auto &rx = mk->rx[q];
        const int r0 = rx.sp[0], r1 = rx.sp[1], p0 = rx.sp[2], p1 = rx.sp[3];
        const double lnkf = fma(rx.b, lnT, fma(-rx.EaR, invT, rx.lnA));
        const double dg = (nd.c.ib[r0][ln] - nd.c.ib[p0][ln]) + (nd.c.ib[r1][ln] - nd.c.ib[p1][ln]);
        const double fwd = exp(lnkf) * nd.c.z[r0][ln] * nd.c.z[r1][ln];
        const double rev = exp(lnkf + dg) * nd.c.z[p0][ln] * nd.c.z[p1][ln];
        const double rate = fwd - rev;
#pragma unroll
        for (int i = 0; i < NS; ++i) wd[i] = fma(rx.nu[i], rate, wd[i]);
      }
    }
#pragma unroll
    for (int v = 0; v < V; ++v) nd.gs[v][ln] = D[v];
#pragma unroll
    for (int i = 0; i < NS; ++i) nd.gs[V + i][ln] = mk->sp[i].W * wd[i];
  }
  // the first operand (the stage input, in the caches): in flight during the last barrier
  double wi[NI][M];
#pragma unroll
  for (int m = 0; m < NI; ++m) {
    int v, e;
    const double *src = ws + item(m, v, e);
#pragma unroll
    for (int j = 0; j < M; ++j) wi[m][j] = src[j * kLayoutBlock];
  }
  __syncthreads();

  // lift, source projection and RK combination: (variable, element) items
#pragma unroll
  for (int m = 0; m < NI; ++m) {
    int v, e;
    const size_t gi = item(m, v, e);
    if (v == V) continue;
    double g[Q], s[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int p = e * Q + q;
      g[q] = L.nd[p >> 6].gs[v][p & 63];
      s[q] = v >= 3 ? L.nd[p >> 6].gs[V + (v >= 3 ? v - 3 : 0)][p & 63] : 0.0;
    }
    const double Fr = L.F[v][e + 1], Fl = L.F[v][e];
#pragma unroll
    for (int j = 0; j < M; ++j) {
      double vol = 0.0, src = 0.0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        vol = fma(a.tb.WG[q][j], g[q], vol);
        src = fma(a.tb.WB[q][j], s[q], src);
      }
      const double half2j1 = 0.5 * (2 * j + 1);
      const double b = vol - Fr + ((j & 1) ? -Fl : Fl);
      const double Lw = 2.0 * a.inv_dx * (half2j1 * b) + half2j1 * src;
      const size_t gj = gi + (size_t)j * kLayoutBlock;
      double o;
      if (rk.two_n) {
        const double kn = use_prev ? fma(rk.ca, pi[m][j], a.dt * Lw) : a.dt * Lw;
        kbuf[gj] = kn;
        o = fma(rk.cb, kn, wi[m][j]);
      } else {
        const double y = fma(a.dt, Lw, wi[m][j]);
        o = use_prev ? fma(rk.ca, pi[m][j], rk.cb * y) : y;
      }
      wout[gj] = o;
    }
  }
  if (!ok) atomicOr(a.err, (int)kErrState);
  if (advance) advance_step(a.step, par, n, e0 == 0);
}

// Elements per tile: the points and the four outer traces fill three wavefronts to within a few
// lanes, the nodes two of them.
template <int M>
constexpr int kLaneTile = M == 2 ? 46 : M == 3 ? 37 : M == 4 ? 31 : 25;
constexpr int kLaneThreads = 192;
// Wavefronts per SIMD that the registers are bounded for: four let five tiles share a CU
// (E = 2^18, N_p = 3, one box: 154 us against 165 at three); with 16 species that would spill.
constexpr int lane_waves(int ns) { return ns > kNsMaxSpecies ? 3 : 4; }

template <int M, int NS>
__global__ __launch_bounds__(kLaneThreads, lane_waves(NS)) void ns_lane_kernel(NsArgs a) {
  constexpr int TE = kLaneTile<M>;
  static_assert(LaneTile<M, NS, TE>::NTH == kLaneThreads, "three wavefronts");
  __shared__ LaneLds<M, NS, TE> L;
  __shared__ LanePe<TE + 3> P;
  ns_lane_tile<M, NS, TE>(a, a.ws, a.rk.two_n ? a.kbuf : a.w0, a.wout, a.stage, a.advance, a.rk, a.kbuf,
                          xcd_item(blockIdx.x, gridDim.x) * TE, a.step[a.par], a.par, L, P);
}

// LDS of the batched kernel: room for the orders up to MMAX - 1.
template <int M>
struct LaneBatchTile {
  LaneLds<M, kNsMaxSpecies, kLaneTile<M>> L;
  LanePe<kLaneTile<M> + 3> P;
};
template <int MMAX>
union LaneBatchLds {
  LaneBatchLds<MMAX - 1> lower;
  LaneBatchTile<MMAX> t;
};
template <>
union LaneBatchLds<2> {
  LaneBatchTile<2> t;
};

template <int MMAX>
__device__ __forceinline__ void lane_batch_tile(const NsArgs &a, int stage, int e0, long long n, int par,
                                                LaneBatchLds<MMAX> &L) {
  if constexpr (MMAX > 2) {
    if (a.M < MMAX) return lane_batch_tile<MMAX - 1>(a, stage, e0, n, par, L.lower);
  }
  ns_lane_tile<MMAX, kNsMaxSpecies, kLaneTile<MMAX>>(a, a.W[stage], a.W[0], a.W[stage == 2 ? 0 : stage + 1], stage,
                                                     stage == 2, rk_stage(ADG_SSPRK3, stage), nullptr, e0, n, par,
                                                     L.t.L, L.t.P);
}

// Batched stage: one workgroup per (instance, first element) entry of the work list, all at step
// counter parity par; instances differ in size, order (up to MMAX modes: the LDS is sized for the
// largest order present), PE layout and delays.  An instance whose step count has reached its target
// is skipped by all of its workgroups (its first tile carries the count over to the other parity at
// the last stage).  Batches run SSP-RK3.
template <int MMAX>
__global__ __launch_bounds__(kLaneThreads, lane_waves(kNsMaxSpecies)) void ns_lane_batch_kernel(
    const NsArgs *__restrict__ insts, const int2 *__restrict__ tiles, int stage, int par) {
  __shared__ LaneBatchLds<MMAX> L;
  const int2 tl = tiles[blockIdx.x];
  const NsArgs &a = insts[tl.x];
  const long long n = a.step[par];
  if (n >= a.target) {
    if (stage == 2 && tl.y == 0 && threadIdx.x == 0) a.step[par ^ 1] = n;
    return;
  }
  lane_batch_tile<MMAX>(a, stage, tl.y, n, par, L);
}

// ------------------------------------------------------------------ host side

int ns_lane_tile_elems(int M) {
  return M == 2 ? kLaneTile<2> : M == 3 ? kLaneTile<3> : M == 4 ? kLaneTile<4> : kLaneTile<5>;
}

template <int M>
static hipError_t lane_M(const NsArgs &a, hipStream_t s) {
  constexpr int TE = kLaneTile<M>;
  const dim3 grid((a.E + TE - 1) / TE), block(kLaneThreads);
  if (ns_capacity(a.ns) == kNsMaxSpecies) hipLaunchKernelGGL((ns_lane_kernel<M, kNsMaxSpecies>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((ns_lane_kernel<M, kNsWideSpecies>), grid, block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_ns_lane(int M, const NsArgs &a, hipStream_t s) {
  switch (M) {
    case 2: return lane_M<2>(a, s);
    case 3: return lane_M<3>(a, s);
    case 4: return lane_M<4>(a, s);
    case 5: return lane_M<5>(a, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_ns_lane_batch(int max_m, const NsArgs *insts, const int2 *tiles, int ntiles, int stage, int par,
                                hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  const dim3 grid(ntiles), block(kLaneThreads);
  switch (max_m) {
    case 2: hipLaunchKernelGGL((ns_lane_batch_kernel<2>), grid, block, 0, s, insts, tiles, stage, par); break;
    case 3: hipLaunchKernelGGL((ns_lane_batch_kernel<3>), grid, block, 0, s, insts, tiles, stage, par); break;
    case 4: hipLaunchKernelGGL((ns_lane_batch_kernel<4>), grid, block, 0, s, insts, tiles, stage, par); break;
    case 5: hipLaunchKernelGGL((ns_lane_batch_kernel<5>), grid, block, 0, s, insts, tiles, stage, par); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace adg

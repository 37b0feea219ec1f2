// Detailed-chemistry Navier-Stokes stage kernel (LDG): declarations.
#pragma once

#include "adg.h"
#include "adg_internal.hpp"

namespace adg {

// Species capacities of the kernels: a mechanism of Ns species runs in the kernels of the
// smallest capacity that holds it, the species past Ns padded with zero density, no thermo
// and no reactions (they add exact zeros to every species sum and are never stored).
constexpr int kNsMaxSpecies = 9;      // the batched kernel, and single problems with Ns <= 9
constexpr int kNsWideSpecies = 16;    // single problems with 9 < Ns <= 16
constexpr int kNsMaxReactions = 32;
constexpr int kNsReactionGroup = 2;   // reactions that a lane of the lane-per-point kernels forms side by side
// Reactions of a batched mechanism.  The batched kernel could take kNsMaxReactions; the limit is the one that
// adg.h states, which callers may rely on for the refusal.
constexpr int kNsBatchReactions = 24;
// Ea/Ru (K) from which a reaction has no rate in either direction at any temperature of the thermo
// (exp underflows by 2000 and more at 5e5 K), and the size of ln k_f up to which the lane-per-point
// kernels form a reverse rate from k_f.
constexpr double kNsNoRate = 1e9, kNsMaxLnRate = 650.0;
inline int ns_capacity(int n_species) { return n_species <= kNsMaxSpecies ? kNsMaxSpecies : kNsWideSpecies; }

// Mechanism in device memory, read with wave-uniform indices (scalar loads), for kernels of
// species capacity NSC.
template <int NSC>
struct NsMechCoreT {
  static constexpr int kSpecies = NSC;
  int ns, nr;
  double Ru, p_ref, T_guess;
  double mu_ref, ln_T_ref, mu_exp, inv_prandtl;   // mu = mu_ref exp(mu_exp (ln T - ln T_ref))
  double ln_p_over_Ru;              // ln(p_ref / Ru)
  double W[NSC], invW[NSC], Ri[NSC];
  // NASA-7 in Horner-ready form, per species:
  //   cv/R - ... : c0m1 = a0 - 1, a1 .. a4       (cp/R - 1)
  //   (h - R T)/R = T (a0-1 + T (a1/2 + T (a2/3 + T (a3/4 + T a4/5)))) + a5
  //   h/(R T) = a0 + T (a1/2 + ...) + a5 / T
  //   s/R = a0 ln T + T (a1 + T (a2/2 + T (a3/3 + T a4/4))) + a6
  double a[NSC][7];
  double h2[NSC][4];      // a1/2, a2/3, a3/4, a4/5
  double s2[NSC][3];      // a2/2, a3/3, a4/4
  // R_i times the coefficients of the mixture energy quintic (cv/R - 1 form) and R_i:
  // R_i (a0 - 1), R_i a1/2, R_i a2/3, R_i a3/4, R_i a4/5, R_i a5, R_i, 0
  double ek[NSC][8];
  double lnA[kNsMaxReactions], b[kNsMaxReactions], EaR[kNsMaxReactions];
  int dnu[kNsMaxReactions];
  // compact per-reaction form for one lane per (point, reaction): the species
  // multiplied into the forward and reverse rates (-1 = none) and the nonzero
  // net coefficients nu_i = nu''_i - nu'_i with their species, padded to four
  // entries with coefficient 0 (species 0)
  int rf[kNsMaxReactions][2], rr[kNsMaxReactions][2];
  int gidx[kNsMaxReactions][4];
  double gnu[kNsMaxReactions][4];
  // per species, the reactions with a nonzero net coefficient (increasing r) and that
  // coefficient; the entries past the count hold reaction 0 with coefficient 0
  int spn[NSC];
  unsigned char spr[NSC][kNsMaxReactions];
  signed char spnu[NSC][kNsMaxReactions];
  int pad_;
};

// The whole device mechanism: the core (copied to LDS by the kernels that spread species and
// reactions over lanes) and, for the lane-per-point kernels, one record per species and reaction
// in the order they are read, each a whole number of 64-byte scalar loads.
template <int NSC>
struct NsMechT : NsMechCoreT<NSC> {
  // Largest 1/T at which no forward rate constant is near the end of the range of exp: there the
  // rates may be formed from it and the species' factors, whose product would be lost with it.
  double invT_factored;
  struct alignas(64) Species {
    double a0, h2[4], a5;          // h_i/R_i = T (a0 + T (h2[0] + ...)) + a5
    double a1, s2[3], a6;          // s_i/R_i = a0 ln T + T (a1 + T (s2[0] + ...)) + a6
    double Ri, invW, W;
  };
  struct alignas(64) Reaction {
    double lnA, b, EaR;
    unsigned short sp[4];          // species of the reactants and products (two each; NSC: none)
    double nu[NSC];                // net coefficients nu''_i - nu'_i of all species
  };
  Species sp[NSC];
  // padded with reactions of rate zero to whole groups
  Reaction rx[(kNsMaxReactions + kNsReactionGroup - 1) / kNsReactionGroup * kNsReactionGroup];
};
using NsMech = NsMechT<kNsMaxSpecies>;
using NsMechWide = NsMechT<kNsWideSpecies>;

struct NsArgs {
  const double *w0;
  const double *ws;
  double *wout;
  double *W[3];         // the three state buffers (batched kernel picks them by stage)
  int M;                // N_p + 1
  int ns;               // species of the problem (the kernel's capacity may be larger)
  int periodic;         // 1: periodic domain; 0: transmissive ends (ghost trace = interior trace)
  const int *face_if;   // [E+1] interface index of face f, or -1
  long long *step;      // step counters of the two parities (as in EulerArgs)
  int par;              // parity of a single-problem launch
  int advance;          // this launch ends the time step
  int *err;
  long long target;     // batched launches skip the instance once its step reaches it
  const void *mech;     // NsMechT<capacity> of the kernel that runs the problem
  // AT combinations carried between launches (single problems; nullptr: gathered in the launch).
  // Record of face f at f * (2 Vg + 1), Vg = 3 + ns: [0, Vg) the AT central traces, [Vg, 2 Vg)
  // the AT fluxes, [2 Vg] the delay (PE-interface faces).  at_in holds this launch's values
  // (written by the previous launch), at_out receives the next launch's (stage + 1 of this
  // step, or stage 0 of the next; nst stages per step).
  const double *at_in;
  double *at_out;
  int nst;
  int E;
  int stage;
  RkStage rk;
  double *kbuf;         // 2N register (2N schemes)
  int viscous;
  double dt;
  double inv_dx;       // 1/dx
  DelayParams dl;
  RingParams ring;
  Tables tb;
};

bool ns_supported(int n_species, int n_reactions);
// Bytes of the device mechanism of a problem with n_species species.
size_t ns_mech_bytes(int n_species);
void ns_setup(NsArgs &a, const adg_physics *ph, const adg_discretization *d, int E, int M, bool periodic,
              double dx, const DelayParams &dl, const RingParams &rp, const Tables &tb, const int *face_if,
              long long *step, int *err, void *dev_mech);
// The device form of a mechanism to dev_mech (waits; validates the mechanism).
adg_status ns_upload_mech(const adg_physics *ph, void *dev_mech);
// The device form of a mechanism (host side; validates it).
template <int NSC>
adg_status ns_build_mech(const adg_physics *ph, NsMechT<NSC> &hm);
// Kernels of the single-problem stage.  0..4 spread a point's species and reactions over lanes,
// (tile elements, threads) = (8, 512), (8, 256), (4, 256), (4, 512), (8, 1024); kNsLane gives each
// point a lane.
constexpr int kNsLane = 5;
// Work decompositions that adg_set_kernel_config and adg_autotune choose from: 0..4, 1 standing for
// the throughput kernel of the problem's size.
constexpr int kNsConfigs = 5;
// The kernel of work decomposition cfg (-1: none chosen) for E elements of order M - 1, ns species.
int ns_kernel_of(int cfg, int E, int M, int ns);
// Capacity from a.ns; mixed = FP32 modal operators of the kernels 0..4 (for N_p <= 3; N_p = 4 keeps
// FP64 ones).
hipError_t launch_ns_stage(int M, int kernel, const NsArgs &a, bool mixed, hipStream_t s);
// Lane-per-point kernels (FP64 throughout): elements per tile of order M - 1, one stage of a single
// problem, and one stage for every (instance, first element) entry of `tiles` (device) at step
// counter parity par, max_m = the largest N_p + 1 among the listed instances.
int ns_lane_tile_elems(int M);
hipError_t launch_ns_lane(int M, const NsArgs &a, hipStream_t s);
hipError_t launch_ns_lane_batch(int max_m, const NsArgs *insts, const int2 *tiles, int ntiles, int stage, int par,
                                hipStream_t s);
// Elements per work item that a batch's header is sized for: smaller than any tile, so that a header's size,
// which callers keep, does not depend on the kernels' tiles.
constexpr int kNsMinTile = 4;

}  // namespace adg

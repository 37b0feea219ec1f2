// One ADG problem placed in device memory: layout of its region of a
// workspace, device pointers and the argument blocks of its kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "adg.h"
#include "adg_internal.hpp"
#include "adg_ns.hpp"

namespace adg {

constexpr long long kNoTarget = 0x7fffffffffffffffLL;

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
  size_t state, flags, face_if, counters, ring, sched, mech, at, total;
  int nbuf;             // state-sized buffers (3; 4 for a 2N scheme with the limiter)
  int nif, nfaces, D, rec, q, V, M, E;
  int S;                // RK stages per step
  int off_F, off_Wc, off_U;
  bool carry_at;        // AT combinations carried between launches (single detailed problems with PE interfaces)
};

struct Problem {
  adg_physics phys{};
  adg_discretization disc{};
  adg_async as{};
  Layout lay{};
  char *base = nullptr;
  double *W[3] = {nullptr, nullptr, nullptr};
  int8_t *flags = nullptr;
  int *face_if = nullptr;
  long long *step = nullptr;   // [2]: the step counters of the two parities
  int *err = nullptr;
  unsigned long long *flag_count = nullptr;
  double *ring = nullptr;
  double *at = nullptr;        // detailed model with PE interfaces: two per-face AT buffers
  size_t at_stride = 0;        // doubles per buffer
  EulerArgs ea{};
  LimiterArgs la{};
  NsArgs na{};
};

// Validates a problem and computes the layout of its device region (bytes in L.total).
// batched: the layout of a batch instance (no AT carry buffers: the batched kernel gathers).
bool make_layout(const adg_physics *ph, const adg_discretization *d, const adg_async *as, Layout &L,
                 std::string *why, bool batched = false);
// ADG_ERR_UNSUPPORTED for precisions a single problem cannot run (MIXED_BF16; MIXED_FP32 with
// the one-step model), with the reason in *why.
adg_status check_precision(const adg_physics *ph, const adg_discretization *d, std::string *why);
// Places the problem at `base` (256-byte aligned, L.total bytes), fills the kernel arguments and the
// interface index of every face (no device work).
adg_status setup_problem(const adg_physics *phys, const adg_discretization *disc, const adg_async *as, char *base,
                         const Layout &L, Problem &P, std::vector<int> &faces);
// Its constant data to the device: the faces, the schedule and the mechanism (waits).
adg_status upload_problem(const Problem &P, const std::vector<int> &faces);
// Up to kCopies regions of 4-byte words for one launch to copy (either side may be pinned host memory).
constexpr int kCopies = 3;
struct Copies {
  const unsigned *src[kCopies];
  unsigned *dst[kCopies];
  size_t words[kCopies];
};
hipError_t launch_copies(const Copies &c, hipStream_t st);
// Whether the caller is capturing stream st into a graph of its own.  The host does not see the replays
// of such a graph, so from the first capture on the calls that step are bracketed by the two below: what
// the host holds (counter parity, state buffer) then fits whatever ran in between.
bool capturing(hipStream_t st);
// Both parities' counters of n problems to the greater one, the steps done.
hipError_t launch_level_counts(long long *counters, int n, hipStream_t st);
// The same for one problem, whose state is in buffer W[steps done mod 2] between calls where it alternates
// (`alternates`): moved to W[cur] (begin) or from W[cur] back there.
hipError_t launch_align(const Problem &P, bool alternates, int cur, bool begin, hipStream_t st);
// A new state w ([E][V][M]) in W[0], the step counters, error flag, history ring and flags back to
// zero, with `copies` in the same launch: enqueued (capturable); the host form copies w first and waits.
hipError_t set_state_device(const Problem &P, const double *w, hipStream_t st, const Copies *copies = nullptr);
hipError_t set_state_host(const Problem &P, const double *w, hipStream_t st, const Copies *copies = nullptr);
// The state in buffer `state` (one of P.W) in the caller's layout, and the error flag in *err_out
// (device-accessible; null: not reported): enqueued; the host form waits.  With `count` (device) the
// buffer is W[*count mod 2] instead.
hipError_t get_state_device(const Problem &P, const double *state, double *w, int *err_out, hipStream_t st,
                            const long long *count = nullptr);
hipError_t get_state_host(const Problem &P, const double *state, double *w, int *err_out, hipStream_t st,
                          const long long *count = nullptr);

}  // namespace adg

// A HIP runtime and kernel launchers that only record what they are called for, so that the host code of the
// solver and the batch runs on a machine without a GPU, a launch or a capture can be made to fail, and the
// decompositions of the detailed-chemistry kernel take the times that a test gives them.
#include <hip/hip_runtime.h>

#include <cstring>
#include <string>

#include "adg.h"
#include "adg_problem.hpp"

namespace {
std::string calls;                 // "name:argument " per recorded call
std::string fail_name;
int fail_at = -1, seen = 0;        // the fail_at-th call of that name fails (0: the first)

hipError_t call(const char *name, const void *arg) {
  calls += std::string(name) + ":" + std::to_string((uintptr_t)arg) + " ";
  if (fail_name == name && seen++ == fail_at) return hipErrorUnknown;
  return hipSuccess;
}
uintptr_t next_handle = 1000;
int default_kernel = 0, last_kernel = 0;
double kernel_ms[16];
}  // namespace

extern "C" {
void fake_fail(const char *name, int at) { fail_name = name; fail_at = at; seen = 0; calls.clear(); }
const char *fake_calls() { return calls.c_str(); }
void fake_kernels(int untuned, const double *ms) { default_kernel = untuned; std::memcpy(kernel_ms, ms, 6 * sizeof(double)); }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)++next_handle; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return call("sync", s); }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)++next_handle; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) { return call("record", s); }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = (float)kernel_ms[last_kernel]; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { *p = (void *)s; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *, size_t n, hipMemcpyKind) { std::memset(d, 0, n); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) { return call("wait", s); }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { return call("begin", s); }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) { *g = (hipGraph_t)++next_handle; return call("end", s); }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *x = (hipGraphExec_t)++next_handle;
  return call("instantiate", nullptr);
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return call("graph", s); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = malloc(n); return call("pinned", nullptr); }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "failed"; }
}

namespace adg {
bool make_layout(const adg_physics *ph, const adg_discretization *d, const adg_async *, Layout &L, std::string *, bool) {
  L = Layout{};
  L.E = d->n_elem;
  L.M = d->order_p + 1;
  L.V = 3 + ph->n_species;
  L.total = 256;
  return true;
}
adg_status setup_problem(const adg_physics *ph, const adg_discretization *d, const adg_async *as, char *, const Layout &L,
                         Problem &P, std::vector<int> &faces) {
  P = Problem{};
  P.phys = *ph;
  P.disc = *d;
  P.as = *as;
  P.lay = L;
  P.lay.S = 3;
  P.at = (double *)4096;
  P.at_stride = 512;
  faces.assign(L.E + 1, -1);
  return ADG_OK;
}
hipError_t launch_copies(const Copies &c, hipStream_t) {   // counters read back: each one's index
  for (int r = 0; r < kCopies; ++r)
    for (size_t i = 0; i < c.words[r]; ++i) c.dst[r][i] = r == 0 && i % 2 == 0 ? (unsigned)(i / 2) : 0;
  return hipSuccess;
}
bool capturing(hipStream_t) { return false; }
hipError_t launch_level_counts(long long *, int, hipStream_t) { return hipSuccess; }
hipError_t set_state_device(const Problem &, const double *, hipStream_t, const Copies *) { return hipSuccess; }
hipError_t set_state_host(const Problem &, const double *, hipStream_t, const Copies *) { return hipSuccess; }
hipError_t get_state_device(const Problem &, const double *, double *, int *flag, hipStream_t, const long long *) {
  if (flag) *flag = 0;
  return call("read", flag);
}
hipError_t get_state_host(const Problem &, const double *, double *, int *, hipStream_t, const long long *) { return hipSuccess; }
template <int NSC>
adg_status ns_build_mech(const adg_physics *, NsMechT<NSC> &) { return ADG_OK; }
template adg_status ns_build_mech<kNsMaxSpecies>(const adg_physics *, NsMech &);
adg_status check_precision(const adg_physics *, const adg_discretization *, std::string *) { return ADG_OK; }
adg_status upload_problem(const Problem &, const std::vector<int> &) { return ADG_OK; }
hipError_t launch_align(const Problem &, bool, int, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_euler_step(int, int, int, const EulerArgs &, const LimiterArgs *, hipStream_t s) { return call("onestep", s); }
int ns_kernel_of(int cfg, int, int, int) { return cfg < 0 ? default_kernel : cfg == 1 && default_kernel == kNsLane ? kNsLane : cfg; }
hipError_t launch_ns_stage(int, int kernel, const NsArgs &a, bool, hipStream_t) {
  last_kernel = kernel;
  return call(a.at_in ? "carried" : "gathered", (const void *)(uintptr_t)kernel);
}
int ns_lane_tile_elems(int) { return 32; }
int euler_blocks(int E, int, bool) { return (E + 51) / 52; }
hipError_t launch_ns_lane_batch(int, const NsArgs *, const int2 *, int, int, int, hipStream_t s) { return call("detailed", s); }
hipError_t launch_euler_batch(int, int, bool, const EulerSet *, const int2 *, int, int par, hipStream_t s) {
  calls += "par:" + std::to_string(par) + " ";
  return call("onestep", s);
}
}  // namespace adg

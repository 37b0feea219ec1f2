// Host runtime of the ADG library: the C ABI of include/adg.h.
//
// The solver owns no device memory: the caller's workspace is carved into
// 256-byte aligned regions (state planes, limiter buffers, history ring, face
// map, counters).  Every launch goes to the caller's stream; adg_set_graph()
// switches adg_step to a captured HIP graph of several time steps.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "adg.h"
#include "adg_internal.hpp"
#include "adg_ns.hpp"
#include "adg_problem.hpp"

using namespace adg;

// Device memory of the solver that adg_create_noalloc places without allocating: one
// array per device (every device the library runs on holds it until the process ends).
// In host code `scratch` names a host-side stand-in, not the device array: its device
// address comes from hipGetSymbolAddress, once per device with that device current, and
// only that address is ever passed on.
constexpr size_t kScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

struct adg_solver {
  Problem P;
  hipStream_t stream = nullptr;
  int cur = 0;            // state buffer at the start of the next step (2N schemes alternate 0 and 1)
  int par = 0;            // step counter parity of the next step (P.step[par] holds its count)
  // Captured graphs of graph_steps time steps.  A step moves (cur, par) to the other of two
  // alignments (the counter parity flips every step; the state buffer, where it moves, flips
  // with it), and a graph replays only from the alignment it was captured at: graph k starts
  // from (graph_cur[k], graph_par[k]), graph 1 from the alignment one step after graph 0's,
  // so every alignment has a graph and no realigning plain step is ever needed.
  int graph_cur[2] = {0, 0}, graph_cur_after[2] = {0, 0};
  int graph_par[2] = {0, 0}, graph_par_after[2] = {0, 0};
  int ns_cfg = -1;  // work decomposition of the detailed-chemistry stage kernel (-1: none chosen)
  bool at_ready = false;   // the last launch left its successor's AT combinations (set_at_buffers)
  bool captured = false;   // the caller has captured calls on this solver into graphs of its own
  int graph_steps = 0;
  int graph_built_for = 0;
  hipGraph_t graph[2] = {nullptr, nullptr};
  hipGraphExec_t gexec[2] = {nullptr, nullptr};
  long long graph_replays = 0;   // graphs launched since set_state (adg_graph_replays)
  hipStream_t cap_stream = nullptr;
  std::vector<hipEvent_t> prof_events;
  std::string msg;
  int *host_err = nullptr;   // pinned: the error flag as adg_get_state's kernel stores it (null: copied instead)
  int noalloc_dev = -1;   // device whose static scratch holds this solver (adg_create_noalloc), else -1
};

namespace {

// Message of the last failed create call on this thread (adg_last_error(NULL)).
thread_local std::string g_create_msg = "no error";

adg_status create_fail(adg_status code, const std::string &m) {
  g_create_msg = m;
  return code;
}

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` per device (hipGetSymbolAddress)
adg_solver g_noalloc_solver[kMaxDevices];
bool g_noalloc_busy[kMaxDevices] = {};

// Pinned words that adg_get_state's kernels store the error flag in beside the state, so that one wait gives
// both (16 us for a small state on the device, 25 with the flag copied after it).  One block for the process,
// since allocating pinned memory takes as long as many reads (40 to 400 us), handed out word by word: taken at
// a solver's first read, given back by adg_destroy.  A process that reads one state never allocates it, and
// solvers beyond its words copy their flags.
class FlagWords {
 public:
  int *take() {
    std::lock_guard<std::mutex> lock(m_);
    if (reads_ < 1) { reads_ += 1; return nullptr; }
    if (!block_) {
      if (hipHostMalloc((void **)&block_, kWords * kStride * sizeof(int), hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        block_ = nullptr;
        return nullptr;
      }
      for (int i = kWords - 1; i >= 0; --i) free_.push_back(block_ + i * kStride);
    }
    if (free_.empty()) return nullptr;
    int *p = free_.back();
    free_.pop_back();
    return p;
  }
  void give(int *p) {
    if (!p) return;
    std::lock_guard<std::mutex> lock(m_);
    free_.push_back(p);
  }

 private:
  static constexpr int kWords = 64, kStride = 16;   // a cache line each
  std::mutex m_;
  int *block_ = nullptr;
  int reads_ = 0;
  std::vector<int *> free_;
};
FlagWords &g_flags = *new FlagWords;   // never destroyed: solvers may outlive static objects

adg_status fail(adg_solver *s, adg_status code, const std::string &m) {
  if (s) s->msg = m;
  return code;
}

adg_status hip_fail(adg_solver *s, hipError_t e, const char *where) {
  return fail(s, ADG_ERR_HIP, std::string(where) + ": " + hipGetErrorString(e));
}

#define HIP_TRY(s, expr)                          \
  do {                                            \
    hipError_t _e = (expr);                       \
    if (_e != hipSuccess) return hip_fail(s, _e, #expr); \
  } while (0)

// Launch the kernels of one time step.  `timer` (optional) records an event
// pair around each launch for adg_profile.
typedef void (*TimerFn)(adg_solver *, int cls, bool begin);

int ns_kernel(const adg_solver *s, int cfg) {
  return ns_kernel_of(cfg, s->P.lay.E, s->P.lay.M, s->P.phys.n_species);
}

// Carried AT combinations of the launch of `stage` in the step at parity s->par: launch number
// n S + stage of the run (n mod 2 = s->par: both start at zero) reads buffer (n S + stage) mod 2
// and leaves its successor's values in the other one.  The lane-per-point kernels neither read nor
// write them, so a launch reads them only if its predecessor wrote them (s->at_ready); it forms
// the same values from the history otherwise.
void set_at_buffers(const adg_solver *s, NsArgs &a, int stage) {
  if (!s->P.at) return;
  const int b = (s->par * s->P.lay.S + stage) & 1;
  a.at_in = s->at_ready ? s->P.at + (size_t)b * s->P.at_stride : nullptr;
  a.at_out = s->P.at + (size_t)(1 - b) * s->P.at_stride;
}

// The state buffer and step counter parity after one time step from (cur, par).
void next_alignment(const adg_solver *s, int &cur, int &par) {
  if (s->P.phys.model == ADG_ONESTEP) cur = 1 - cur;
  else if (rk_stage(s->P.disc.rk, 0).two_n) cur = (cur + s->P.lay.S) % 2;
  par ^= 1;   // the step's last launch wrote the next count into the other counter
}

adg_status enqueue_step(adg_solver *s, hipStream_t st, TimerFn timer) {
  const int M = s->P.lay.M, S = s->P.lay.S;
  const int rk = s->P.disc.rk;
  if (s->P.phys.model == ADG_ONESTEP) {
    // the whole step in one launch; its halo lanes read other wavefronts' elements, so the
    // state alternates between buffers 0 and 1
    EulerArgs a = s->P.ea;
    a.ws = s->P.W[s->cur];
    a.wout = s->P.W[1 - s->cur];
    a.par = s->par;
    if (timer) timer(s, 0, true);
    HIP_TRY(s, launch_euler_step(M, s->P.disc.flux, S, a, s->P.disc.limiter ? &s->P.la : nullptr, st));
    if (timer) timer(s, 0, false);
    next_alignment(s, s->cur, s->par);
    return ADG_OK;
  }
  const int in_buf[3] = {0, 1, 2}, out_buf[3] = {1, 2, 0};
  for (int stage = 0; stage < S; ++stage) {
    const RkStage r = rk_stage(rk, stage);
    // Shu-Osher SSP-RK3: w^n in buffer 0, stages in 1 and 2, the last stage back into 0.
    // 2N schemes: the state alternates between buffers 0 and 1 (s->cur holds it at the start
    // of the step), the register is buffer 2.
    const int bi = r.two_n ? (s->cur + stage) % 2 : in_buf[stage];
    const int bo = r.two_n ? (s->cur + stage + 1) % 2 : out_buf[stage];
    NsArgs a = s->P.na;
    a.w0 = s->P.W[0];
    a.ws = s->P.W[bi];
    a.wout = s->P.W[bo];
    a.stage = stage;
    a.rk = r;
    a.advance = stage == S - 1;
    a.par = s->par;
    set_at_buffers(s, a, stage);
    if (timer) timer(s, 0, true);
    const int kernel = ns_kernel(s, s->ns_cfg);
    HIP_TRY(s, launch_ns_stage(M, kernel, a, s->P.disc.precision == ADG_MIXED_FP32, st));
    s->at_ready = kernel != kNsLane;
    if (timer) timer(s, 0, false);
  }
  next_alignment(s, s->cur, s->par);
  return ADG_OK;
}

// Brackets of the calls that launch steps.  A solver that the caller has captured (or is capturing) may
// have been stepped by replays since the last call: the state goes to the buffer that the host steps from
// and back, and the first launch relies on no carried AT values.
hipError_t align(adg_solver *s, bool begin) {
  if (!s->captured) return hipSuccess;
  s->at_ready = false;
  int cur = 0, par = 0;
  next_alignment(s, cur, par);
  return launch_align(s->P, cur != 0, s->cur, begin, s->stream);
}

void destroy_graph(adg_solver *s) {
  for (int k = 0; k < 2; ++k) {
    if (s->gexec[k]) (void)hipGraphExecDestroy(s->gexec[k]);
    if (s->graph[k]) (void)hipGraphDestroy(s->graph[k]);
    s->gexec[k] = nullptr;
    s->graph[k] = nullptr;
  }
  s->graph_built_for = 0;
}

// Capture graph k from alignment (cur0, par0); nothing runs, the capture only records.
adg_status capture_graph(adg_solver *s, int k, int cur0, int par0) {
  const int cur_keep = s->cur, par_keep = s->par;
  const bool at_keep = s->at_ready;
  HIP_TRY(s, hipStreamBeginCapture(s->cap_stream, hipStreamCaptureModeThreadLocal));
  s->cur = cur0;
  s->par = par0;
  s->at_ready = false;   // whatever ran before a replay: its first launch reads no carried values
  adg_status rc = ADG_OK;
  for (int i = 0; i < s->graph_steps && rc == ADG_OK; ++i) rc = enqueue_step(s, s->cap_stream, nullptr);
  s->graph_cur[k] = cur0;
  s->graph_par[k] = par0;
  s->graph_cur_after[k] = s->cur;
  s->graph_par_after[k] = s->par;
  s->cur = cur_keep;
  s->par = par_keep;
  s->at_ready = at_keep;
  hipGraph_t g = nullptr;
  hipError_t e = hipStreamEndCapture(s->cap_stream, &g);
  if (rc != ADG_OK) { if (g) (void)hipGraphDestroy(g); return rc; }
  if (e != hipSuccess) return hip_fail(s, e, "hipStreamEndCapture");
  s->graph[k] = g;
  HIP_TRY(s, hipGraphInstantiate(&s->gexec[k], g, nullptr, nullptr, 0));
  return ADG_OK;
}

adg_status build_graph(adg_solver *s) {
  destroy_graph(s);
  if (!s->cap_stream) HIP_TRY(s, hipStreamCreateWithFlags(&s->cap_stream, hipStreamNonBlocking));
  int cur1 = s->cur, par1 = s->par;
  next_alignment(s, cur1, par1);
  adg_status rc = capture_graph(s, 0, s->cur, s->par);
  if (rc == ADG_OK) rc = capture_graph(s, 1, cur1, par1);
  if (rc != ADG_OK) { destroy_graph(s); return rc; }
  s->graph_built_for = s->graph_steps;
  return ADG_OK;
}

}  // namespace

extern "C" {

size_t adg_workspace_bytes(const adg_physics *phys, const adg_discretization *disc, const adg_async *as) {
  Layout L;
  if (!make_layout(phys, disc, as, L, nullptr)) return 0;
  return L.total;
}

adg_status adg_create(const adg_physics *phys, const adg_discretization *disc, const adg_async *as,
                      void *device_workspace, size_t workspace_bytes, void *hip_stream, adg_solver **out) {
  if (!out) return create_fail(ADG_ERR_ARG, "out is null");
  *out = nullptr;
  Layout L;
  std::string why;
  if (!make_layout(phys, disc, as, L, &why)) return create_fail(ADG_ERR_ARG, why);
  if (check_precision(phys, disc, &why) != ADG_OK) return create_fail(ADG_ERR_UNSUPPORTED, why);
  if (!device_workspace || ((uintptr_t)device_workspace & 255))
    return create_fail(ADG_ERR_ARG, "workspace must be a non-null 256-byte aligned device pointer");
  if (workspace_bytes < L.total) return create_fail(ADG_ERR_NOMEM, "workspace smaller than adg_workspace_bytes()");
  adg_solver *s = new adg_solver();
  std::vector<int> faces;
  adg_status rc = setup_problem(phys, disc, as, (char *)device_workspace, L, s->P, faces);
  if (rc == ADG_OK) rc = upload_problem(s->P, faces);
  if (rc != ADG_OK) { delete s; return create_fail(rc, "problem set-up failed (unsupported combination or HIP error)"); }
  s->stream = (hipStream_t)hip_stream;
  *out = s;
  return ADG_OK;
}

adg_status adg_create_noalloc(const adg_physics *phys, const adg_discretization *disc, const adg_async *as,
                              void *hip_stream, adg_solver **out) {
  if (!out) return create_fail(ADG_ERR_ARG, "out is null");
  *out = nullptr;
  Layout L;
  std::string why;
  if (!make_layout(phys, disc, as, L, &why)) return create_fail(ADG_ERR_ARG, why);
  if (check_precision(phys, disc, &why) != ADG_OK) return create_fail(ADG_ERR_UNSUPPORTED, why);
  if (L.total > kScratchBytes)
    return create_fail(ADG_ERR_NOMEM, "problem needs " + std::to_string(L.total) + " bytes; the static scratch of "
                                          "adg_create_noalloc holds " + std::to_string(kScratchBytes));
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return create_fail(ADG_ERR_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return create_fail(ADG_ERR_UNSUPPORTED, "device index beyond 63");
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return create_fail(ADG_ERR_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  if (g_noalloc_busy[dev])
    return create_fail(ADG_ERR_STATE, "a solver of adg_create_noalloc is alive on this device (destroy it first)");
  adg_solver *s = &g_noalloc_solver[dev];
  *s = adg_solver();
  std::vector<int> faces;
  adg_status rc = setup_problem(phys, disc, as, (char *)g_scratch_ptr[dev], L, s->P, faces);
  if (rc == ADG_OK) rc = upload_problem(s->P, faces);
  if (rc != ADG_OK) return create_fail(rc, "problem set-up failed (unsupported combination or HIP error)");
  s->stream = (hipStream_t)hip_stream;
  s->noalloc_dev = dev;
  g_noalloc_busy[dev] = true;
  *out = s;
  return ADG_OK;
}

adg_status adg_set_state(adg_solver *s, const double *w, int64_t count, int32_t where) {
  if (!s || !w) return ADG_ERR_ARG;
  const Layout &L = s->P.lay;
  if (count != (int64_t)L.E * L.V * L.M) return fail(s, ADG_ERR_ARG, "state size mismatch");
  if (where == ADG_HOST) {
    HIP_TRY(s, set_state_host(s->P, w, s->stream));
  } else if (where == ADG_DEVICE) {
    HIP_TRY(s, set_state_device(s->P, w, s->stream));
  } else {
    return fail(s, ADG_ERR_ARG, "where must be ADG_HOST or ADG_DEVICE");
  }
  s->cur = 0;
  s->par = 0;
  s->at_ready = false;
  s->graph_replays = 0;
  if (capturing(s->stream)) s->captured = true;
  return ADG_OK;
}

static adg_status run_steps(adg_solver *s, int n_steps, bool graphs) {
  if (graphs) {
    if (s->graph_built_for != s->graph_steps) {
      adg_status rc = build_graph(s);
      if (rc != ADG_OK) return rc;
    }
    // whole graphs from the graph of the current alignment, then plain steps for the rest
    int left = n_steps;
    while (left > 0) {
      int k = -1;
      for (int c = 0; c < 2; ++c)
        if (s->cur == s->graph_cur[c] && s->par == s->graph_par[c]) k = c;
      if (left >= s->graph_steps && k >= 0) {
        HIP_TRY(s, hipGraphLaunch(s->gexec[k], s->stream));
        s->cur = s->graph_cur_after[k];
        s->par = s->graph_par_after[k];
        s->at_ready = ns_kernel(s, s->ns_cfg) != kNsLane;
        left -= s->graph_steps;
        s->graph_replays += 1;
      } else {
        adg_status rc = enqueue_step(s, s->stream, nullptr);
        if (rc != ADG_OK) return rc;
        left -= 1;
      }
    }
    return ADG_OK;
  }
  for (int i = 0; i < n_steps; ++i) {
    adg_status rc = enqueue_step(s, s->stream, nullptr);
    if (rc != ADG_OK) return rc;
  }
  return ADG_OK;
}

adg_status adg_step(adg_solver *s, int32_t n_steps) {
  if (!s || n_steps < 0) return ADG_ERR_ARG;
  // into a graph of the caller's: plain launches (a graph launched while its stream is captured runs at once)
  const bool cap = capturing(s->stream);
  if (cap) s->captured = true;
  HIP_TRY(s, align(s, true));
  adg_status rc = run_steps(s, n_steps, s->graph_steps > 0 && !cap);
  if (rc == ADG_OK) HIP_TRY(s, align(s, false));
  return rc;
}

static adg_status state_status(adg_solver *s, int err) {
  if (err) return fail(s, ADG_ERR_STATE, "non-physical state (rho <= 0, p <= 0, non-finite or no T convergence)");
  return ADG_OK;
}

adg_status adg_sync(adg_solver *s) {
  if (!s) return ADG_ERR_ARG;
  HIP_TRY(s, hipStreamSynchronize(s->stream));
  int err = 0;
  HIP_TRY(s, hipMemcpy(&err, s->P.err, sizeof(int), hipMemcpyDeviceToHost));
  return state_status(s, err);
}

adg_status adg_get_state(adg_solver *s, double *w, int64_t count, int32_t where) {
  if (!s || !w) return ADG_ERR_ARG;
  const Layout &L = s->P.lay;
  if (count != (int64_t)L.E * L.V * L.M) return fail(s, ADG_ERR_ARG, "state size mismatch");
  if (!s->host_err && s->noalloc_dev < 0) s->host_err = g_flags.take();
  HIP_TRY(s, align(s, true));
  if (where == ADG_HOST) {
    HIP_TRY(s, get_state_host(s->P, s->P.W[s->cur], w, s->host_err, s->stream));
  } else if (where == ADG_DEVICE) {
    HIP_TRY(s, get_state_device(s->P, s->P.W[s->cur], w, s->host_err, s->stream));
  } else {
    return fail(s, ADG_ERR_ARG, "where must be ADG_HOST or ADG_DEVICE");
  }
  if (!s->host_err) return adg_sync(s);
  HIP_TRY(s, hipStreamSynchronize(s->stream));
  return state_status(s, *(volatile int *)s->host_err);
}

adg_status adg_get_flags(adg_solver *s, int8_t *flags, int64_t *total) {
  if (!s) return ADG_ERR_ARG;
  HIP_TRY(s, hipStreamSynchronize(s->stream));
  if (flags) HIP_TRY(s, hipMemcpy(flags, s->P.flags, (size_t)s->P.lay.E, hipMemcpyDeviceToHost));
  if (total) {
    unsigned long long c = 0;
    HIP_TRY(s, hipMemcpy(&c, s->P.flag_count, sizeof c, hipMemcpyDeviceToHost));
    *total = (int64_t)c;
  }
  return ADG_OK;
}

int64_t adg_step_count(adg_solver *s) {
  if (!s) return -1;
  if (hipStreamSynchronize(s->stream) != hipSuccess) return -1;
  long long n = 0;
  if (hipMemcpy(&n, s->P.step + s->par, sizeof n, hipMemcpyDeviceToHost) != hipSuccess) return -1;
  return n;
}

int32_t adg_n_interfaces(const adg_solver *s) { return s ? s->P.lay.nif : -1; }

static void prof_timer(adg_solver *s, int cls, bool begin) {
  (void)cls;
  (void)begin;
  hipEvent_t ev;
  if (hipEventCreate(&ev) != hipSuccess) return;
  (void)hipEventRecord(ev, s->stream);
  s->prof_events.push_back(ev);
}

adg_status adg_profile(adg_solver *s, int32_t n_steps, double *ms_out, int64_t *launches_out, int32_t n_classes) {
  if (!s || n_steps < 1 || !ms_out || !launches_out || n_classes < 1) return ADG_ERR_ARG;
  s->prof_events.clear();
  HIP_TRY(s, align(s, true));
  for (int i = 0; i < n_steps; ++i) {
    adg_status rc = enqueue_step(s, s->stream, prof_timer);
    if (rc != ADG_OK) return rc;
  }
  HIP_TRY(s, align(s, false));
  // the launches of one step, all of class 0
  const std::vector<int> order(s->prof_events.size() / 2 / n_steps, 0);
  HIP_TRY(s, hipStreamSynchronize(s->stream));
  std::vector<double> sum(n_classes, 0.0);
  std::vector<int64_t> cnt(n_classes, 0);
  size_t per_step = order.size();
  for (int i = 0; i < n_steps; ++i)
    for (size_t k = 0; k < per_step; ++k) {
      size_t idx = ((size_t)i * per_step + k) * 2;
      float ms = 0.0f;
      (void)hipEventElapsedTime(&ms, s->prof_events[idx], s->prof_events[idx + 1]);
      int c = order[k];
      if (c < n_classes) { sum[c] += ms; cnt[c] += 1; }
    }
  for (hipEvent_t ev : s->prof_events) (void)hipEventDestroy(ev);
  s->prof_events.clear();
  for (int c = 0; c < n_classes; ++c) {
    ms_out[c] = cnt[c] ? sum[c] / cnt[c] : 0.0;
    launches_out[c] = cnt[c];
  }
  return adg_sync(s);
}

adg_status adg_autotune(adg_solver *s, int32_t n_reps, int32_t *choice) {
  if (!s || n_reps < 1) return ADG_ERR_ARG;
  if (choice) *choice = 0;
  if (s->P.phys.model != ADG_DETAILED) return ADG_OK;   // one decomposition only
  const int M = s->P.lay.M;
  HIP_TRY(s, align(s, true));
  // first-stage launches only: they read the state and write the first stage's output
  // buffer (and the 2N register, whose old value the first stage does not read) and the
  // level's first-stage history, all of which the next step recomputes; the state is untouched
  NsArgs a = s->P.na;
  const bool mixed = s->P.disc.precision == ADG_MIXED_FP32;
  a.rk = rk_stage(s->P.disc.rk, 0);
  const int bi = a.rk.two_n ? s->cur : 0, bo = a.rk.two_n ? (s->cur + 1) % 2 : 1;
  a.w0 = s->P.W[0];
  a.ws = s->P.W[bi];
  a.wout = s->P.W[bo];
  a.stage = 0;
  a.advance = 0;
  a.par = s->par;
  set_at_buffers(s, a, 0);   // writes only the successor's buffer, which the next step rewrites
  if (s->P.at && !a.at_in) {
    // The steps to come read carried AT values, so that is what is timed, also where no launch has left
    // any: one that gathers leaves those of the next stage, of the same faces and delays.  The step after
    // the tuning gathers.
    HIP_TRY(s, launch_ns_stage(M, 0, a, mixed, s->stream));
    double *other = s->P.at + (a.at_out == s->P.at ? s->P.at_stride : 0);
    a.at_in = a.at_out;
    a.at_out = other;
  }
  // every candidate warmed up first, then timed in three interleaved rounds; each keeps
  // its fastest round (clock ramp-up and other transients then bias no candidate)
  double t[kNsConfigs];
  hipEvent_t e0, e1;
  HIP_TRY(s, hipEventCreate(&e0));
  HIP_TRY(s, hipEventCreate(&e1));
  for (int c = 0; c < kNsConfigs; ++c) {
    for (int r = 0; r < 2; ++r) HIP_TRY(s, launch_ns_stage(M, ns_kernel(s, c), a, mixed, s->stream));
    t[c] = 1e30;
  }
  for (int round = 0; round < 3; ++round)
    for (int c = 0; c < kNsConfigs; ++c) {
      HIP_TRY(s, hipEventRecord(e0, s->stream));
      for (int r = 0; r < n_reps; ++r) HIP_TRY(s, launch_ns_stage(M, ns_kernel(s, c), a, mixed, s->stream));
      HIP_TRY(s, hipEventRecord(e1, s->stream));
      HIP_TRY(s, hipEventSynchronize(e1));
      float ms = 0.0f;
      HIP_TRY(s, hipEventElapsedTime(&ms, e0, e1));
      t[c] = std::min(t[c], (double)ms);
    }
  // the decomposition that an untuned solver takes stays unless the fastest beats it by more than 3 %:
  // candidates closer than that trade places from run to run (and under a profiler's dispatch overhead)
  const int untuned = ns_kernel(s, -1) == kNsLane ? 1 : ns_kernel(s, -1);
  int best = untuned;
  for (int c = 0; c < kNsConfigs; ++c)
    if (t[c] < t[best]) best = c;
  if (t[best] > 0.97 * t[untuned]) best = untuned;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  HIP_TRY(s, align(s, false));
  if (best != s->ns_cfg) {
    s->ns_cfg = best;
    destroy_graph(s);
  }
  if (choice) *choice = best;
  return adg_sync(s);
}

adg_status adg_set_kernel_config(adg_solver *s, int32_t config) {
  if (!s) return ADG_ERR_ARG;
  const int n = s->P.phys.model == ADG_DETAILED ? kNsConfigs : 1;
  if (config < 0 || config >= n) return fail(s, ADG_ERR_ARG, "no such work decomposition");
  if (s->P.phys.model == ADG_DETAILED && config != s->ns_cfg) {
    s->ns_cfg = config;
    destroy_graph(s);
  }
  return ADG_OK;
}

int64_t adg_graph_replays(const adg_solver *s) { return s ? s->graph_replays : -1; }

adg_status adg_set_graph(adg_solver *s, int32_t steps_per_graph) {
  if (!s || steps_per_graph < 0) return ADG_ERR_ARG;
  s->graph_steps = steps_per_graph;
  if (steps_per_graph == 0) destroy_graph(s);
  return ADG_OK;
}

void adg_destroy(adg_solver *s) {
  if (!s) return;
  destroy_graph(s);
  if (s->cap_stream) (void)hipStreamDestroy(s->cap_stream);
  s->cap_stream = nullptr;
  g_flags.give(s->host_err);
  s->host_err = nullptr;
  if (s->noalloc_dev >= 0) {
    g_noalloc_busy[s->noalloc_dev] = false;   // the static solver and scratch are free again
    s->noalloc_dev = -1;
    return;
  }
  delete s;
}

const char *adg_last_error(const adg_solver *s) { return s ? s->msg.c_str() : g_create_msg.c_str(); }

}  // extern "C"

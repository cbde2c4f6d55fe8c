// A device that runs on the CPU, for tests of the library's host layer (lbm_api, host_copy): HIP
// calls and kernel launchers with the orders that streams promise and no others. An operation
// waits in its stream's queue until something synchronises with it; the per-thread stream is
// another queue in every thread. A stored state is one number, the steps it has taken.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

#include "lbm_internal.h"
#include "routes.h"

namespace {
using Op = std::function<void()>;
struct Queue {
  std::vector<Op> ops;
  size_t done = 0;
  bool capturing = false;
  std::vector<Op> graph;
};
struct Event {
  Queue* q = nullptr;
  size_t at = 0;
  int device = 0;
};
std::recursive_mutex mu;
std::map<std::pair<void*, std::thread::id>, Queue> queues;
std::map<char*, size_t> pinned;
std::map<void*, size_t> allocated;
std::vector<double> uploaded;
std::thread::id home;  // the thread that calls the library
long foreign = 0, pins = 0, copies = 0;
int record_room = 0, fail_in = 0, streams_device = 0, next_launches = 0;
size_t malloc_limit = ~(size_t)0;
thread_local int current = 0;

using Lock = std::lock_guard<std::recursive_mutex>;

Queue& queue(hipStream_t s) {
  if (std::this_thread::get_id() != home) ++foreign;
  const std::thread::id none;
  return queues[{(void*)s, s == hipStreamPerThread ? std::this_thread::get_id() : none}];
}
void run(Queue& q, size_t upto) {
  for (; q.done < upto; ++q.done) q.ops[q.done]();
}
hipError_t put(hipStream_t s, Op op) {
  Lock lock(mu);
  Queue& q = queue(s);
  (q.capturing ? q.graph : q.ops).push_back(std::move(op));
  return hipSuccess;
}
hipError_t step(hipStream_t s, Op op) {  // a time step's launch, which may be made to fail
  Lock lock(mu);
  ++next_launches;
  if (fail_in > 0 && --fail_in == 0) return hipErrorLaunchFailure;
  return put(s, std::move(op));
}
bool is_pinned(const void* p) {
  const char* c = static_cast<const char*>(p);
  for (auto& r : pinned)
    if (c >= r.first && c < r.first + r.second) return true;
  return false;
}
long& count(const void* A) { return *static_cast<long*>(const_cast<void*>(A)); }
}  // namespace

extern "C" {
void fake_reset() {
  Lock lock(mu);
  queues.clear();
  uploaded.clear();
  home = std::this_thread::get_id();
  foreign = pins = copies = 0;
  fail_in = next_launches = 0;
  streams_device = current = 0;
  malloc_limit = ~(size_t)0;
}
long fake_foreign() { return foreign; }
long fake_pins() { return pins; }
long fake_copies() { return copies; }
long fake_pinned_bytes() {
  long b = 0;
  for (auto& r : pinned) b += (long)r.second;
  return b;
}
int fake_record_room() { return record_room; }
int fake_step_launches() { return next_launches; }
void fake_fail_step_launch(int k) { fail_in = k; }
void fake_malloc_limit(size_t bytes) { malloc_limit = bytes; }
int fake_current_device() { return current; }
void fake_set_device(int d) { current = d; }
const double* fake_uploaded() { return uploaded.data(); }
void fake_capture(void* s, int on) { queue((hipStream_t)s).capturing = on != 0; }
void fake_replay(void* s) {
  Queue& q = queue((hipStream_t)s);
  for (const Op& op : q.graph) q.ops.push_back(op);
}

// the library's rules for the double distribution (D2Q9)
int fake_ddf_records(int nx, int ny, int phi, int fmt) {
  const lbm::Layout L = lbm::make_layout(nx, ny, 1, 4);
  return lbm::ddf_max_records(L, lbm::make_grid_ddf(L, phi == 2 ? 2 : 1, fmt >= 2), phi, fmt);
}
int fake_ddf_rows(int nx, int ny, int phi, int fmt, int collision, int bounce) {
  const lbm::Layout L = lbm::make_layout(nx, ny, 1, 4);
  return lbm::ddf_step_grid(lbm::make_grid_ddf(L, phi == 2 ? 2 : 1, fmt >= 2), L, phi, fmt, (lbm::DdfCollision)collision, bounce, 1 << 30).rows;
}
int fake_bgk3_pair(int nx, int ny, int nz) {
  const lbm::Layout L = lbm::make_layout(nx, ny, nz, 4);
  return lbm::bgk3_pair_supported(L, lbm::bgk3_pair_shape(L));
}
int fake_ddf_pair(int nx, int ny, int src, int full, int eos, int neq) {
  const lbm::Layout L = lbm::make_layout(nx, ny, 1, 4);
  lbm::DdfParams prm{};
  prm.phi = 1;
  prm.src = src;
  prm.full = full || eos;
  prm.eos = eos;
  prm.neq = neq;
  return lbm::ddf_pair_supported(0, L, prm, lbm::ddf_pair_shape(L, prm));
}

// ---- HIP ------------------------------------------------------------------------------------
hipError_t hipMalloc(void** p, size_t n) {
  Lock lock(mu);
  if (n > malloc_limit) return hipErrorOutOfMemory;
  *p = aligned_alloc(256, (n + 255) / 256 * 256);
  std::memset(*p, 0x5a, n);
  allocated[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  Lock lock(mu);
  allocated.erase(p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  Lock lock(mu);
  ++pins;
  *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096);
  pinned[static_cast<char*>(*p)] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  Lock lock(mu);
  pinned.erase(static_cast<char*>(p));
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st) {
  Lock lock(mu);
  ++copies;
  (void)put(st, [=] { std::memcpy(d, s, n); });
  const void* host = k == hipMemcpyHostToDevice ? s : d;
  Queue& q = queue(st);
  if (k != hipMemcpyDeviceToDevice && !is_pinned(host) && !q.capturing) run(q, q.ops.size());
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
  return put(st, [=] { std::memset(d, v, n); });
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  Lock lock(mu);
  Queue& q = queue(s);
  if (q.capturing) return hipErrorStreamCaptureUnsupported;
  run(q, q.ops.size());
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  Lock lock(mu);
  *st = queue(s).capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) {
  *d = s ? streams_device : current;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t) new Event{nullptr, 0, current};
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete (Event*)e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  Lock lock(mu);
  Event* v = (Event*)e;
  if (v->device != (s ? streams_device : current)) return hipErrorInvalidHandle;
  v->q = &queue(s);
  v->at = v->q->ops.size();
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  Lock lock(mu);
  Event* v = (Event*)e;
  if (v->q) run(*v->q, v->at);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = current;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  current = d;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  Lock lock(mu);
  std::memset((void*)a, 0, sizeof(*a));
  a->type = is_pinned(p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake"; }
}  // extern "C"

// ---- launchers --------------------------------------------------------------------------------
namespace lbm {
Layout make_layout(int nx, int ny, int nz, int) {
  Layout L{nx, ny, nz, (nx + 63) / 64 * 64, 0};
  L.plane = L.pitch * ny * nz;
  return L;
}
static Grid grid() { return Grid{256, 4, 4, 8}; }
Grid make_grid(const Layout&) { return grid(); }
Grid make_grid_ddf3(const Layout&) { return grid(); }
Grid make_grid_red(const Layout&) { return grid(); }
Grid make_grid_mlp(const Layout&) { return grid(); }
size_t red_state_bytes(const Layout& L) { return (size_t)L.plane * 24; }
int64_t ddf3_max_records(const Layout&, const Grid&) { return 32; }
int mlp_partial_count(int B) { return (B + 63) / 64; }

static hipError_t take(const void* A, void* B, int steps, hipStream_t s) {
  return step(s, [=] { count(B) = count(A) + steps; });
}
hipError_t launch_bgk_d2q9(int, const void* A, void* B, const Layout&, const Grid&, double, const Force&, bool, double*, hipStream_t s) { return take(A, B, 1, s); }
hipError_t launch_bgk_d3q27(int, const void* A, void* B, const Layout&, const Grid&, double, const Force&, bool, double*, hipStream_t s) { return take(A, B, 1, s); }
hipError_t launch_bgk_d2q9_aa(int, bool, void* A, const Layout&, const Grid&, double, const Force&, bool, double*, hipStream_t s) { return take(A, A, 1, s); }
hipError_t launch_bgk_d3q27_aa(int, bool, void* A, const Layout&, const Grid&, double, const Force&, bool, double*, hipStream_t s) { return take(A, A, 1, s); }
hipError_t launch_bgk_d2q9_multi(int, const void* A, void* B, const Layout&, bool, double, const Force&, bool, int steps, hipStream_t s) { return take(A, B, steps, s); }
hipError_t launch_bgk_d3q27_pair(const void* A, void* B, const Layout&, const Pair3Shape&, double, hipStream_t s) { return take(A, B, 2, s); }
hipError_t launch_bgk_d2q9_red(int, const void* A, void* B, const Layout&, const Grid&, double, bool, float, float, double*, hipStream_t s) { return take(A, B, 1, s); }
hipError_t launch_bgk_d2q9_mlp(const void* A, void* B, const Layout&, const Grid&, double, bool, const float*, double, unsigned long long*, double*, hipStream_t s) { return take(A, B, 1, s); }
hipError_t launch_ddf(int, bool, bool pull, const void* A, void* B, const Layout&, const Grid&, const DdfParams&, float, float, double*, void*, int* records, hipStream_t s) {
  if (records) record_room = *records;
  if (records) *records = 32;
  return pull ? take(A, B, 1, s) : put(s, [=] { count(B) = count(A); });
}
hipError_t launch_ddf3(int, bool, bool pull, const void* A, void* B, const Layout&, const Grid&, const DdfParams&, double*, void*, double*, int* records, hipStream_t s) {
  if (records) *records = 32;
  return pull ? take(A, B, 1, s) : put(s, [=] { count(B) = count(A); });
}
hipError_t launch_ddf_pair(int, bool, const void* A, void* B, const Layout&, const DdfParams&, const PairShape&, hipStream_t s) { return take(A, B, 2, s); }

static hipError_t init(const double* rho, void* A, const Layout& L, hipStream_t s) {
  const size_t n = (size_t)L.nodes();
  return put(s, [=] {
    uploaded.assign(rho, rho + n);
    count(A) = 0;
  });
}
hipError_t launch_init_bgk(int, int, const double* rho, const double*, void* A, const Layout& L, bool, double, const Force&, hipStream_t s) { return init(rho, A, L, s); }
hipError_t launch_init_bgk_red(const double* rho, const double*, void* A, const Layout& L, hipStream_t s) { return init(rho, A, L, s); }
hipError_t launch_init_ddf(int, const double* rho, const double*, const double*, void* A, const Layout& L, const DdfParams&, hipStream_t s) { return init(rho, A, L, s); }
hipError_t launch_init_ddf3(int, const double* rho, const double*, const double*, void* A, const Layout& L, const DdfParams&, hipStream_t s) { return init(rho, A, L, s); }

// every read-out value is the steps of the state plus a tag of its place
static hipError_t fill(const void* A, double* out, size_t n, double tag, hipStream_t s) {
  return put(s, [=] {
    const double c = (double)count(A);
    for (size_t i = 0; i < n; ++i) out[i] = c + tag + (double)(i % 4099) / 8192.0;
  });
}
hipError_t launch_moments_bgk(int, int D, const void* A, const Layout& L, int, bool, const Force&, double* rho, double* u, hipStream_t s) {
  // the state is read before any of the outputs is written, as one kernel over many nodes may
  const size_t n = (size_t)L.nodes();
  return put(s, [=] {
    const double c = (double)count(A);
    for (size_t i = 0; i < (1 + (size_t)D) * n; ++i) (i < n ? rho[i] : u[i - n]) = c + (double)(i % 4099) / 8192.0;
  });
}
hipError_t launch_moments_bgk_red(const void* A, const Layout& L, double* rho, double* u, hipStream_t s) { return launch_moments_bgk(0, 2, A, L, 0, false, Force{}, rho, u, s); }
hipError_t launch_moments_ddf(int, const void* A, const Layout& L, const DdfParams&, double* rho, double* u, double* T, double*, hipStream_t s) {
  (void)fill(A, T, (size_t)L.nodes(), 0.0, s);
  return launch_moments_bgk(0, 2, A, L, 0, false, Force{}, rho, u, s);
}
hipError_t launch_moments_ddf3(int, const void* A, const Layout& L, const DdfParams&, double* rho, double* u, double* T, double*, hipStream_t s) {
  (void)fill(A, T, (size_t)L.nodes(), 0.0, s);
  return launch_moments_bgk(0, 3, A, L, 0, false, Force{}, rho, u, s);
}
hipError_t launch_decode_f(int, int, int i, const void* A, const Layout& L, int, bool, double* f, hipStream_t s) { return fill(A, f, (size_t)L.nodes(), 1000.0 * i, s); }
hipError_t launch_decode_ddf(int, int, int i, const void* A, const Layout& L, const DdfParams&, float, double* f, hipStream_t s) { return fill(A, f, (size_t)L.nodes(), 1000.0 * i, s); }
hipError_t launch_decode_bgk_red(int, int i, const void* A, const Layout& L, float, double* f, hipStream_t s) { return fill(A, f, (size_t)L.nodes(), 1000.0 * i, s); }
hipError_t launch_ddf_rest_state(const DdfParams&, double* out, hipStream_t s) { return put(s, [=] { std::memset(out, 0, 18 * 8); }); }
hipError_t launch_ddf3_rest_state(const DdfParams&, double* out, hipStream_t s) { return put(s, [=] { std::memset(out, 0, 54 * 8); }); }
hipError_t launch_diag_finalize(const double*, int, double t, double* out, hipStream_t s) {
  return put(s, [=] {
    out[0] = t;
    for (int k = 1; k < 6; ++k) out[k] = 0.0;
  });
}
hipError_t launch_field_totals(int, const double*, const double*, const double*, int64_t, bool, double*, int, double* out, hipStream_t s) { return put(s, [=] { std::memset(out, 0, 48); }); }
hipError_t launch_harvest(const void*, const Layout&, bool, int, double, const int64_t*, int64_t, float*, float*, hipStream_t) { return hipSuccess; }
hipError_t launch_mlp_grad(const float*, const float*, int64_t, int64_t, int, const float*, float*, hipStream_t) { return hipSuccess; }
hipError_t launch_mlp_reduce_adam(const float*, int, float*, float*, float*, float*, float*, bool, float, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_mlp_forward(const float*, int64_t, const float*, float*, hipStream_t) { return hipSuccess; }
}  // namespace lbm

#include "host_copy.h"

#include <algorithm>
#include <cstring>
#include <mutex>
#include <thread>

namespace lbm {

// Staging memory of the process: pinning it takes milliseconds, so a slab that no copy uses waits
// here for the next one, of any object. At most two wait, and the last object to go frees them.
namespace {
std::mutex g_mutex;
int g_objects = 0;
std::vector<HostCopy::Slab> g_idle;
constexpr size_t kMaxIdle = 2;
}  // namespace

HostCopy::HostCopy() {
  std::lock_guard<std::mutex> lock(g_mutex);
  ++g_objects;
}

HostCopy::~HostCopy() {
  for (hipEvent_t e : ev_) (void)hipEventDestroy(e);
  std::vector<Slab> drop;
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    if (--g_objects == 0) drop.swap(g_idle);
  }
  for (const Slab& s : drop) (void)hipHostFree(s.p);
}

bool HostCopy::take(size_t bytes, Slab& slab) {
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    for (size_t i = 0; i < g_idle.size(); ++i)
      if (g_idle[i].bytes >= bytes) {
        slab = g_idle[i];
        g_idle.erase(g_idle.begin() + i);
        return true;
      }
  }
  void* p = nullptr;
  if (hipHostMalloc(&p, bytes, hipHostMallocPortable) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  slab = {static_cast<char*>(p), bytes};
  return true;
}

void HostCopy::give(const Slab& slab) {
  Slab drop = slab;
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    if (g_idle.size() < kMaxIdle) {
      g_idle.push_back(slab);
      return;
    }
    for (Slab& s : g_idle)
      if (s.bytes < drop.bytes) std::swap(s, drop);  // the largest stay
  }
  (void)hipHostFree(drop.p);
}

bool HostCopy::events(int n) {
  while ((int)ev_.size() < n) {
    hipEvent_t e;
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    ev_.push_back(e);
  }
  return true;
}

// Chunks w, w + threads, ... of the concatenated pieces.
hipError_t HostCopy::lane(int w, const Shape& sh, char* slab, const HostPiece* p, int n,
                          size_t total, hipMemcpyKind kind, int device, hipStream_t s) {
  hipError_t e = hipSetDevice(device);  // a thread's current device is its own
  // fn(piece, offset in it, length, offset in the chunk) for the parts of chunk c
  auto parts = [&](size_t c, auto&& fn) {
    const size_t a = c * sh.chunk, b = std::min(total, a + sh.chunk);
    size_t base = 0;
    for (int i = 0; i < n; base += p[i++].bytes) {
      const size_t lo = std::max(a, base), hi = std::min(b, base + p[i].bytes);
      if (lo < hi) fn(p[i], lo - base, hi - lo, lo - a);
    }
  };
  auto buf = [&](int k) { return slab + (2 * w + k) * sh.chunk; };
  auto fetch = [&](size_t c, int k) {
    parts(c, [&](const HostPiece& q, size_t off, size_t len, size_t at) {
      if (e == hipSuccess)
        e = hipMemcpyAsync(buf(k) + at, static_cast<const char*>(q.src) + off, len,
                           hipMemcpyDeviceToHost, s);
    });
    if (e == hipSuccess) e = hipEventRecord(ev_[2 * w + k], s);
  };
  const size_t chunks = (total + sh.chunk - 1) / sh.chunk;
  int k = 0;
  if (kind == hipMemcpyHostToDevice) {
    for (size_t c = w; c < chunks && e == hipSuccess; c += sh.threads, k ^= 1) {
      if (c >= (size_t)w + 2 * sh.threads) e = hipEventSynchronize(ev_[2 * w + k]);
      if (e != hipSuccess) break;
      parts(c, [&](const HostPiece& q, size_t off, size_t len, size_t at) {
        std::memcpy(buf(k) + at, static_cast<const char*>(q.src) + off, len);
        if (e == hipSuccess)
          e = hipMemcpyAsync(static_cast<char*>(q.dst) + off, buf(k) + at, len, kind, s);
      });
      if (e == hipSuccess) e = hipEventRecord(ev_[2 * w + k], s);
    }
    return e;
  }
  if ((size_t)w < chunks && e == hipSuccess) fetch(w, 0);
  for (size_t c = w; c < chunks && e == hipSuccess; c += sh.threads, k ^= 1) {
    if (c + sh.threads < chunks) fetch(c + sh.threads, k ^ 1);
    if (e == hipSuccess) e = hipEventSynchronize(ev_[2 * w + k]);
    if (e != hipSuccess) break;
    parts(c, [&](const HostPiece& q, size_t off, size_t len, size_t at) {
      std::memcpy(static_cast<char*>(q.dst) + off, buf(k) + at, len);
    });
  }
  return e;
}

hipError_t HostCopy::copy(const HostPiece* p, int n, hipMemcpyKind kind, int device,
                          hipStream_t s) {
  size_t total = 0;
  for (int i = 0; i < n; ++i) total += p[i].bytes;
  const size_t mib = (size_t)1 << 20;
  const Shape sh = total > 256 * mib ? Shape{6, 4 * mib}
                                     : Shape{4, total > 16 * mib ? 2 * mib : mib};
  Slab slab;
  if (total <= 4 * mib || !events(2 * sh.threads) || !take(2 * sh.threads * sh.chunk, slab)) {
    hipError_t e = hipSuccess;
    for (int i = 0; i < n && e == hipSuccess; ++i)
      e = hipMemcpyAsync(p[i].dst, p[i].src, p[i].bytes, kind, s);
    const hipError_t es = hipStreamSynchronize(s);
    return e != hipSuccess ? e : es;
  }
  hipError_t res[8];
  std::thread th[8];
  int started = 1;  // this thread takes lane 0, and the lanes that get no thread
  try {
    for (; started < sh.threads; ++started)
      th[started] = std::thread([&, w = started] { res[w] = lane(w, sh, slab.p, p, n, total, kind, device, s); });
  } catch (...) {
  }
  res[0] = lane(0, sh, slab.p, p, n, total, kind, device, s);
  for (int w = started; w < sh.threads; ++w) res[w] = lane(w, sh, slab.p, p, n, total, kind, device, s);
  for (int w = 1; w < started; ++w) th[w].join();
  // also after an error: nothing still writes to the staging memory when it is given back
  hipError_t e = hipStreamSynchronize(s);
  give(slab);
  for (int w = 0; w < sh.threads; ++w)
    if (res[w] != hipSuccess) e = res[w];
  return e;
}

}  // namespace lbm

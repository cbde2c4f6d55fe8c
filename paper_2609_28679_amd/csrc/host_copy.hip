#include "host_copy.h"

#include <algorithm>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>

namespace lbm {

// Staging memory of the process: pinning it takes milliseconds, so a slab that no copy uses waits
// here for the next one, of any object. At most two wait, and the last object to go frees them.
namespace {
std::mutex g_mutex;
int g_objects = 0;
constexpr int kMaxIdle = 2;
HostCopy::Slab g_idle[kMaxIdle];
}  // namespace

HostCopy::HostCopy() {
  std::lock_guard<std::mutex> lock(g_mutex);
  ++g_objects;
}

HostCopy::~HostCopy() {
  for (int i = 0; i < events_; ++i) (void)hipEventDestroy(ev_[i]);
  Slab drop[kMaxIdle];
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    if (--g_objects == 0)
      for (int i = 0; i < kMaxIdle; ++i) std::swap(drop[i], g_idle[i]);
  }
  for (const Slab& d : drop)
    if (d.p) (void)hipHostFree(d.p);
}

bool HostCopy::take(size_t bytes, Slab& slab) {
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    for (Slab& idle : g_idle)
      if (idle.bytes >= bytes) {
        slab = idle;
        idle = Slab{};
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
    for (Slab& idle : g_idle)
      if (idle.bytes < drop.bytes) std::swap(idle, drop);  // the largest stay
  }
  if (drop.p) (void)hipHostFree(drop.p);
}

// An event belongs to the device that is current when it is made, which need not be the stream's:
// a program with several GPUs may call with another one current, and keeps it.
bool HostCopy::events(int n, hipStream_t s) {
  if (events_ >= n) return true;
  int device = 0, current = 0;
  if (hipStreamGetDevice(s, &device) != hipSuccess || hipGetDevice(&current) != hipSuccess ||
      (device != current && hipSetDevice(device) != hipSuccess)) {
    (void)hipGetLastError();
    return false;
  }
  while (events_ < n && hipEventCreateWithFlags(&ev_[events_], hipEventDisableTiming) == hipSuccess)
    ++events_;
  if (events_ < n) (void)hipGetLastError();
  if (device != current) (void)hipSetDevice(current);
  return events_ >= n;
}

namespace {
// One staged copy under way. The calling thread alone works on the stream, whose handle may mean
// another queue in another thread (hipStreamPerThread): it queues the copies of the chunks between
// device and buffers in order, chunk c in buffer c mod `buffers`, with an event behind each. The
// movers take the chunks in order and move them between the buffers and the caller's memory.
struct Staging {
  const HostPiece* p;
  int n;
  hipMemcpyKind kind;
  hipStream_t s;
  char* slab;
  hipEvent_t* ev;
  size_t chunk, total, chunks;
  int buffers;

  std::mutex m;
  std::condition_variable cv;
  size_t next = 0;        // next chunk that a mover takes
  size_t queued = 0;      // chunks whose device copy is on the stream
  size_t moved[kMaxBuffers] = {};  // per buffer: chunks the movers have moved through it
  hipError_t err = hipSuccess;

  bool upload() const { return kind == hipMemcpyHostToDevice; }
  char* buffer(size_t c) const { return slab + c % buffers * chunk; }
  // fn(piece, offset in it, length, offset in the chunk) for the parts of chunk c
  template <typename Fn>
  void parts(size_t c, Fn&& fn) const {
    const size_t a = c * chunk, b = std::min(total, a + chunk);
    size_t base = 0;
    for (int i = 0; i < n; base += p[i++].bytes) {
      const size_t lo = std::max(a, base), hi = std::min(b, base + p[i].bytes);
      if (lo < hi) fn(p[i], lo - base, hi - lo, lo - a);
    }
  }
  void fail(hipError_t e) {
    std::lock_guard<std::mutex> lock(m);
    if (err == hipSuccess) err = e;
    cv.notify_all();
  }
  // Waits until ready() or an error; false after an error.
  template <typename Fn>
  bool wait(Fn&& ready) {
    std::unique_lock<std::mutex> lock(m);
    cv.wait(lock, [&] { return err != hipSuccess || ready(); });
    return err == hipSuccess;
  }

  void move() {
    for (;;) {
      size_t c;
      {
        std::lock_guard<std::mutex> lock(m);
        if (err != hipSuccess || next >= chunks) return;
        c = next++;
      }
      // read-out: the chunk has arrived; upload: the buffer's last chunk has left
      const size_t ahead = upload() ? (size_t)buffers : 0;
      if (c >= ahead) {
        if (!wait([&] { return queued > c - ahead; })) return;
        const hipError_t e = hipEventSynchronize(ev[c % buffers]);
        if (e != hipSuccess) return fail(e);
      }
      parts(c, [&](const HostPiece& q, size_t off, size_t len, size_t at) {
        if (upload())
          std::memcpy(buffer(c) + at, static_cast<const char*>(q.src) + off, len);
        else
          std::memcpy(static_cast<char*>(q.dst) + off, buffer(c) + at, len);
      });
      std::lock_guard<std::mutex> lock(m);
      ++moved[c % buffers];
      cv.notify_all();
    }
  }

  void queue() {
    for (size_t c = 0; c < chunks; ++c) {
      // read-out: the buffer is free again; upload: it holds the chunk
      const size_t uses = c / buffers + (upload() ? 1 : 0);
      if (!wait([&] { return moved[c % buffers] >= uses; })) return;
      hipError_t e = hipSuccess;
      parts(c, [&](const HostPiece& q, size_t off, size_t len, size_t at) {
        if (e != hipSuccess) return;
        e = upload() ? hipMemcpyAsync(static_cast<char*>(q.dst) + off, buffer(c) + at, len, kind, s)
                     : hipMemcpyAsync(buffer(c) + at, static_cast<const char*>(q.src) + off, len, kind, s);
      });
      if (e == hipSuccess) e = hipEventRecord(ev[c % buffers], s);
      if (e != hipSuccess) return fail(e);
      std::lock_guard<std::mutex> lock(m);
      queued = c + 1;
      cv.notify_all();
    }
  }
};
}  // namespace

// Ordinary memory of the caller, which the device cannot reach by itself.
static bool pageable(const void* host) {
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, host) == hipSuccess) return a.type == hipMemoryTypeUnregistered;
  (void)hipGetLastError();
  return true;
}

hipError_t HostCopy::copy(const HostPiece* p, int n, hipMemcpyKind kind, hipStream_t s) {
  size_t total = 0;
  bool stage = true;
  for (int i = 0; i < n; ++i) {
    total += p[i].bytes;
    stage = stage && pageable(kind == hipMemcpyHostToDevice ? p[i].src : p[i].dst);
  }
  const size_t mib = (size_t)1 << 20;
  const int movers = total > 256 * mib ? 6 : 4;
  const size_t chunk = total > 256 * mib ? 4 * mib : (total > 16 * mib ? 2 * mib : mib);
  const int buffers = 2 * movers;
  std::thread th[kMaxBuffers / 2];
  Slab slab;
  if (stage && total > (kind == hipMemcpyHostToDevice ? 64 : 8) * mib && events(buffers, s) &&
      take(buffers * chunk, slab)) {
    Staging g{p, n, kind, s, slab.p, ev_, chunk, total, (total + chunk - 1) / chunk, buffers};
    int started = 0;
    try {
      for (; started < movers; ++started) th[started] = std::thread([&g] { g.move(); });
    } catch (...) {  // fewer threads
    }
    if (started) g.queue();
    for (int i = 0; i < started; ++i) th[i].join();
    // also after an error: nothing still uses the staging memory when it is given back
    const hipError_t e = hipStreamSynchronize(s);
    give(slab);
    if (started) return g.err != hipSuccess ? g.err : e;
  }
  hipError_t e = hipSuccess;
  for (int i = 0; i < n && e == hipSuccess; ++i)
    e = hipMemcpyAsync(p[i].dst, p[i].src, p[i].bytes, kind, s);
  const hipError_t es = hipStreamSynchronize(s);
  return e != hipSuccess ? e : es;
}

}  // namespace lbm

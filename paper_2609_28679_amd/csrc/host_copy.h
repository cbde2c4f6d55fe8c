// Copies of read-outs and initial fields between device and host.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace lbm {

constexpr int kMaxBuffers = 12;  // staging buffers of one copy

struct HostPiece {
  void* dst;        // one of them device memory, the other the caller's
  const void* src;
  size_t bytes;
};

// Copies through pinned staging buffers, several host threads moving them on to the caller's memory
// (or from it, for the initial fields). A plain copy to pageable memory runs through one staging path
// of the runtime on one host thread, which also takes the page faults of newly allocated memory:
// about 10 GB/s, 20-30% of an output interval. Measured for a whole read-out (moments kernel, totals
// and copy): 4096^2 D2Q9, 403 MB, 40 -> 10.5 ms; 2048^2, 101 MB, 10 -> 3.5 ms; 12.4 MB 0.74 -> 0.57.
//
// Threads x chunk by the bytes of the call, two chunks in flight per thread, from sweeps of 1-16
// threads and 1-8 MiB: above 256 MiB 6 x 4 MiB (403 MB: 10.5 ms; 4 x 2: 11.4, 3 x 4: 12.2, 1 x 4:
// 29), above 16 MiB 4 x 2 MiB (101 MB: 3.2 ms, the first call 5.7; 6 x 4: 3.1, the first call 7.6,
// most of it the pinned allocation), above 8 MiB 4 x 1 MiB. What stays with the plain copy:
//   - read-outs up to 8 MiB (4.3 MB: 0.29 ms, staged 0.30 and with a new slab 0.33);
//   - initial fields, whose pages exist, up to 64 MiB (a context made while no other lives, plain /
//     staged: 4.3 MB 0.53 / 0.67 ms, 12.4 MB 1.37 / 1.53, 16.6 MB 1.92 / 2.23, 43 MB 4.9 / 4.7, but
//     7.1 for the first of a process; 72 MB 8.6 / 8.1, 101 MB 11.6 / 10.5, 216 MB 30 / 25);
//   - memory of the caller that is pinned itself, which the device reaches at the link's rate (12 /
//     101 / 403 MB: 0.27 / 1.9 / 7.4 ms, staged 0.55 / 2.6 / 9.1).
// An object copies for one caller at a time like the context that owns it; several objects may copy
// at once. The staging memory is shared by the objects of the process, one slab per copy under way.
class HostCopy {
 public:
  struct Slab {
    char* p = nullptr;
    size_t bytes = 0;
  };
  HostCopy();
  HostCopy(const HostCopy&) = delete;
  HostCopy& operator=(const HostCopy&) = delete;
  ~HostCopy();
  // Copies the pieces after the work queued on s, from the device or to it; returns when done.
  hipError_t copy(const HostPiece* p, int n, hipMemcpyKind kind, hipStream_t s);

 private:
  static bool take(size_t bytes, Slab& slab);
  static void give(const Slab& slab);
  bool events(int n, hipStream_t s);
  hipEvent_t ev_[kMaxBuffers];  // one per staging buffer
  int events_ = 0;
};

}  // namespace lbm

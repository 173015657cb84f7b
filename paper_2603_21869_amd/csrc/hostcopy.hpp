// Copies between a program's own (pageable) arrays and the device, and within
// host memory, on several threads.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include <functional>

namespace nfvm {

// Whoever may call the copies below while it exists (a grid, a server).  The
// pinned staging areas that calls leave behind and the helper threads are kept
// while there is one and end with the last.
struct StagingUser {
  StagingUser();
  ~StagingUser();
  StagingUser(const StagingUser&) = delete;
  StagingUser& operator=(const StagingUser&) = delete;
};

// n arrays of `bytes` each through one device buffer dev, in order on stream s:
//   to_host: for each f, fill(f) enqueues what writes dev; dev goes to dst[f]
//   to_device: for each f, src[f] goes to dev; use(f) enqueues what reads it
// Complete when they return (to_device: with a synchronisation of s).  Large
// calls are moved in chunks, by a kernel or (engine) by the copy engine.
void to_host(const void* dev, void* const* dst, int n, size_t bytes, hipStream_t s, bool engine,
             const std::function<void(int)>& fill);
void to_device(void* dev, const void* const* src, int n, size_t bytes, hipStream_t s, bool engine,
               const std::function<void(int)>& use);

// dst[f][0 .. bytes) = src[f][...] for f < n (null dst: left out).
void host_copy(void* const* dst, const void* const* src, int n, size_t bytes);

}  // namespace nfvm

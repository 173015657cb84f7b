// Transfers of a grid's fields.  The runtime's copy of pageable memory stages
// through its own pinned buffers with one host thread, which also takes the
// page faults of a result array's first touch: 10 GB/s into fresh arrays and
// 27 GB/s out of touched ones (940 MB in seven arrays), against 32 and 48 here,
// where a kernel moves chunks between the device and a pinned ring and up to
// COPY_THREADS threads between the ring and the arrays.  (Not the copy engine:
// the driver clears freed device memory with it, 34 ms per GB, and chunks then
// wait for it.  Fields of 7.5 GB into a grid made after a 22 GB one was freed:
// 377 ms through the engine, 228 with the runtime's copy, 155 here.  Beside
// other lanes' kernels, in a server, the copy kernel waits for compute units
// and the engine is the better one all the same: 256 requests on 9 slots 2116
// Mcell-steps/s with it, 2050 with the kernel, 1845 with the runtime's copy.)
#include "hostcopy.hpp"

#include <pthread.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <condition_variable>
#include <exception>
#include <memory>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "engine.hpp"

namespace nfvm {
namespace {

// 940 MB into the device / into fresh arrays: chunks of 1 MiB 22.3 / 35.2 ms (a
// launch and its event have a fixed cost), 2 MiB 19.7 / 29.7, 4 MiB 18.6 / 26.7
// at twice the pinned memory; four slots 26.9 / 46.3; one thread 33.9 / 68.7,
// two 19.7 / 39.6, six 19.7 / 31.4.
constexpr size_t CHUNK = 2 << 20;
constexpr int SLOTS = 8;         // chunks of a staging area
constexpr int COPY_THREADS = 4;  // the calling one and its helpers
constexpr int STAGE_KEEP = 2;    // idle areas kept, 16 MiB each
// Below this many bytes a call stays with the runtime's copy: it moves them
// about as fast, and a grid need not make a ring and threads for them.  Out of
// the device into fresh arrays, with the ring / without: 3.7 MB 0.2 / 0.3 ms,
// 8.3 MB 1.0 / 2.0, 14.7 MB 1.7 / 3.5.
constexpr size_t STAGE_MIN = 4 << 20;
// An area and the helper threads cost 0.2 ms to make and end, for every grid of
// a program that has one grid at a time (they end with the last).  Without an
// idle area, a call of fewer than STAGE_COLD bytes makes one only once such
// calls have moved STAGE_WARM bytes.  Made and freed / made, read and freed, a
// mixed-precision grid of 48^3 cells (6.2 MB of fields) 2.55 / 2.83 ms with the
// ring, 2.50 / 2.94 without; 64 x 48 x 48 (8.3 MB) 2.77 / 3.08, 2.85 / 3.48;
// 64^3 (14.7 MB) 2.97 / 3.62, 3.09 / 4.17.
constexpr size_t STAGE_COLD = 15 << 19, STAGE_WARM = 16 << 20;

struct Staging {
  unsigned char* p = nullptr;
  unsigned char* d = nullptr;  // as the device addresses it
  hipEvent_t ev[SLOTS] = {};
  int device = 0;
  ~Staging() {
    for (hipEvent_t e : ev)
      if (e) (void)hipEventDestroy(e);
    if (p) (void)hipHostFree(p);
  }
};

class Job;
struct Pool {
  std::mutex mu;
  std::unique_ptr<Staging> idle[STAGE_KEEP];
  int users = 0;
  size_t cold = 0;  // bytes of calls that found no idle area, since the first user
  // helper threads, their calls' jobs; helpers of an older `gen` end
  std::vector<std::thread> helpers;
  std::vector<Job*> jobs;
  std::condition_variable cv;
  unsigned gen = 0;
};
void pool_in_child();
Pool*& pool_of_process() {
  static Pool* p = [] {
    (void)pthread_atfork(nullptr, nullptr, pool_in_child);
    return new Pool();  // (never destroyed: grids may outlive static objects)
  }();
  return p;
}
Pool& pool() { return *pool_of_process(); }
// A forked child has its parent's users but none of its threads: it goes on
// with a pool of its own, as the parent's may be locked and its condition
// variable counts waiters that the child does not have.
void pool_in_child() {
  Pool* p = new (std::nothrow) Pool();
  if (!p) return;
  p->users = pool().users;
  pool_of_process() = p;
}

// A staging area for a call of `bytes` on stream s, or null where none is worth
// making or can be had (s on another device than the current one among them:
// events belong to a device).
std::unique_ptr<Staging> take_staging(hipStream_t s, size_t bytes) {
  int dev = 0, sdev = 0;
  if (hipGetDevice(&dev) != hipSuccess || (s && hipStreamGetDevice(s, &sdev) != hipSuccess)) {
    (void)hipGetLastError();
    return nullptr;
  }
  if (s && sdev != dev) return nullptr;
  {
    std::lock_guard<std::mutex> lk(pool().mu);
    for (std::unique_ptr<Staging>& st : pool().idle)
      if (st && st->device == dev) return std::move(st);
    pool().cold += bytes;
    if (bytes < STAGE_COLD && pool().cold < STAGE_WARM) return nullptr;
  }
  std::unique_ptr<Staging> st(new (std::nothrow) Staging());
  if (!st) return nullptr;
  st->device = dev;
  bool ok = hipHostMalloc((void**)&st->p, CHUNK * SLOTS,
                          hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess &&
            hipHostGetDevicePointer((void**)&st->d, st->p, 0) == hipSuccess;
  for (int i = 0; ok && i < SLOTS; ++i)
    ok = hipEventCreateWithFlags(&st->ev[i], hipEventDisableTiming) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    return nullptr;
  }
  return st;
}
void give_staging(std::unique_ptr<Staging> st) {
  std::lock_guard<std::mutex> lk(pool().mu);
  if (pool().users == 0) return;
  for (std::unique_ptr<Staging>& slot : pool().idle)
    if (!slot) {
      slot = std::move(st);
      return;
    }
}

// Memory the runtime does not know: not pinned, not the device's.  (Arrays it
// knows go to its own copy, which reaches them directly.)
bool pageable(const void* p) {
  hipPointerAttribute_t a;
  memset(&a, 0, sizeof a);
  if (hipPointerGetAttributes(&a, p) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return a.type == hipMemoryTypeUnregistered;
}
bool all_pageable(const void* const* p, int n) {
  for (int f = 0; f < n; ++f)
    if (!pageable(p[f])) return false;
  return true;
}
// Result arrays that share memory are written one after the other.
bool disjoint(void* const* p, int n, size_t bytes) {
  for (int f = 0; f < n; ++f)
    for (int h = 0; h < f; ++h) {
      const uintptr_t a = (uintptr_t)p[f], b = (uintptr_t)p[h];
      if (a && b && (a > b ? a - b : b - a) < bytes) return false;
    }
  return true;
}

// The chunks of n arrays of `bytes` each, one array after the other.
struct Chunks {
  size_t bytes, per, total;
  Chunks(int n, size_t b) : bytes(b), per((b + CHUNK - 1) / CHUNK), total(per * n) {}
  int array(size_t i) const { return (int)(i / per); }
  size_t off(size_t i) const { return i % per * CHUNK; }
  size_t len(size_t i) const { return std::min(CHUNK, bytes - off(i)); }
};

// A reference to a function of a chunk's index (a std::function of more than
// two captures would allocate).
class ChunkCopy {
 public:
  template <class F>
  explicit ChunkCopy(const F& f)
      : call_([](const void* p, size_t i) { (*(const F*)p)(i); }), f_(&f) {}
  void operator()(size_t i) const { call_(f_, i); }

 private:
  void (*call_)(const void*, size_t);
  const void* f_;
};

// One call's host copies, chunk by chunk.  The calling thread copies too and
// helpers take chunks only while they run, so a call never waits for a helper
// to be scheduled: on a machine whose processors are busy (the spinning
// threads of an OpenMP program's last parallel loop) it goes on alone.
class Job {
 public:
  Job(size_t chunks, const ChunkCopy& copy)
      : n_(chunks), copy_(copy), done_(chunks, 0) {
    std::lock_guard<std::mutex> lk(pool().mu);
    start_helpers();
    pool().jobs.push_back(this);
  }
  ~Job() {  // (also after an error: helpers finish the chunks they hold)
    std::unique_lock<std::mutex> lk(pool().mu);
    auto& v = pool().jobs;
    v.erase(std::find(v.begin(), v.end(), this));
    cv_.wait(lk, [&] { return active_ == 0; });
  }
  Job(const Job&) = delete;
  Job& operator=(const Job&) = delete;

  // chunks below `upto` may be copied
  void ready(size_t upto) {
    {
      std::lock_guard<std::mutex> lk(pool().mu);
      ready_ = std::max(ready_, std::min(upto, n_));
    }
    pool().cv.notify_all();
  }
  // copies one chunk, if there is one to take
  bool copy_one() {
    std::unique_lock<std::mutex> lk(pool().mu);
    return take(lk);
  }
  size_t copied() {
    std::lock_guard<std::mutex> lk(pool().mu);
    return copied_;
  }
  // waits for more than `seen` chunks, in order from the first, to be copied
  size_t wait_copied(size_t seen) {
    std::unique_lock<std::mutex> lk(pool().mu);
    cv_.wait(lk, [&] { return copied_ > seen; });
    return copied_;
  }

 private:
  bool take(std::unique_lock<std::mutex>& lk) {
    if (next_ >= ready_) return false;
    const size_t i = next_++;
    ++active_;
    lk.unlock();
    copy_(i);
    lk.lock();
    --active_;
    done_[i] = 1;
    while (copied_ < n_ && done_[copied_]) ++copied_;
    cv_.notify_all();
    return true;
  }
  static void help(unsigned gen) {
    std::unique_lock<std::mutex> lk(pool().mu);
    while (pool().gen == gen) {
      bool any = false;
      for (size_t j = 0; !any && j < pool().jobs.size(); ++j) any = pool().jobs[j]->take(lk);
      if (!any) pool().cv.wait(lk);
    }
  }
  static void start_helpers() {  // (with the pool locked)
    const size_t hw = std::thread::hardware_concurrency();
    try {
      while (pool().helpers.size() + 1 < std::min<size_t>(COPY_THREADS, hw))
        pool().helpers.emplace_back(help, pool().gen);
    } catch (const std::exception&) {  // as many as there are
    }
  }

  const size_t n_;
  const ChunkCopy copy_;
  std::vector<char> done_;
  size_t ready_ = 0, next_ = 0, copied_ = 0;
  int active_ = 0;
  std::condition_variable cv_;
};

// Null where there is no host memory for it.
std::unique_ptr<Job> make_job(size_t chunks, const ChunkCopy& copy) {
  try {
    return std::unique_ptr<Job>(new Job(chunks, copy));
  } catch (const std::bad_alloc&) {
    return nullptr;
  }
}

// fn(), which launches kernels: a launch that fails leaves its code as the
// thread's last error, which is taken here, before an event query that is not
// ready overwrites it.  (An error from before the call is not the call's.)
template <class F>
void launched(F&& fn) {
  const bool clean = hipPeekAtLastError() == hipSuccess;
  fn();
  if (clean) NFVM_CK(hipGetLastError());
}

void copy_values(const void* src, void* dst, size_t bytes, hipStream_t s) {
  launch_copy_values((const double*)src, (double*)dst, (int)(bytes / sizeof(double)), s);
}
// Whether a call's device buffer can be copied by it.
bool copyable(const void* dev, size_t bytes) {
  return (uintptr_t)dev % 16 == 0 && bytes % sizeof(double) == 0;
}

// Whether the device has passed an event.
bool ended(hipEvent_t e) {
  const hipError_t r = hipEventQuery(e);
  if (r == hipErrorNotReady) {
    (void)hipGetLastError();
    return false;
  }
  NFVM_CK(r);
  return true;
}

// The staging area of one call: back in the pool when the stream is idle.
struct StagingCall {
  std::unique_ptr<Staging> st;
  hipStream_t s;
  bool idle = false;
  StagingCall(hipStream_t stream, size_t bytes) : st(take_staging(stream, bytes)), s(stream) {}
  ~StagingCall() {
    if (!st) return;
    if (!idle) (void)hipStreamSynchronize(s);  // (after an error)
    give_staging(std::move(st));
  }
};

}  // namespace

StagingUser::StagingUser() {
  std::lock_guard<std::mutex> lk(pool().mu);
  ++pool().users;
}
StagingUser::~StagingUser() {
  std::unique_ptr<Staging> old[STAGE_KEEP];
  std::vector<std::thread> ended;
  {
    std::lock_guard<std::mutex> lk(pool().mu);
    if (--pool().users > 0) return;
    pool().cold = 0;
    std::swap(old, pool().idle);
    ended.swap(pool().helpers);
    ++pool().gen;
  }
  pool().cv.notify_all();
  for (std::thread& t : ended) t.join();
}

void to_host(const void* dev, void* const* dst, int n, size_t bytes, hipStream_t s, bool engine,
             const std::function<void(int)>& fill) {
  if (n * bytes >= STAGE_MIN && copyable(dev, bytes) && all_pageable(dst, n) &&
      disjoint(dst, n, bytes)) {
    StagingCall c(s, n * bytes);
    const Chunks ch(n, bytes);
    unsigned char* const ring = c.st ? c.st->p : nullptr;
    const auto copy = [&](size_t i) {
      memcpy((unsigned char*)dst[ch.array(i)] + ch.off(i), ring + i % SLOTS * CHUNK, ch.len(i));
    };
    if (const std::unique_ptr<Job> job = ring ? make_job(ch.total, ChunkCopy(copy)) : nullptr) {
      size_t issued = 0, arrived = 0, copied = 0;  // device copies begun, ended; chunks done
      while (copied < ch.total) {
        for (; issued < ch.total && issued < copied + SLOTS; ++issued) {
          if (ch.off(issued) == 0) launched([&] { fill(ch.array(issued)); });
          const unsigned char* from = (const unsigned char*)dev + ch.off(issued);
          const size_t slot = issued % SLOTS * CHUNK, len = ch.len(issued);
          if (engine)
            NFVM_CK(hipMemcpyAsync(ring + slot, from, len, hipMemcpyDeviceToHost, s));
          else
            launched([&] { copy_values(from, c.st->d + slot, len, s); });
          NFVM_CK(hipEventRecord(c.st->ev[issued % SLOTS], s));
        }
        size_t now = arrived;
        while (now < issued && ended(c.st->ev[now % SLOTS])) ++now;
        if (now > arrived) job->ready(arrived = now);
        if (job->copy_one()) {
        } else if (arrived < issued) {
          NFVM_CK(hipEventSynchronize(c.st->ev[arrived % SLOTS]));
          job->ready(++arrived);
        } else {
          job->wait_copied(copied);  // (helpers hold the rest)
        }
        copied = job->copied();
      }
      c.idle = true;
      return;
    }
  }
  for (int f = 0; f < n; ++f) {
    launched([&] { fill(f); });
    NFVM_CK(hipMemcpyAsync(dst[f], dev, bytes, hipMemcpyDeviceToHost, s));
    NFVM_CK(hipStreamSynchronize(s));
  }
}

void to_device(void* dev, const void* const* src, int n, size_t bytes, hipStream_t s, bool engine,
               const std::function<void(int)>& use) {
  if (n * bytes >= STAGE_MIN && copyable(dev, bytes) && all_pageable(src, n)) {
    StagingCall c(s, n * bytes);
    const Chunks ch(n, bytes);
    unsigned char* const ring = c.st ? c.st->p : nullptr;
    const auto copy = [&](size_t i) {
      memcpy(ring + i % SLOTS * CHUNK, (const unsigned char*)src[ch.array(i)] + ch.off(i),
             ch.len(i));
    };
    if (const std::unique_ptr<Job> job = ring ? make_job(ch.total, ChunkCopy(copy)) : nullptr) {
      size_t issued = 0, freed = 0, copied = 0;  // device copies begun, ended; chunks in the ring
      job->ready(SLOTS);
      while (issued < ch.total) {
        for (; issued < copied; ++issued) {
          unsigned char* to = (unsigned char*)dev + ch.off(issued);
          const size_t slot = issued % SLOTS * CHUNK, len = ch.len(issued);
          if (engine)
            NFVM_CK(hipMemcpyAsync(to, ring + slot, len, hipMemcpyHostToDevice, s));
          else
            launched([&] { copy_values(c.st->d + slot, to, len, s); });
          NFVM_CK(hipEventRecord(c.st->ev[issued % SLOTS], s));
          if (ch.off(issued) + ch.len(issued) == bytes)
            launched([&] { use(ch.array(issued)); });
        }
        size_t now = freed;
        while (now < issued && ended(c.st->ev[now % SLOTS])) ++now;
        if (now > freed) job->ready((freed = now) + SLOTS);
        if (issued < ch.total && !job->copy_one()) {
          if (freed + SLOTS == copied) {  // every slot waits for its device copy
            NFVM_CK(hipEventSynchronize(c.st->ev[freed % SLOTS]));
            job->ready(++freed + SLOTS);
          } else {
            job->wait_copied(copied);  // (helpers hold the next)
          }
        }
        copied = job->copied();
      }
      NFVM_CK(hipStreamSynchronize(s));
      c.idle = true;
      return;
    }
  }
  for (int f = 0; f < n; ++f) {
    NFVM_CK(hipMemcpyAsync(dev, src[f], bytes, hipMemcpyHostToDevice, s));
    launched([&] { use(f); });
    NFVM_CK(hipStreamSynchronize(s));
  }
}

void host_copy(void* const* dst, const void* const* src, int n, size_t bytes) {
  const Chunks ch(n, bytes);
  const auto copy = [&](size_t i) {
    const int f = ch.array(i);
    if (dst[f])
      memcpy((unsigned char*)dst[f] + ch.off(i), (const unsigned char*)src[f] + ch.off(i),
             ch.len(i));
  };
  if (n * bytes >= STAGE_MIN && disjoint(dst, n, bytes)) {
    if (const std::unique_ptr<Job> job = make_job(ch.total, ChunkCopy(copy))) {
      job->ready(ch.total);
      while (job->copy_one()) {
      }
      for (size_t c = job->copied(); c < ch.total;) c = job->wait_copied(c);
      return;
    }
  }
  for (size_t i = 0; i < ch.total; ++i) copy(i);
}

}  // namespace nfvm

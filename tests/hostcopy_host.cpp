// The field transfers (csrc/hostcopy.cpp) on the CPU: a runtime whose streams
// run each call at once, whose event queries say "not ready" the first time,
// and whose last error behaves as HIP's (kept until read, overwritten by a
// query that is not ready); allocations of the calling thread can be made to
// fail.  Usage: hostcopy_host CASE; ends with 0 if the case
// holds, with a message and 1 if not.
#include "../paper_2603_21869_amd/csrc/hostcopy.cpp"

#include <stdio.h>
#include <stdlib.h>
#include <sys/wait.h>
#include <unistd.h>

namespace fake {
thread_local hipError_t last = hipSuccess;
int pins = 0;    // pinned areas made
int copies = 0;  // calls of the runtime's copy
struct Event {
  bool asked = false;
};
hipError_t set(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
// the allocation of this thread that fails: 0 the next one (-1: none)
thread_local long deny = -1;
thread_local bool denied = false;
}  // namespace fake

void* operator new(size_t n) {
  if (fake::deny >= 0 && fake::deny-- == 0) {
    fake::denied = true;
    throw std::bad_alloc();
  }
  void* p = malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept {
  try {
    return operator new(n);
  } catch (const std::bad_alloc&) {
    return nullptr;
  }
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {
hipError_t hipGetLastError() {
  const hipError_t e = fake::last;
  fake::last = hipSuccess;
  return e;
}
hipError_t hipPeekAtLastError() { return fake::last; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { return *d = 0, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  a->type = hipMemoryTypeUnregistered;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  ++fake::pins;
  *p = malloc(n);
  return *p ? hipSuccess : fake::set(hipErrorOutOfMemory);
}
hipError_t hipHostGetDevicePointer(void** d, void* p, unsigned) { return *d = p, hipSuccess; }
hipError_t hipHostFree(void* p) { return free(p), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)calloc(1, sizeof(fake::Event));
  return *e ? hipSuccess : fake::set(hipErrorOutOfMemory);
}
hipError_t hipEventDestroy(hipEvent_t e) { return free(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  ((fake::Event*)e)->asked = false;
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  bool& asked = ((fake::Event*)e)->asked;
  if (asked) return hipSuccess;
  asked = true;
  return fake::set(hipErrorNotReady);
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  ++fake::copies;
  memcpy(d, s, n);
  return hipSuccess;
}
}

void nfvm::launch_copy_values(const double* src, double* dst, int n, hipStream_t) {
  memcpy(dst, src, n * sizeof(double));
}

namespace {
using namespace nfvm;

int fail(const char* what) {
  printf("FAILED: %s\n", what);
  return 1;
}

// n arrays of `count` values with a value of their own at every place
struct Arrays {
  size_t count;
  std::vector<std::vector<double>> a;
  Arrays(int n, size_t c, bool fill) : count(c), a(n, std::vector<double>(c, -1.0)) {
    if (fill)
      for (int f = 0; f < n; ++f)
        for (size_t i = 0; i < c; ++i) a[f][i] = value(f, i);
  }
  static double value(int f, size_t i) { return f * 1e9 + (double)i; }
  bool right() const {
    for (size_t f = 0; f < a.size(); ++f)
      for (size_t i = 0; i < count; ++i)
        if (a[f][i] != value((int)f, i)) return false;
    return true;
  }
  std::vector<void*> ptrs() {
    std::vector<void*> p;
    for (auto& v : a) p.push_back(v.data());
    return p;
  }
};

// seven arrays through one "device" buffer
struct Seven {
  Arrays h;
  std::vector<double> dev;
  std::vector<void*> p;
  Seven(size_t count, bool fill) : h(7, count, fill), dev(count), p(h.ptrs()) {}
  size_t bytes() const { return h.count * sizeof(double); }
  // (get: the kernel that writes dev; set: the one that reads it)
  void get(int bad = -1, bool engine = false) {
    to_host(dev.data(), p.data(), 7, bytes(), nullptr, engine, [&](int f) {
      if (f == bad) {
        fake::set(hipErrorInvalidConfiguration);  // a launch that fails leaves its code
        return;
      }
      for (size_t i = 0; i < h.count; ++i) dev[i] = Arrays::value(f, i);
    });
  }
  bool set(int bad = -1, bool engine = false) {
    bool ok = true;
    to_device(dev.data(), p.data(), 7, bytes(), nullptr, engine, [&](int f) {
      if (f == bad) {
        fake::set(hipErrorInvalidConfiguration);
        return;
      }
      for (size_t i = 0; i < h.count; ++i) ok = ok && dev[i] == Arrays::value(f, i);
    });
    return ok;
  }
};

template <class F>
bool throws(F&& f) {
  try {
    f();
  } catch (const Error& e) {
    (void)hipGetLastError();
    return e.st == NFVM_E_DEVICE;
  }
  return false;
}

// A kernel launch that fails inside a transfer is an error of the call, through
// the ring and through the runtime's copy, whichever array it belongs to; an
// error that the thread had before is not.
int launch_error() {
  StagingUser user;
  for (size_t count : {1000u, 300001u}) {
    for (int bad : {0, 3, 6}) {
      Seven g(count, false), s(count, true);
      if (!throws([&] { g.get(bad); })) return fail("a field that was not unpacked was returned");
      if (!throws([&] { s.set(bad); })) return fail("a field that was not packed was accepted");
      if (!throws([&] { g.get(bad, true); }) || !throws([&] { s.set(bad, true); }))
        return fail("a failed launch beside the copy engine");
    }
    Seven g(count, false);
    fake::last = hipErrorInvalidValue;
    g.get();
    if (!g.h.right()) return fail("fields after an older error");
    fake::last = hipSuccess;
    Seven s(count, true);
    if (!s.set()) return fail("fields loaded");
  }
  return 0;
}

// A transfer that finds no host memory for its own bookkeeping does without:
// it neither fails nor throws (it runs inside C entry points and, for a served
// request, at the end of a worker's round), whichever allocation fails.
template <class F>
int each_allocation(F&& f) {
  for (int n = 0; n < 1000; ++n) {
    StagingUser user;  // (the ring and the threads are made anew)
    fake::denied = false;
    if (!f(n)) return fail("a copy without memory");
    if (!fake::denied) return 0;
  }
  return fail("the allocations never ended");
}
template <class F>
bool denying(int n, F&& f) {
  bool ok = true;
  fake::deny = n;
  try {
    f();
  } catch (const std::exception&) {
    ok = false;
  }
  fake::deny = -1;
  return ok;
}

int no_memory() {
  const size_t count = 300001, bytes = count * sizeof(double);
  int rc = each_allocation([&](int n) {
    Seven g(count, false);
    const std::function<void(int)> fill = [&g](int f) {
      for (size_t i = 0; i < g.h.count; ++i) g.dev[i] = Arrays::value(f, i);
    };
    return denying(n, [&] { to_host(g.dev.data(), g.p.data(), 7, bytes, nullptr, false, fill); }) &&
           g.h.right();
  });
  if (rc) return rc;
  rc = each_allocation([&](int n) {
    Seven s(count, true);
    bool ok = true;
    struct {
      Seven& s;
      bool& ok;
    } c{s, ok};
    const std::function<void(int)> use = [&c](int f) {
      for (size_t i = 0; i < c.s.h.count; ++i) c.ok = c.ok && c.s.dev[i] == Arrays::value(f, i);
    };
    return denying(n, [&] { to_device(s.dev.data(), s.p.data(), 7, bytes, nullptr, false, use); }) && ok;
  });
  if (rc) return rc;
  return each_allocation([&](int n) {
    Arrays a(7, count, true), b(7, count, false);
    const auto pa = a.ptrs(), pb = b.ptrs();
    return denying(n, [&] { host_copy(pb.data(), pa.data(), 7, bytes); }) && b.right();
  });
}

// A forked child has none of its parent's helper threads: transfers there work,
// and so does the end of the last user (which must not wait for them).
int forked_child() {
  StagingUser* user = new StagingUser();
  Seven g(300001, false);
  g.get();
  usleep(200000);  // (the helpers are idle)
  const pid_t pid = fork();
  if (pid == 0) {
    alarm(20);
    Seven c(300001, false);
    c.get();
    const bool ok = c.h.right();
    delete user;
    StagingUser next;
    Seven d(300001, false);
    d.get();
    _exit(ok && d.h.right() ? 0 : 1);
  }
  int st = 0;
  if (pid < 0 || waitpid(pid, &st, 0) != pid) return fail("fork");
  delete user;
  if (!WIFEXITED(st)) return fail("the child did not end by itself");
  return WEXITSTATUS(st) ? fail("the child's fields") : 0;
}

// A grid that is made, read and freed does not pay for a pinned area that its
// fields are too small to earn back; one that lives on gets an area, and so
// does the first transfer of a large one.
int short_lived() {
  const size_t count = 48 * 48 * 48;  // 6.2 MB in seven arrays
  for (int grid = 0; grid < 3; ++grid) {
    StagingUser user;
    Seven s(count, true), g(count, false);
    if (!s.set()) return fail("fields loaded");
    g.get();
    if (!g.h.right()) return fail("fields read");
  }
  if (fake::pins) return fail("an area was pinned for a short-lived grid");
  StagingUser user;
  for (int call = 0; call < 10; ++call) {
    Seven g(count, false);
    g.get();
    if (!g.h.right()) return fail("fields read again");
  }
  if (fake::pins != 1) return fail("areas of a grid that lives on");
  {
    StagingUser other;
    Seven g(64 * 64 * 64, false);  // 14.7 MB: with the area that is there
    g.get();
  }
  if (fake::pins != 1) return fail("an idle area was not taken");
  return 0;
}
// Large transfers pass through the copy engine, which the driver keeps busy
// after a large allocation is freed, only where that is asked for.
int no_copy_engine() {
  StagingUser user;
  for (bool engine : {false, true}) {
    Seven s(300001, true), g(300001, false);
    if (!s.set(-1, engine)) return fail("fields loaded");
    g.get(-1, engine);
    if (!g.h.right()) return fail("fields read");
    if (engine != (fake::copies > 0)) return fail("the way of the chunks");
  }
  return 0;
}
int large_first() {
  StagingUser user;
  Seven s(64 * 64 * 64, true);
  if (!s.set()) return fail("fields loaded");
  return fake::pins == 1 ? 0 : fail("areas of a large grid");
}
}  // namespace

int main(int argc, char** argv) {
  const std::string c = argc > 1 ? argv[1] : "";
  if (c == "launch_error") return launch_error();
  if (c == "no_memory") return no_memory();
  if (c == "forked_child") return forked_child();
  if (c == "short_lived") return short_lived();
  if (c == "no_copy_engine") return no_copy_engine();
  if (c == "large_first") return large_first();
  return fail("unknown case");
}

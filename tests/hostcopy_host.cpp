// The field transfers (csrc/hostcopy.cpp) on the CPU: a runtime whose streams
// run each call at once, whose event queries say "not ready" the first time,
// and whose last error behaves as HIP's (kept until read, overwritten by a
// query that is not ready).  Usage: hostcopy_host CASE; ends with 0 if the case
// holds, with a message and 1 if not.
#include "../paper_2603_21869_amd/csrc/hostcopy.cpp"

#include <stdio.h>
#include <stdlib.h>

namespace fake {
thread_local hipError_t last = hipSuccess;
int pins = 0;  // pinned areas made
struct Event {
  bool asked = false;
};
hipError_t set(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
}  // namespace fake

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
  memcpy(d, s, n);
  return hipSuccess;
}
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
  void get(int bad = -1) {
    to_host(dev.data(), p.data(), 7, bytes(), nullptr, [&](int f) {
      if (f == bad) {
        fake::set(hipErrorInvalidConfiguration);  // a launch that fails leaves its code
        return;
      }
      for (size_t i = 0; i < h.count; ++i) dev[i] = Arrays::value(f, i);
    });
  }
  bool set(int bad = -1) {
    bool ok = true;
    to_device(dev.data(), p.data(), 7, bytes(), nullptr, [&](int f) {
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
}  // namespace

int main(int argc, char** argv) {
  const std::string c = argc > 1 ? argv[1] : "";
  if (c == "launch_error") return launch_error();
  return fail("unknown case");
}

// A stand-in for the HIP runtime and the library's kernels, so that the host
// side of the C ABI (api.cpp) runs on a CPU.  Device memory is host memory.
// Kernels and what follows them on their stream are kept until something waits
// for that stream, and only a while after; a copy on an idle stream is made at
// once.  So a missing wait or a transfer on another stream shows as wrong data.
// Two devices; the per-thread stream is another one in every host thread.
//
// A state's step count stands for the lattice: the first eight bytes of a
// state hold how many steps it has seen.
#include <chrono>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "internal.h"
#include "marker_args.h"

namespace {

struct Stream {
  int device = 0;
  std::deque<std::function<void()>> work;
  long long done = 0, enqueued = 0;
};
struct Event {
  int device;
  Stream* on = nullptr;
  long long at = 0;
};

std::recursive_mutex mu;
thread_local int current = 0;
thread_local Stream own[2];
Stream null_stream[2];
long long pinned = 0, pinned_most = 0;
std::map<void*, size_t> pins;
std::vector<std::string> calls;
int copies = 0;
std::string fail_kind;
int fail_after = 0;

Stream* find(hipStream_t s) {
  if (!s) return null_stream[current].device = current, &null_stream[current];
  if (s == hipStreamPerThread) return own[current].device = current, &own[current];
  return reinterpret_cast<Stream*>(s);
}

void a_while() { std::this_thread::sleep_for(std::chrono::milliseconds(3)); }

void run_to(Stream* s, long long at) {
  while (s->done < at && !s->work.empty()) {
    auto f = std::move(s->work.front());
    s->work.pop_front();
    ++s->done;
    f();
  }
}

void enqueue(hipStream_t st, std::function<void()> f) {
  Stream* s = find(st);
  s->work.push_back(std::move(f));
  ++s->enqueued;
}

// Enqueue a launch of the named kind, or fail as asked for by host_fail.
hipError_t launch(const std::string& kind, const std::string& what, hipStream_t st, std::function<void()> f) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (find(st)->device != current) return hipErrorInvalidDevice;
  if (kind == fail_kind && fail_after-- == 0) return fail_kind.clear(), hipErrorLaunchFailure;
  calls.push_back(what);
  enqueue(st, std::move(f));
  return hipSuccess;
}

int64_t seen(const void* state) {
  int64_t v;
  std::memcpy(&v, state, 8);
  return v;
}
void set(void* state, int64_t v) { std::memcpy(state, &v, 8); }

}  // namespace

extern "C" {

// ------------------------------------------------------------ for the tests
__attribute__((visibility("default"))) void* host_stream(int device) { return new Stream{device, {}, 0, 0}; }
__attribute__((visibility("default"))) void host_device(int device) { current = device; }
__attribute__((visibility("default"))) int host_current() { return current; }
__attribute__((visibility("default"))) long long host_pinned(int most) { return most ? pinned_most : pinned; }
__attribute__((visibility("default"))) void host_fail(const char* kind, int after) {
  fail_kind = kind;
  fail_after = after;
}
__attribute__((visibility("default"))) int host_copies() { return copies; }
// The launches since the last call, one a line.
__attribute__((visibility("default"))) const char* host_calls() {
  static std::string text;
  std::lock_guard<std::recursive_mutex> l(mu);
  text.clear();
  for (auto& c : calls) text += c + "\n";
  calls.clear();
  return text.c_str();
}

// ----------------------------------------------------------------- runtime
hipError_t hipGetDevice(int* d) { return *d = current, hipSuccess; }
hipError_t hipSetDevice(int d) { return d < 0 || d > 1 ? hipErrorInvalidDevice : (current = d, hipSuccess); }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { return *d = find(s)->device, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "an error of the stand-in"; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (fail_kind == "pinned" && fail_after-- <= 0) return hipErrorOutOfMemory;   // from then on
  *p = std::malloc(n);
  pins[*p] = n;
  pinned += (long long)n;
  pinned_most = pinned > pinned_most ? pinned : pinned_most;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::lock_guard<std::recursive_mutex> l(mu);
  pinned -= (long long)pins[p];
  pins.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(new Event{current});
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { return delete reinterpret_cast<Event*>(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t ev, hipStream_t st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  Event* e = reinterpret_cast<Event*>(ev);
  Stream* s = find(st);
  if (e->device != s->device) return hipErrorInvalidHandle;   // an event belongs to one device
  e->on = s;
  e->at = s->enqueued;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t ev) {
  a_while();
  std::lock_guard<std::recursive_mutex> l(mu);
  Event* e = reinterpret_cast<Event*>(ev);
  if (e->on) run_to(e->on, e->at);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t st) {
  a_while();
  std::lock_guard<std::recursive_mutex> l(mu);
  Stream* s = find(st);
  run_to(s, s->enqueued);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  ++copies;
  if (find(st)->work.empty())
    std::memcpy(to, from, n);
  else
    enqueue(st, [=] { std::memcpy(to, from, n); });
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* to, int v, size_t n, hipStream_t st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  enqueue(st, [=] { std::memset(to, v, n); });
  return hipSuccess;
}
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) {
  std::lock_guard<std::recursive_mutex> l(mu);
  std::memcpy(to, from, n);
  return hipSuccess;
}

}  // extern "C"

// ------------------------------------------------------------------ kernels
namespace ibmk {

size_t marker_span_lds(int) { return 0; }
hipError_t scratch_address(int, void**) { return hipErrorNotSupported; }
int pair_blocks(const Geo& g, int ylen) {
  return ((g.nx + kBlockX - 1) / kBlockX) * ((g.nz + kPairRows - 1) / kPairRows) * ((g.ny + ylen - 1) / ylen);
}

hipError_t launch_factor(const MarkerArgs* const*, const void* const*, int n, int, hipStream_t s) {
  return launch("factor", "factor " + std::to_string(n), s, [] {});
}
hipError_t launch_markers(int, const MarkerArgs* const*, const void* const*, const void* const*,
                          unsigned long long alt, int n, hipStream_t s) {
  return launch("markers", "markers " + std::to_string(n) + " alt " + std::to_string(alt), s, [] {});
}
hipError_t launch_near(bool, bool, const CollideArgs* const*, const void* const*, const void* const* src,
                       void* const* dst, int n, hipStream_t s) {
  return launch("near", "near " + std::to_string(n), s, [] {});
}

static hipError_t advance(const char* kind, int steps, const void* const* src, void* const* dst, int n,
                          hipStream_t s) {
  std::vector<const void*> a(src, src + n);
  std::vector<void*> b(dst, dst + n);
  return launch(kind, std::string(kind) + " " + std::to_string(n), s, [=] {
    for (int k = 0; k < n; ++k) set(b[k], seen(a[k]) + steps);
  });
}
hipError_t launch_collide(int, bool, bool, bool, bool, const CollideArgs* const*, const void* const*,
                          const void* const* src, void* const* dst, int n, hipStream_t s) {
  return advance("collide", 1, src, dst, n, s);
}
hipError_t launch_pair(bool, bool, bool, const CollideArgs* const*, const void* const*, const void* const* src,
                       void* const* dst, const int*, int n, hipStream_t s) {
  return advance("pair", 2, src, dst, n, s);
}

hipError_t launch_ghost(int, const Geo&, const Phys&, void*, hipStream_t s) { return launch("ghost", "ghost", s, [] {}); }
hipError_t launch_init_eq(int, const Geo&, const double*, const double*, void* dst, hipStream_t s) {
  return launch("init_eq", "init_eq", s, [=] { set(dst, 0); });
}
// rho and u: the index of the value, modulo a prime
hipError_t launch_moments(int, const Geo& g, const Phys&, const void*, float* out, hipStream_t s) {
  const size_t n = 4 * (size_t)g.nx * g.ny * g.nz;
  return launch("moments", "moments", s, [=] {
    for (size_t i = 0; i < n; ++i) out[i] = (float)(i % 65521);
  });
}
hipError_t launch_mass_reduce(const double*, int, double, double*, long long, hipStream_t s) {
  return launch("mass", "mass", s, [] {});
}
// FP32 states only
static float* cell_row(const Geo& g, const void* state, int q, size_t row) {
  return static_cast<float*>(const_cast<void*>(state)) + ((row + 1) * kQ + q) * (size_t)g.px;
}
hipError_t launch_pack(int, const Geo& g, const float* dense, int q0, int nq, void* state, hipStream_t s) {
  return launch("pack", "pack", s, [=] {
    for (int q = 0; q < nq; ++q)
      for (size_t r = 0; r < (size_t)g.ny * g.nz; ++r)
        std::memcpy(cell_row(g, state, q0 + q, r), dense + ((size_t)q * g.ny * g.nz + r) * g.nx, g.nx * sizeof(float));
  });
}
hipError_t launch_unpack(int, const Geo& g, const void* state, int q0, int nq, float* dense, hipStream_t s) {
  return launch("unpack", "unpack", s, [=] {
    for (int q = 0; q < nq; ++q)
      for (size_t r = 0; r < (size_t)g.ny * g.nz; ++r)
        std::memcpy(dense + ((size_t)q * g.ny * g.nz + r) * g.nx, cell_row(g, state, q0 + q, r), g.nx * sizeof(float));
  });
}
hipError_t launch_export(const double*, long long, long long, int, int, const int*, double* out, hipStream_t s) {
  return launch("export", "export", s, [=] { std::memset(out, 0, (kExportDoubles + 1) * 8); });
}

}  // namespace ibmk

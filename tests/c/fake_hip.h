// A HIP runtime and kernel launchers on the CPU, for checks of the host runtime
// (hc_runtime.cpp) alone: device memory is host memory, a launch runs nothing but
// checks that every buffer it names is allocated and large enough, and work that
// was enqueued on another stream and not waited for is remembered, so that a
// launch which touches the same memory is reported.  Allocations can be made to
// fail; as in HIP, a failed call stays the thread's last error until it is read.
#pragma once

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "hc_internal.h"
#include "hc_plan.h"

namespace fake {

struct Write {               // enqueued and not waited for
  void *base;                // allocation it writes
  hipStream_t stream;
};

inline std::map<uintptr_t, size_t> live;
inline std::vector<Write> pending;
inline std::vector<std::string> faults;
inline hipError_t last = hipSuccess;
inline int fail_malloc_in = 0;        // n: the n-th hipMalloc from now fails
inline hipError_t fail_memcpy = hipSuccess;   // the next hipMemcpy fails with this
inline int fail_new_in = 0;           // n: the n-th host allocation from now throws
inline int quiet = 0;                 // > 0: not the runtime's own allocations
struct Quiet {
  Quiet() { ++quiet; }
  ~Quiet() { --quiet; }
};
inline int launches = 0, syncs = 0;
inline bool dense_wide = false;       // of the last dense launch
inline int dense_units = 0;           // its units with work

inline hipError_t ret(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
inline hipError_t take_last() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
inline void fault(const std::string &what) { faults.push_back(what); }   // (under a Quiet)

// base of the live allocation that holds [p, p + bytes), or null
inline void *owner(const void *p, size_t bytes) {
  const uintptr_t a = (uintptr_t)p;
  auto it = live.upper_bound(a);
  if (it == live.begin()) return nullptr;
  --it;
  return a + bytes <= it->first + it->second ? (void *)it->first : nullptr;
}

inline void touch(const char *what, const void *p, size_t bytes, hipStream_t s, bool write) {
  Quiet q;
  void *base = owner(p, bytes);
  if (!base) {
    char buf[160];
    std::snprintf(buf, sizeof buf, "%s: %p + %zu is not allocated", what, p, bytes);
    return fault(buf);
  }
  for (const Write &w : pending)
    if (w.base == base && w.stream != s)
      fault(std::string(what) + ": memory that another stream may still write");
  if (write) pending.push_back({base, s});
}

inline void done(hipStream_t s) {
  Quiet q;
  std::vector<Write> left;
  for (const Write &w : pending)
    if (w.stream != s) left.push_back(w);
  pending.swap(left);
}

}  // namespace fake

void *operator new(size_t n) {
  if (fake::quiet == 0 && fake::fail_new_in > 0 && --fake::fail_new_in == 0) throw std::bad_alloc();
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
  fake::Quiet q;
  if (fake::fail_malloc_in > 0 && --fake::fail_malloc_in == 0) return fake::ret(hipErrorOutOfMemory);
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  fake::live[(uintptr_t)*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  fake::Quiet q;
  fake::pending.clear();                      // waits for the device
  if (!p) return hipSuccess;
  if (!fake::live.erase((uintptr_t)p)) fake::fault("hipFree of memory that is not allocated");
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n) {   // on the null stream, not waited for
  fake::touch("hipMemset", p, n, nullptr, true);
  std::memset(p, v, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t s) {
  fake::touch("hipMemsetAsync", p, n, s, true);
  std::memset(p, v, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  if (fake::fail_memcpy != hipSuccess) {
    const hipError_t e = fake::fail_memcpy;
    fake::fail_memcpy = hipSuccess;
    return fake::ret(e);
  }
  fake::done(nullptr);                        // ordered after the null stream, and waited for
  fake::touch("hipMemcpy", d, n, nullptr, false);
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { fake::pending.clear(); ++fake::syncs; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { fake::done(s); return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetLastError() { return fake::take_last(); }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
}

namespace hc {
using fake::touch;

hipError_t launch_dense(const DenseArgs &a, int d, DenseRole, hipStream_t s) {
  ++fake::launches;
  fake::dense_wide = a.wide_waves;
  touch("dense work list", a.units, a.n_units * sizeof(DenseUnit), s, false);
  if (!fake::owner(a.units, a.n_units * sizeof(DenseUnit))) return fake::take_last();
  fake::dense_units = 0;
  int64_t slots = 0;
  for (int i = 0; i < a.n_units; ++i) {
    const DenseUnit &u = a.units[i];
    if (u.head < 0) continue;
    ++fake::dense_units;
    slots = std::max<int64_t>(slots, u.slot + 1);
    const int64_t end = u.kv0 + (u.kv1 - u.kv0 + kKTile - 1) / kKTile * kKTile;
    touch("dense keys", u.k, end * d * 2, s, false);
    touch("dense values", u.v, end * d * 2, s, false);
  }
  if (slots) touch("dense partials", a.part, slots * partial_floats(d) * 4, s, true);
  return fake::take_last();
}
hipError_t launch_spatial(const SpatialArgs &a, int d, SpatialRole, hipStream_t s) {
  ++fake::launches;
  const size_t keys = (size_t)a.n_sp * a.head_stride + a.geo.lead * d;
  touch("Spatial keys", a.k - a.geo.lead * d, (keys + a.geo.lead * d) * 2, s, false);
  touch("Spatial values", a.v - a.geo.lead * d, (keys + a.geo.lead * d) * 2, s, false);
  if (a.n_split > 1) {
    const size_t rows = (size_t)a.n_split * a.n_sp * a.L;
    touch("Spatial partials", a.part, rows * d * 4, s, true);
    touch("Spatial maxima and sums", a.part_ml, rows * 8, s, true);
  }
  return fake::take_last();
}
hipError_t launch_merge(const CombineArgs &c, const SpatialArgs &a, int d, hipStream_t s) {
  ++fake::launches;
  if (c.n_items > 0) {
    touch("merge list", c.items, c.n_items * sizeof(CombineItem), s, false);
    int64_t slots = 0;
    for (int i = 0; i < c.n_items; ++i) slots = std::max<int64_t>(slots, c.items[i].slot0 + c.items[i].n_slots);
    touch("merged partials", c.part, slots * partial_floats(d) * 4, s, false);
  }
  if (a.n_split > 1) touch("merged Spatial partials", a.part, (size_t)a.n_split * a.n_sp * a.L * d * 4, s, false);
  return fake::take_last();
}
hipError_t launch_scatter(ScatterArgs a, int, hipStream_t s) {
  ++fake::launches;
  for (const uint16_t *p : {a.k_sd, a.v_sd, a.k_g, a.v_g, a.k_sp, a.v_sp})
    if (p) touch("scatter", p, 1, s, true);
  return fake::take_last();
}
hipError_t launch_stats(const StatsArgs &a, hipStream_t s) {
  ++fake::launches;
  touch("token statistics", a.cos_sp, (size_t)a.n_heads * a.L * 8, s, true);
  return fake::take_last();
}
hipError_t launch_cls_reduce(const ClsReduceArgs &a, hipStream_t s) {
  ++fake::launches;
  touch("head statistics", a.out, (size_t)a.n_heads * 48, s, true);
  std::memset(a.out, 0, (size_t)a.n_heads * 48);
  return fake::take_last();
}
hipError_t static_scratch(int, void **p) {
  fake::Quiet q;
  static void *mem = nullptr;
  if (!mem) {
    mem = std::aligned_alloc(256, kStaticScratchBytes);
    fake::live[(uintptr_t)mem] = kStaticScratchBytes;
  }
  *p = mem;
  return hipSuccess;
}
hipError_t launch_static_plan(const StaticPlan &p, DenseUnit *units, CombineItem *comb, hipStream_t s) {
  ++fake::launches;
  const int nu = static_n_units(p), nc = static_n_comb(p);
  if (nu) touch("static work list", units, nu * sizeof(DenseUnit), s, true);
  if (nc) touch("static merge list", comb, nc * sizeof(CombineItem), s, true);
  for (int i = 0; i < nu; ++i) units[i] = static_dense_unit(p, i);
  for (int i = 0; i < nc; ++i) comb[i] = static_comb_item(p, i);
  return fake::take_last();
}
}  // namespace hc

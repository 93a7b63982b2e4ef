// Checks of the host runtime (hc_runtime.cpp) against a HIP runtime on the CPU
// (fake_hip.h): what is left after an allocation or a copy failed, and the order
// of work on different streams.  One check per run, named by the first argument.
#include <cstdint>

#include "fake_hip.h"
#include "headcast.h"

static int failures = 0;
#define CHECK(cond, ...)                                   \
  do {                                                     \
    if (!(cond)) {                                         \
      std::printf("FAIL %s:%d: ", __FILE__, __LINE__);     \
      std::printf(__VA_ARGS__);                            \
      std::printf("\n");                                   \
      ++failures;                                          \
    }                                                      \
  } while (0)

namespace {

const hipStream_t kA = (hipStream_t)0x100, kB = (hipStream_t)0x200;

// device memory of the caller: only its address is used
alignas(16) unsigned char caller_mem[64];

hc_config config(int layers, int heads) {
  hc_config c;
  hc_config_default(&c);
  c.n_layers = layers; c.n_heads = heads; c.head_dim = 64;
  c.grid_h = 8; c.grid_w = 12; c.frames_per_block = 2; c.window_blocks = 4;
  c.spatial_radius = 1; c.proxy_radius = 1;
  return c;
}

struct Ctx {
  hc_ctx *c = nullptr;
  explicit Ctx(const hc_config &cfg) {
    fake::fail_malloc_in = 0;
    CHECK(hc_create(&cfg, 0, &c) == HC_OK, "hc_create");
  }
  ~Ctx() { hc_destroy(c); }
  hc_status set(int layer, const std::vector<uint8_t> &t, hipStream_t s = nullptr) {
    return hc_set_head_types(c, layer, t.data(), 3, caller_mem, caller_mem, s);
  }
  hc_status attend(int layer, const std::vector<uint8_t> &t, hipStream_t s = nullptr) {
    return hc_attention(c, layer, caller_mem, t.data(), (float *)caller_mem, s);
  }
  hc_status attend_static(int layer, const std::vector<uint8_t> &t, hipStream_t s = nullptr) {
    return hc_attention_static(c, layer, caller_mem, t.data(), (float *)caller_mem, s);
  }
  hc_status append(int layer, hipStream_t s = nullptr) {
    return hc_append_block(c, layer, 3, caller_mem, caller_mem, s);
  }
  hc_status classify(int layer, std::vector<uint8_t> &t, hipStream_t s = nullptr) {
    return hc_classify_heads(c, layer, 3, caller_mem, caller_mem, caller_mem, t.data(), nullptr, s);
  }
};

const std::vector<uint8_t> kFew = {HC_SINK, HC_DUMMY, HC_SPATIAL, HC_GLOBAL};
const std::vector<uint8_t> kMany = {HC_GLOBAL, HC_GLOBAL, HC_GLOBAL, HC_GLOBAL};
const std::vector<uint8_t> kSpatial = {HC_SPATIAL, HC_SPATIAL, HC_SPATIAL, HC_SPATIAL};

// A call that runs out of memory reports it once: the next call, which has
// nothing to do with it, does not find the error again.  The classification
// passes over a failed allocation of the routed work list, and over nothing else.
void errors_are_reported_once() {
  for (int nth = 1; nth <= 4; ++nth) {
    Ctx x(config(2, 4));
    CHECK(x.set(0, kFew) == HC_OK && x.attend(0, kFew) == HC_OK, "first layer");
    fake::fail_malloc_in = nth;
    const hc_status st = x.set(1, kMany);
    fake::fail_malloc_in = 0;
    CHECK(st == HC_OK || st == HC_E_NOMEM, "status %d", st);
    CHECK(x.append(0) == HC_OK, "append after failure %d: %s", nth, hc_last_error(x.c));
  }
  int passed_over = 0;
  for (int nth = 1; nth <= 24; ++nth) {
    Ctx x(config(2, 4));
    CHECK(x.set(0, kFew) == HC_OK, "first layer");
    std::vector<uint8_t> t(4);
    fake::fail_malloc_in = nth;
    const hc_status st = x.classify(1, t);
    passed_over += st == HC_OK && fake::fail_malloc_in == 0;
    fake::fail_malloc_in = 0;
    CHECK(st == HC_OK || st == HC_E_NOMEM, "status %d", st);
    CHECK(x.append(0) == HC_OK, "append after failure %d: %s", nth, hc_last_error(x.c));
    if (st == HC_OK) CHECK(x.attend(1, t) == HC_OK, "layer 1 after failure %d: %s", nth, hc_last_error(x.c));
  }
  CHECK(passed_over > 0, "no failure left the classification without a work list");
  Ctx x(config(2, 4));
  std::vector<uint8_t> t(4);
  CHECK(x.classify(0, t) == HC_OK, "classification");
  fake::fail_memcpy = hipErrorInvalidValue;      // the routed work list's upload
  CHECK(x.classify(1, t) == HC_E_DEVICE, "a failed upload is not passed over");
  CHECK(x.append(0) == HC_OK, "append: %s", hc_last_error(x.c));
}

// A layer that works keeps working when another layer's call runs out of memory
// while it replaces the buffers that all layers share.
void shared_buffers_after_failed_growth() {
  for (const auto &more : {kMany, kSpatial})
    for (int nth = 1; nth <= 6; ++nth) {
      Ctx x(config(2, 4));
      CHECK(x.set(0, kFew) == HC_OK && x.attend(0, kFew) == HC_OK, "first layer");
      fake::fail_malloc_in = nth;
      const hc_status st = x.set(1, more);
      if (st == HC_OK) (void)x.attend(1, more);
      fake::fail_malloc_in = 0;
      CHECK(st == HC_OK || st == HC_E_NOMEM, "status %d", st);
      CHECK(x.attend(0, kFew) == HC_OK, "layer 0 after failure %d: %s", nth, hc_last_error(x.c));
      CHECK(x.set(1, more) == HC_OK && x.attend(1, more) == HC_OK, "layer 1 again");
      CHECK(x.attend(0, kFew) == HC_OK, "layer 0 again");
    }
  for (int nth = 1; nth <= 24; ++nth) {          // the classification's own growth
    hc_config cfg = config(2, 4);
    cfg.theta_sink = cfg.theta_dummy = cfg.theta_spatial = 2.f;   // every head Global
    Ctx x(cfg);
    CHECK(x.set(0, kFew) == HC_OK && x.attend(0, kFew) == HC_OK, "first layer");
    std::vector<uint8_t> t(4);
    fake::fail_malloc_in = nth;
    const hc_status st = x.classify(1, t);
    fake::fail_malloc_in = 0;
    CHECK(st == HC_OK || st == HC_E_NOMEM, "status %d", st);
    CHECK(x.attend(0, kFew) == HC_OK, "layer 0 after failure %d: %s", nth, hc_last_error(x.c));
    if (st == HC_OK) CHECK(x.attend(1, t) == HC_OK, "layer 1 after failure %d", nth);
  }
}

// A table set, or a block appended, on one stream is attended for the first time from
// another; on the same stream nothing is waited for.  Memory that a call clears is clear before the caller's
// stream uses it.
void first_attention_on_another_stream() {
  for (const auto &t : {kFew, kMany}) {
    Ctx x(config(1, 4));
    CHECK(x.set(0, t, kA) == HC_OK && x.attend(0, t, kB) == HC_OK, "%s", hc_last_error(x.c));
    (void)hipDeviceSynchronize();
    CHECK(x.set(0, t, kA) == HC_OK, "%s", hc_last_error(x.c));
    (void)hipDeviceSynchronize();
    CHECK(x.append(0, kB) == HC_OK && x.attend(0, t, kA) == HC_OK, "%s", hc_last_error(x.c));
    (void)hipDeviceSynchronize();
    CHECK(x.set(0, t, kA) == HC_OK, "%s", hc_last_error(x.c));
    const int syncs = fake::syncs;
    CHECK(x.attend(0, t, kA) == HC_OK && fake::syncs == syncs, "%d waits", fake::syncs - syncs);
    CHECK(x.set(0, t, hipStreamPerThread) == HC_OK && x.attend(0, t, hipStreamPerThread) == HC_OK, "per thread");
    CHECK(fake::syncs > syncs + 1, "no wait on hipStreamPerThread");   // one for the kept buffers
    (void)hipDeviceSynchronize();
  }
  // (a layer without dense work has no list to build: its first call only launches)
  Ctx y(config(1, 4));
  CHECK(y.set(0, kSpatial, kA) == HC_OK && y.attend(0, kSpatial, kA) == HC_OK, "%s", hc_last_error(y.c));
  (void)hipDeviceSynchronize();
  Ctx x(config(1, 4));
  std::vector<uint8_t> t(4);
  CHECK(x.classify(0, t, kA) == HC_OK && x.attend(0, t, kB) == HC_OK, "%s", hc_last_error(x.c));
  (void)hipDeviceSynchronize();
}

// Small Global windows are one unit per query tile, except where other partials of
// the layer are merged anyway: two-block Sink/Dummy heads, split Spatial heads.
void small_windows() {
  const std::vector<uint8_t> dense = {HC_GLOBAL, HC_SINK, HC_DUMMY, HC_GLOBAL};
  for (int sd = 1; sd <= 2; ++sd)
    for (const auto &t : {dense, kMany, kFew}) {
      hc_config cfg = config(1, 4);
      cfg.frames_per_block = 1;                   // 96 tokens: one query tile, six key tiles
      cfg.sd_blocks = sd;
      Ctx x(cfg);
      int n[4] = {};
      for (uint8_t k : t) ++n[k];
      const int n_sd = n[HC_SINK] + n[HC_DUMMY];
      const int per_global = (sd == 2 && n_sd > 0) || n[HC_SPATIAL] > 0 ? 4 : 1;
      const int want = n[HC_GLOBAL] * per_global + n_sd * sd;
      CHECK(x.set(0, t) == HC_OK && x.attend(0, t) == HC_OK, "%s", hc_last_error(x.c));
      CHECK(fake::dense_units == want, "hc_attention: %d units, not %d", fake::dense_units, want);
      CHECK(x.attend_static(0, t) == HC_OK, "%s", hc_last_error(x.c));
      CHECK(fake::dense_units == want, "hc_attention_static: %d units, not %d", fake::dense_units, want);
    }
}

// No call lets a failed host allocation out: it returns HC_E_NOMEM, and the context
// works on.  (The checks' own vectors are made outside the calls.)
void host_memory() {
  std::vector<uint8_t> labels(4);
  auto failing = [&](const char *what, int nth, auto &&call) -> bool {   // false: no allocation failed
    fake::fail_new_in = nth;
    hc_status st = HC_OK;
    bool threw = false;
    try {
      st = call();
    } catch (const std::bad_alloc &) {
      threw = true;
    }
    const bool failed = fake::fail_new_in == 0;
    fake::fail_new_in = 0;
    CHECK(!threw, "%s: allocation %d thrown across the ABI", what, nth);
    CHECK(st == HC_OK || st == HC_E_NOMEM, "%s: status %d", what, st);
    return failed;
  };
  hc_config cfg = config(2, 4);
  for (int cell = 0; cell <= 4; cell += 4) {
    cfg.spatial_cell = cell;
    for (int nth = 1;; ++nth) {
      hc_ctx *c = nullptr;
      const bool more = failing("hc_create", nth, [&] { return hc_create(&cfg, 0, &c); });
      hc_destroy(c);
      if (!more) break;
    }
  }
  cfg.spatial_cell = 0;
  enum { kSet, kAttend, kStatic, kAppend, kClassify, kCalls };
  const char *names[] = {"hc_set_head_types", "hc_attention", "hc_attention_static", "hc_append_block", "hc_classify_heads"};
  int n[kCalls] = {};
  for (int call = 0; call < kCalls; ++call)
    for (int nth = 1; nth < 400; ++nth) {
      Ctx x(cfg);
      CHECK(x.set(0, kFew) == HC_OK && x.attend(0, kFew) == HC_OK && x.set(1, kMany) == HC_OK, "%s", hc_last_error(x.c));
      const bool more = failing(names[call], nth, [&] {
        switch (call) {
          case kSet: return x.set(1, kFew);
          case kAttend: return x.attend(1, kMany);
          case kStatic: return x.attend_static(1, kMany);
          case kAppend: return x.append(1);
          default: return x.classify(1, labels);
        }
      });
      n[call] += more;
      CHECK(x.attend(0, kFew) == HC_OK, "layer 0 after allocation %d of %s: %s", nth, names[call], hc_last_error(x.c));
      CHECK(x.set(1, kFew) == HC_OK && x.attend(1, kFew) == HC_OK, "layer 1 again: %s", hc_last_error(x.c));
      if (!more) break;
    }
  CHECK(n[kSet] > 0 && n[kAttend] > 0 && n[kClassify] > 0, "allocations: %d %d %d", n[kSet], n[kAttend], n[kClassify]);
  CHECK(n[kStatic] == 0, "hc_attention_static allocates host memory (%d)", n[kStatic]);
}

struct { const char *name; void (*run)(); } checks[] = {
    {"errors_are_reported_once", errors_are_reported_once},
    {"shared_buffers_after_failed_growth", shared_buffers_after_failed_growth},
    {"first_attention_on_another_stream", first_attention_on_another_stream},
    {"small_windows", small_windows},
    {"host_memory", host_memory},
};

}  // namespace

int main(int argc, char **argv) {
  for (auto &c : checks) {
    if (argc > 1 && std::strcmp(argv[1], c.name) != 0) continue;
    c.run();
    for (size_t i = 0; i < fake::faults.size() && i < 20; ++i) std::printf("FAULT %s\n", fake::faults[i].c_str());
    if (failures || !fake::faults.empty()) return 1;
    std::printf("%s: ok\n", c.name);
  }
  return 0;
}

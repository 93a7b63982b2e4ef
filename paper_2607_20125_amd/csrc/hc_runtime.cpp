// Host runtime of the HeadCast routed-attention library: context, validation,
// per-layer head tables and compact buffers (Sec. 4.3), work lists of the
// head-specific attention (Sec. 4.4), and the one-time online classification
// (Sec. 4.2, Eq. 2-5).  Every entry point of include/headcast.h lives here.
#include "headcast.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "hc_internal.h"
#include "hc_plan.h"

using namespace hc;

namespace {

struct DevBuf {
  void *p = nullptr;
  size_t bytes = 0;
};

struct Layer {
  bool has_types = false;
  std::vector<uint8_t> types;
  std::vector<int32_t> slot;
  std::vector<int> sd_heads, sp_heads, g_heads;
  int64_t cur_block = -1;
  // the compact buffers: parts of one allocation, `kv`
  DevBuf kv, k_sd, v_sd, k_g, v_g, k_sp, v_sp;
  // dense work units and, behind them, combine items of the current plan
  DevBuf plan;
  const DenseUnit *units = nullptr;
  const CombineItem *comb = nullptr;
  int n_units = 0, n_comb = 0;
  bool plan_wide = false;      // 128-dim heads: the units run on waves of 64 queries
  int64_t plan_slots = 0;      // partial slots that the units write
  int plan_nv = -1;            // valid window blocks the plan was built for
  bool plan_used = false;      // launches may still read the plan's memory
  hipStream_t kv_stream = nullptr;   // the stream that last wrote the compact buffers
  int static_nv = -1;          // window fill that `chosen` is for
  StaticChoice chosen{};       // the device-built work list
  int sp_split = 1;            // key-frame split of the Spatial work (full window)
};

struct EventPair {
  hipEvent_t a, b;
};

}  // namespace

struct hc_ctx {
  hc_config cfg{};
  int device = 0;
  float scale = 0.f;
  int L = 0, P = 0;
  SpatialGeom geo{};          // frame storage of the Spatial buffers (centred window)
  int64_t sd_keys = 0, g_keys = 0, sp_keys = 0;
  std::vector<Layer> layers;
  std::string err;
  bool profile = false;
  std::vector<EventPair> pending[HC_K_COUNT];
  std::vector<EventPair> pool;
  double prof_ms[HC_K_COUNT] = {};
  int64_t prof_n[HC_K_COUNT] = {};
  DevBuf part;                 // partial-result slots shared by all layers
  int64_t part_slots = 0;
  DevBuf sp_part, sp_ml;       // Spatial split partials shared by all layers
  int64_t sp_part_rows = 0;
  int n_cu = 0;                // compute units of the device
  // cell variant of the Spatial path (cfg.spatial_cell > 0)
  CellTables cells;
  DevBuf cell_off_d, qmap_d;   // cells.off and cells.qmap on the device
  // device memory of hc_classify_heads, allocated (and zeroed) by the first call
  // and reused by the next ones: the window in Global and in Spatial layout, the
  // four proxy outputs, the block partials, the work lists, the token statistics
  DevBuf cls_k, cls_v, cls_pk, cls_pv, cls_o[4], cls_part, cls_units, cls_comb, cls_tok;
  int cls_n_units = 0, cls_n_comb = 0;
  bool cls_wide = false;       // 128-dim heads: the sweep runs on waves of 64 queries
  bool cls_done = false;       // cls_o holds the outputs of a successful classification
  void *scratch = nullptr;     // this device's fixed scratch (hc_attention_static)
  // the last choices of hc_attention_static: layers with as many heads of each kind
  // at the same window fill share one
  struct {
    int n_g, n_sd, nv;
    bool merged;
    StaticChoice choice;
  } static_memo[16];
  int static_memos = 0;        // choices made
};

namespace {

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

hc_status fail(hc_ctx *c, hc_status s, const char *fmt, ...) {
  if (c) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    try {
      c->err = buf;
    } catch (const std::bad_alloc &) {
      c->err.clear();
    }
  }
  return s;
}

// Ends the functions that allocate host memory: nothing is thrown across the ABI.
#define HC_NO_HOST_MEMORY(ctx) \
  catch (const std::bad_alloc &) { return fail(ctx, HC_E_NOMEM, "out of host memory"); }

// A failed HIP call stays the thread's last error until it is read, and the next
// launch would take it for its own: every failure that is reported or passed over
// here is read off first.
#define HC_HIP(ctx, call)                                                               \
  do {                                                                                  \
    hipError_t e_ = (call);                                                             \
    if (e_ != hipSuccess) {                                                             \
      (void)hipGetLastError();                                                          \
      return fail(ctx, e_ == hipErrorOutOfMemory ? HC_E_NOMEM : HC_E_DEVICE, "%s: %s", \
                  #call, hipGetErrorString(e_));                                        \
    }                                                                                   \
  } while (0)

hc_status dev_malloc(hc_ctx *c, DevBuf &b, size_t bytes) {
  const hipError_t e = hipMalloc(&b.p, bytes);
  if (e != hipSuccess) {
    b = DevBuf{};
    (void)hipGetLastError();
    return fail(c, HC_E_NOMEM, "hipMalloc(%zu bytes): %s", bytes, hipGetErrorString(e));
  }
  b.bytes = bytes;
  return HC_OK;
}

void free_buf(DevBuf &b) {
  if (b.p) (void)hipFree(b.p);
  b = DevBuf{};
}

// Memory cleared on `s`, the stream that uses it next.
hc_status alloc_zero(hc_ctx *c, DevBuf &b, size_t bytes, hipStream_t s) {
  free_buf(b);
  if (bytes == 0) return HC_OK;
  hc_status st = dev_malloc(c, b, bytes);
  if (st != HC_OK) return st;
  const hipError_t cleared = hipMemsetAsync(b.p, 0, bytes, s);
  if (cleared != hipSuccess) free_buf(b);      // not kept as if it were clear
  HC_HIP(c, cleared);
  return HC_OK;
}

void drop_plan(Layer &l) {
  l.units = nullptr;
  l.comb = nullptr;
  l.n_units = l.n_comb = 0;
  l.plan_nv = l.static_nv = -1;
}

void free_layer(Layer &l) {
  free_buf(l.kv);
  free_buf(l.plan);
  l.k_sd = l.v_sd = l.k_g = l.v_g = l.k_sp = l.v_sp = DevBuf{};
  drop_plan(l);
  l.plan_used = false;
}

// --- profiling ----------------------------------------------------------------
hc_status prof_begin(hc_ctx *c, hipStream_t s, EventPair *ep) {
  if (!c->profile) return HC_OK;
  if (c->pool.empty()) {
    EventPair p;
    HC_HIP(c, hipEventCreate(&p.a));
    const hipError_t e = hipEventCreate(&p.b);
    if (e != hipSuccess) {
      (void)hipEventDestroy(p.a);
      (void)hipGetLastError();
      return fail(c, HC_E_DEVICE, "hipEventCreate: %s", hipGetErrorString(e));
    }
    c->pool.push_back(p);
  }
  *ep = c->pool.back();
  c->pool.pop_back();
  HC_HIP(c, hipEventRecord(ep->a, s));
  return HC_OK;
}

hc_status prof_end(hc_ctx *c, hipStream_t s, int kind, const EventPair &ep) {
  if (!c->profile) return HC_OK;
  HC_HIP(c, hipEventRecord(ep.b, s));
  c->pending[kind].push_back(ep);
  return HC_OK;
}

template <class F>
hc_status timed_launch(hc_ctx *c, hipStream_t s, int kind, F &&launch) {
  EventPair ep{};
  hc_status st = prof_begin(c, s, &ep);
  if (st != HC_OK) return st;
  hipError_t e = launch();
  if (e != hipSuccess) return fail(c, HC_E_DEVICE, "kernel launch: %s", hipGetErrorString(e));
  return prof_end(c, s, kind, ep);
}

// --- geometry helpers ---------------------------------------------------------------
int n_valid_blocks(const hc_ctx *c, int64_t cur) {
  const int W = c->cfg.window_blocks;
  return (int)std::min<int64_t>(cur + 1, W);
}

// Block id held at logical window position i (sink first, current last).
int64_t logical_block(int64_t cur, int W, int i) {
  if (cur < W - 1) return i;
  return i == 0 ? 0 : cur - W + 1 + i;
}

hc_status check_layer(hc_ctx *c, int layer) {
  if (!c) return HC_E_INVAL;
  if (layer < 0 || layer >= c->cfg.n_layers)
    return fail(c, HC_E_INVAL, "layer %d out of range [0, %d)", layer, c->cfg.n_layers);
  return HC_OK;
}

hc_status check_types(hc_ctx *c, const uint8_t *types) {
  if (!types) return fail(c, HC_E_INVAL, "head types pointer is NULL");
  for (int h = 0; h < c->cfg.n_heads; ++h)
    if (types[h] > HC_GLOBAL) return fail(c, HC_E_INVAL, "head %d has invalid type %d", h, types[h]);
  return HC_OK;
}

int spatial_split(const hc_ctx *c, int n_sp, int radius);

// Keys of zeros before the first frame (and after the last) of a Spatial
// buffer in the centred-window layout; none in the cell-major one.
int64_t sp_lead(const hc_ctx *c) { return c->cfg.spatial_cell > 0 ? 0 : c->geo.lead; }

// First frame of a Spatial buffer (past its leading keys).
uint16_t *sp_frames(const hc_ctx *c, const DevBuf &b) {
  return b.p ? (uint16_t *)b.p + sp_lead(c) * c->cfg.head_dim : nullptr;
}

// The partial results that all layers share: at least `slots` dense slots, and at
// least `rows` rows of Spatial splits.  The old memory is released before the new is
// allocated, so while that fails there is none: the counts say so, and the next
// hc_attention of any layer asks again.
hc_status need_part(hc_ctx *c, int64_t slots, hipStream_t s) {
  if (slots <= c->part_slots) return HC_OK;
  HC_HIP(c, hipDeviceSynchronize());
  c->part_slots = 0;
  hc_status st = alloc_zero(c, c->part, (size_t)slots * partial_floats(c->cfg.head_dim) * 4, s);
  if (st == HC_OK) c->part_slots = slots;
  return st;
}

hc_status need_sp_part(hc_ctx *c, int64_t rows, hipStream_t s) {
  if (rows <= c->sp_part_rows) return HC_OK;
  HC_HIP(c, hipDeviceSynchronize());
  c->sp_part_rows = 0;
  hc_status st = alloc_zero(c, c->sp_part, (size_t)rows * c->cfg.head_dim * 4, s);
  if (st == HC_OK) st = alloc_zero(c, c->sp_ml, (size_t)rows * 2 * 4, s);
  if (st == HC_OK) c->sp_part_rows = rows;
  return st;
}

int64_t sp_split_rows(const hc_ctx *c, const Layer &l) {
  return l.sp_split > 1 ? (int64_t)l.sp_split * (int64_t)l.sp_heads.size() * c->L : 0;
}

// Build the layer's head table and its compact buffers, zeroed on `s`.  The six
// buffers are one allocation, which is kept when the new table needs exactly as
// many bytes; either way everything that read the old buffers is over before
// they are written (hipFree waits for the device, and so does the other branch).
// Six buffers and two work lists allocated, cleared and freed one by one left the
// GPU idle for 1.4 ms (480P) to 1.9 ms (720P) of a layer's classification.
hc_status install_types(hc_ctx *c, Layer &l, const uint8_t *types, hipStream_t s) try {
  const int H = c->cfg.n_heads, D = c->cfg.head_dim;
  l.has_types = false;
  l.types.assign(types, types + H);
  l.slot.assign(H, 0);
  l.sd_heads.clear(); l.sp_heads.clear(); l.g_heads.clear();
  for (int h = 0; h < H; ++h) {
    switch (types[h]) {
      case HC_SINK:
      case HC_DUMMY: l.slot[h] = (int)l.sd_heads.size(); l.sd_heads.push_back(h); break;
      case HC_SPATIAL: l.slot[h] = (int)l.sp_heads.size(); l.sp_heads.push_back(h); break;
      default: l.slot[h] = (int)l.g_heads.size(); l.g_heads.push_back(h); break;
    }
  }
  const size_t row = (size_t)D * 2;
  const int64_t spk = c->cfg.spatial_cell > 0 ? c->cells.keys : c->sp_keys;
  const int64_t sp_all = l.sp_heads.empty() ? 0 : (int64_t)l.sp_heads.size() * spk + 2 * sp_lead(c);
  l.k_sd.bytes = l.v_sd.bytes = l.sd_heads.size() * c->sd_keys * row;
  l.k_g.bytes = l.v_g.bytes = l.g_heads.size() * c->g_keys * row;
  l.k_sp.bytes = l.v_sp.bytes = sp_all * row;
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  size_t total = 0;
  for (const DevBuf *b : {&l.k_sd, &l.v_sd, &l.k_g, &l.v_g, &l.k_sp, &l.v_sp}) total += al(b->bytes);
  drop_plan(l);
  hc_status st;
  if (l.kv.p && l.kv.bytes == total) {
    HC_HIP(c, hipDeviceSynchronize());
  } else {
    free_buf(l.kv);
    if ((st = dev_malloc(c, l.kv, total)) != HC_OK) return st;
  }
  l.plan_used = false;
  l.kv_stream = s;
  HC_HIP(c, hipMemsetAsync(l.kv.p, 0, total, s));
  unsigned char *at = (unsigned char *)l.kv.p;
  for (DevBuf *b : {&l.k_sd, &l.v_sd, &l.k_g, &l.v_g, &l.k_sp, &l.v_sp}) {
    b->p = b->bytes ? at : nullptr;
    at += al(b->bytes);
  }

  // Spatial work split over key frames when the layer has few Spatial heads
  l.sp_split = c->cfg.spatial_cell > 0 ? 1
                                         : spatial_split(c, (int)l.sp_heads.size(), c->cfg.spatial_radius);
  if ((st = need_sp_part(c, sp_split_rows(c, l), s)) != HC_OK) return st;
  // partial slots for the largest plan of this layer (full window)
  const int64_t nqt = (c->L + kQTile - 1) / kQTile;
  const int64_t need = ((int64_t)l.g_heads.size() * c->cfg.window_blocks +
                        (int64_t)l.sd_heads.size() * (c->cfg.sd_blocks == 2 ? 2 : 0)) * nqt;
  if ((st = need_part(c, need, s)) != HC_OK) return st;
  l.has_types = true;
  return HC_OK;
} HC_NO_HOST_MEMORY(c)

// Whether a layer-step has partials to merge however its Global heads are cut: those of
// split Spatial heads, or of two-block Sink/Dummy heads.
bool merged_anyway(const hc_ctx *c, const Layer &l, int nv) {
  return l.sp_split > 1 || (c->cfg.sd_blocks == 2 && nv >= 2 && !l.sd_heads.empty());
}

// Dense work of one layer with `nv` valid window blocks (hc_plan.h).
void plan_units(const hc_ctx *c, const Layer &l, int nv, std::vector<DenseUnit> &units,
                std::vector<CombineItem> &comb) {
  const int D = c->cfg.head_dim;
  auto parts = [&](const std::vector<int> &heads, const DevBuf &k, const DevBuf &v, int64_t keys) {
    std::vector<HeadKV> out;
    for (int h : heads)
      out.push_back(HeadKV{h, (const uint16_t *)k.p + (size_t)l.slot[h] * keys * D,
                           (const uint16_t *)v.p + (size_t)l.slot[h] * keys * D});
    return out;
  };
  DensePlanShape shape;
  shape.d = D;
  shape.L = c->L;
  shape.nv = nv;
  shape.g_parts = merged_anyway(c, l, nv) ? 0 : global_parts(D, c->L, nv);
  shape.sd_blocks = c->cfg.sd_blocks;
  shape.F = c->cfg.frames_per_block;
  shape.grid_h = c->cfg.grid_h;
  shape.grid_w = c->cfg.grid_w;
  shape.cell = c->cfg.spatial_cell;
  shape.cells = &c->cells;
  const std::vector<HeadKV> cell_heads =
      c->cfg.spatial_cell > 0 ? parts(l.sp_heads, l.k_sp, l.v_sp, c->cells.keys)
                              : std::vector<HeadKV>{};
  plan_dense_units(shape, parts(l.g_heads, l.k_g, l.v_g, c->g_keys),
                   parts(l.sd_heads, l.k_sd, l.v_sd, c->sd_keys), cell_heads, c->n_cu, units, comb);
}

template <class T>
hc_status upload(hc_ctx *c, DevBuf &b, const std::vector<T> &v) {
  free_buf(b);
  if (v.empty()) return HC_OK;
  hc_status st = dev_malloc(c, b, v.size() * sizeof(T));
  if (st != HC_OK) return st;
  HC_HIP(c, hipMemcpy(b.p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  return HC_OK;
}

hc_status ensure_plan(hc_ctx *c, Layer &l, int nv, hipStream_t s) try {
  if (l.plan_nv == nv) return HC_OK;
  std::vector<DenseUnit> units;
  std::vector<CombineItem> comb;
  plan_units(c, l, nv, units, comb);
  // every tile a unit's DMA reads (whole 64-key tiles from kv0) must lie inside
  // its head's part of the buffer
  {
    const int D = c->cfg.head_dim;
    std::vector<KeyRegion> regions = {
        {(const uint16_t *)l.k_g.p, (int64_t)l.g_heads.size(), c->g_keys},
        {(const uint16_t *)l.k_sd.p, (int64_t)l.sd_heads.size(), c->sd_keys}};
    if (c->cfg.spatial_cell > 0)
      regions.push_back({(const uint16_t *)l.k_sp.p, (int64_t)l.sp_heads.size(), c->cells.keys});
    const int bad = first_unit_outside(units, regions, D);
    if (bad >= 0) {
      const DenseUnit &u = units[bad];
      return fail(c, HC_E_STATE, "internal: work unit of head %d reads keys [%d, %lld) of %lld",
                  u.head, u.kv0, (long long)unit_read_end(u),
                  (long long)unit_region_keys(u, regions, D));
    }
  }
  // launches of the previous plan are over before its memory is written again, and so
  // is a split or append of this window fill on another stream than the caller's
  // (hipStreamPerThread is another stream in every thread).  Not asked on the same
  // stream: 8 us of the smallest layer's first call.
  if (l.plan_used || (!units.empty() && (l.kv_stream != s || s == hipStreamPerThread)))
    HC_HIP(c, hipDeviceSynchronize());
  // no plan until this one is complete: a failure below leaves a rebuild for
  // the next call instead of a list that does not match its counts
  drop_plan(l);
  l.plan_used = false;
  hc_status st;
  int64_t slots = 0;
  for (const CombineItem &it : comb) slots = std::max<int64_t>(slots, (int64_t)it.slot0 + it.n_slots);
  if ((st = need_part(c, slots, s)) != HC_OK) return st;
  // both lists in one copy
  const size_t b_units = (units.size() * sizeof(DenseUnit) + 255) / 256 * 256;
  std::vector<unsigned char> both(b_units + comb.size() * sizeof(CombineItem));
  if (!units.empty()) std::memcpy(both.data(), units.data(), units.size() * sizeof(DenseUnit));
  if (!comb.empty())
    std::memcpy(both.data() + b_units, comb.data(), comb.size() * sizeof(CombineItem));
  if (!both.empty()) {
    if (l.plan.bytes < both.size()) {
      free_buf(l.plan);
      if ((st = dev_malloc(c, l.plan, both.size())) != HC_OK) return st;
    }
    HC_HIP(c, hipMemcpy(l.plan.p, both.data(), both.size(), hipMemcpyHostToDevice));
  }
  l.units = (const DenseUnit *)l.plan.p;
  l.comb = (const CombineItem *)((const unsigned char *)l.plan.p + b_units);
  l.n_units = (int)units.size();
  l.n_comb = (int)comb.size();
  l.plan_wide = c->cfg.head_dim == 128 && dense_wide_waves(units, c->n_cu, true);
  l.plan_slots = slots;
  l.plan_nv = nv;
  l.plan_used = true;
  return HC_OK;
} HC_NO_HOST_MEMORY(c)

ScatterArgs scatter_args(const hc_ctx *c, const Layer &l) {
  ScatterArgs a{};
  a.L = c->L; a.D = c->cfg.head_dim; a.Hg = c->cfg.grid_h; a.Wg = c->cfg.grid_w;
  a.geo = c->geo; a.F = c->cfg.frames_per_block;
  a.cell = c->cfg.spatial_cell; a.ncy = c->cells.ncy; a.ncx = c->cells.ncx;
  a.cell_off = (const int64_t *)c->cell_off_d.p;
  a.sd_keys = c->sd_keys; a.g_keys = c->g_keys;
  a.sp_keys = a.cell > 0 ? c->cells.keys : c->sp_keys;
  a.k_sd = (uint16_t *)l.k_sd.p; a.v_sd = (uint16_t *)l.v_sd.p;
  a.k_g = (uint16_t *)l.k_g.p; a.v_g = (uint16_t *)l.v_g.p;
  a.k_sp = sp_frames(c, l.k_sp); a.v_sp = sp_frames(c, l.v_sp);
  for (int h = 0; h < c->cfg.n_heads; ++h) {
    a.head_kind[h] = l.types[h];
    a.head_slot[h] = (uint8_t)l.slot[h];
  }
  return a;
}

// Sink-Dummy slot (L keys each) that block `b` takes in a head of archetype
// `kind` when `cur` is the current block, or -1.  One block: Sink keeps block
// 0, Dummy the current block, both in slot 0.  Two blocks: Sink keeps block 0
// in slot 0 and the current block in slot 1; Dummy keeps the previous and the
// current block in slots b mod 2.
int sd_slot(const hc_ctx *c, int kind, int64_t b, int64_t cur) {
  if (c->cfg.sd_blocks == 2) {
    if (kind == HC_SINK) return b == 0 ? 0 : (b == cur ? 1 : -1);
    return (b == cur || b == cur - 1) ? (int)(b % 2) : -1;
  }
  if (kind == HC_SINK) return b == 0 ? 0 : -1;
  return b == cur ? 0 : -1;
}

// Split a logical-order window of n = min(cur+1, W) blocks into the layer's buffers.
hc_status split_window(hc_ctx *c, Layer &l, int64_t cur, const void *k_win, const void *v_win,
                       hipStream_t s) {
  const int W = c->cfg.window_blocks;
  const int n = n_valid_blocks(c, cur);
  ScatterArgs a = scatter_args(c, l);
  a.src_k = (const uint16_t *)k_win;
  a.src_v = (const uint16_t *)v_win;
  a.n_src = n;
  for (int i = 0; i < n; ++i) {
    const int64_t b = logical_block(cur, W, i);
    a.src_slot[i] = (int8_t)hc_ring_slot(b, W);
    a.sink_slot[i] = (int8_t)sd_slot(c, HC_SINK, b, cur);
    a.dummy_slot[i] = (int8_t)sd_slot(c, HC_DUMMY, b, cur);
  }
  return timed_launch(c, s, HC_K_SCATTER, [&] { return launch_scatter(a, c->cfg.n_heads, s); });
}

// Key-frame split of a layer's Spatial work (spatial_split_count): a layer
// with few Spatial heads has fewer work groups than the GPU holds at once (four
// per CU), and the launch then takes as long as one group's walk over all W F
// key frames, so the frames are cut into ranges merged afterwards.
int spatial_split(const hc_ctx *c, int n_sp, int radius) {
  if (n_sp == 0) return 1;
  int c_lo, c_hi;
  spatial_tiles(c->cfg.grid_w, radius, &c_lo, &c_hi);
  const int64_t groups =
      (int64_t)n_sp * ((c->cfg.grid_h + kSpRows - 1) / kSpRows) * (c_hi - c_lo + 1);
  const int64_t resident = 4 * (int64_t)std::max(c->n_cu, 1);
  const int64_t frames = (int64_t)c->cfg.window_blocks * c->cfg.frames_per_block;
  return spatial_split_count(groups, resident, frames);
}

SpatialArgs spatial_args(const hc_ctx *c, int radius, int n_slots) {
  SpatialArgs a{};
  a.L = c->L; a.Hg = c->cfg.grid_h; a.Wg = c->cfg.grid_w; a.geo = c->geo;
  a.F = c->cfg.frames_per_block; a.n_slots = n_slots; a.r = radius;
  int c_hi;
  spatial_tiles(a.Wg, radius, &a.c_lo, &c_hi);
  a.n_ct = c_hi - a.c_lo + 1;
  a.n_rowgroups = (a.Hg + kSpRows - 1) / kSpRows;
  a.n_split = 1;
  a.scale_log2 = c->scale * 1.4426950408889634f;
  return a;
}

// Checks shared by hc_attention and hc_attention_static.
hc_status check_attention(hc_ctx *c, int layer, const void *q, const uint8_t *head_types,
                          const float *o) {
  hc_status st = check_layer(c, layer);
  if (st != HC_OK) return st;
  if (!q || !o) return fail(c, HC_E_INVAL, "q and o must not be NULL");
  if (!aligned16(q) || !aligned16(o)) return fail(c, HC_E_INVAL, "q and o must be 16-byte aligned");
  if ((st = check_types(c, head_types)) != HC_OK) return st;
  const Layer &l = c->layers[layer];
  if (!l.has_types) return fail(c, HC_E_STATE, "layer %d has no head table", layer);
  if (std::memcmp(head_types, l.types.data(), c->cfg.n_heads) != 0)
    return fail(c, HC_E_STATE, "head types differ from the table of layer %d", layer);
  return HC_OK;
}

StaticChoice static_choice_shared(hc_ctx *c, const StaticPlan &p, bool merged) {
  constexpr int kMemos = (int)(sizeof c->static_memo / sizeof c->static_memo[0]);
  for (int i = 0; i < std::min(c->static_memos, kMemos); ++i) {
    const auto &m = c->static_memo[i];
    if (m.n_g == p.n_g && m.n_sd == p.n_sd && m.nv == p.nv && m.merged == merged) return m.choice;
  }
  const StaticChoice choice = static_choice(p, c->n_cu, static_max_slots(p, kStaticScratchBytes), merged);
  c->static_memo[c->static_memos % kMemos] = {p.n_g, p.n_sd, p.nv, merged, choice};
  c->static_memos = c->static_memos < 2 * kMemos - 1 ? c->static_memos + 1 : kMemos;
  return choice;
}

// Device memory one routed layer-step works in: the dense work list and merge
// items, the partial-result slots, and the Spatial split partials.
struct LayerWork {
  const DenseUnit *units = nullptr;
  int n_units = 0;
  bool wide_waves = false;     // 128-dim heads: 64 queries per wave
  const CombineItem *comb = nullptr;
  int n_comb = 0;
  float *part = nullptr;
  int sp_split = 1;
  float *sp_part = nullptr, *sp_ml = nullptr;
  bool shared_part = false;    // Spatial and dense partials take turns in the same place
};

// The launches of one routed layer-step (Sec. 4.4): the split Spatial heads, the
// dense units (Global, Sink/Dummy, cells), one merge of the partials of both.
// One merge instead of one after each kernel: 480P layers 1-3% faster (one Spatial
// head 193 -> 187 us, three 179 -> 177 us), the smallest 28.5 -> 25.5 us.  The
// Spatial heads go first: with the dense partials written before them and merged
// after them the same layers took 189 and 182 us.  Unsplit Spatial heads have
// nothing to merge and go last (first they cost a 1080P layer 0.2%).  Where the
// partials share memory the Spatial ones are merged before the dense units run.
hc_status run_layer(hc_ctx *c, const Layer &l, int nv, const void *q, float *o,
                    const LayerWork &wk, hipStream_t s) {
  const int D = c->cfg.head_dim, H = c->cfg.n_heads;
  hc_status st;
  CombineArgs ca{};
  ca.part = wk.part;
  ca.items = wk.comb;
  ca.o[0] = ca.o[1] = ca.o[2] = o;
  ca.n_items = wk.n_comb;
  ca.L = c->L;
  ca.D = D;
  SpatialArgs sa{};
  sa.n_split = 1;
  auto merge = [&] {
    return wk.n_comb == 0 ? HC_OK : timed_launch(c, s, HC_K_COMBINE, [&] { return launch_merge(ca, sa, D, s); });
  };
  auto spatial = [&]() -> hc_status {
    if (l.sp_heads.empty() || c->cfg.spatial_cell > 0) return HC_OK;
    sa = spatial_args(c, c->cfg.spatial_radius, nv);
    sa.q = (const uint16_t *)q;
    sa.o = o;
    sa.k = sp_frames(c, l.k_sp);
    sa.v = sp_frames(c, l.v_sp);
    sa.head_stride = c->sp_keys * D;
    sa.n_sp = (int)l.sp_heads.size();
    for (int j = 0; j < sa.n_sp; ++j) sa.heads[j] = (int8_t)l.sp_heads[j];
    // every split range holds at least one valid key frame
    sa.n_split = std::min(wk.sp_split, nv * c->cfg.frames_per_block);
    sa.part = wk.sp_part;
    sa.part_ml = wk.sp_ml;
    const SpatialRole role = (int)l.sp_heads.size() == H ? SpatialRole::kSpatialOnly
                                                         : SpatialRole::kRouted;
    // a merge of the splits alone is timed with the Spatial launch
    const bool merge_now = wk.n_comb == 0 || wk.shared_part;
    const hc_status ss = timed_launch(c, s, HC_K_SPATIAL, [&] {
      const hipError_t e = launch_spatial(sa, D, role, s);
      if (e != hipSuccess || !merge_now) return e;
      CombineArgs none{};
      return launch_merge(none, sa, D, s);
    });
    if (merge_now) sa.n_split = 1;
    return ss;
  };
  const bool split = std::min(wk.sp_split, nv * c->cfg.frames_per_block) > 1;
  if (split && (st = spatial()) != HC_OK) return st;
  if (wk.n_units > 0) {
    DenseArgs a{};
    a.units = wk.units;
    a.qmap = (const int32_t *)c->qmap_d.p;
    a.q = (const uint16_t *)q;
    a.o[0] = a.o[1] = a.o[2] = o;
    a.part = wk.part;
    a.n_units = wk.n_units;
    a.L = c->L;
    a.scale_log2 = c->scale * 1.4426950408889634f;
    a.wide_waves = wk.wide_waves;
    const DenseRole role = (int)l.g_heads.size() == H ? DenseRole::kFullWindow
                           : (c->cfg.spatial_cell > 0 || c->cfg.sd_blocks == 2)
                               ? DenseRole::kVariant
                           : (int)l.sd_heads.size() == H ? DenseRole::kSinkDummyOnly
                                                          : DenseRole::kRouted;
    st = timed_launch(c, s, HC_K_DENSE, [&] { return launch_dense(a, D, role, s); });
    if (st != HC_OK) return st;
  }
  if ((st = merge()) != HC_OK || split) return st;
  return spatial();
}

}  // namespace

// ===========================================================================
// Public ABI
// ===========================================================================
extern "C" {

void hc_config_default(hc_config *cfg) {
  if (!cfg) return;
  hc_config d{};
  d.n_layers = 30; d.n_heads = 12; d.head_dim = 128;
  d.grid_h = 30; d.grid_w = 52; d.frames_per_block = 3; d.window_blocks = 7;
  d.spatial_radius = 4; d.proxy_radius = 2;
  d.theta_sink = d.theta_dummy = d.theta_spatial = 0.95f;
  d.theta_score = 0.755f; d.gamma = 5.0f; d.softmax_scale = 0.f;
  d.spatial_cell = 0; d.sd_blocks = 1;
  *cfg = d;
}

hc_status hc_validate_config(const hc_config *c) {
  if (!c) return HC_E_INVAL;
  if (c->n_layers < 1 || c->n_heads < 1 || c->n_heads > kMaxHeads) return HC_E_INVAL;
  if (c->head_dim != 64 && c->head_dim != 128) return HC_E_INVAL;
  if (c->grid_h < 1 || c->grid_w < 1 || c->frames_per_block < 1 || c->frames_per_block > 4)
    return HC_E_INVAL;
  if (c->window_blocks < 2 || c->window_blocks > kMaxSrcBlocks) return HC_E_INVAL;
  if (c->spatial_radius < 0 || c->spatial_radius > 12) return HC_E_INVAL;
  if (c->proxy_radius < 0 || c->proxy_radius > 12) return HC_E_INVAL;
  if (c->sd_blocks != 1 && c->sd_blocks != 2) return HC_E_INVAL;
  // The two-block Dummy set needs the previous block inside the window (block 0 plus
  // at least two recent blocks).
  if (c->sd_blocks == 2 && c->window_blocks < 3) return HC_E_INVAL;
  if (c->spatial_cell != 0) {
    if (c->spatial_cell < 2 || c->spatial_cell > 64) return HC_E_INVAL;
    if (n_cells(c->grid_h, c->spatial_cell) > 64 || n_cells(c->grid_w, c->spatial_cell) > 64)
      return HC_E_INVAL;
  }
  const int64_t L = (int64_t)c->frames_per_block * c->grid_h * c->grid_w;
  if (L % 8 != 0) return HC_E_INVAL;
  if (L * c->window_blocks + 4 * kKTile > INT32_MAX / 2) return HC_E_INVAL;
  if (!(c->softmax_scale >= 0.f) || !std::isfinite(c->softmax_scale)) return HC_E_INVAL;
  if (!std::isfinite(c->gamma) || !std::isfinite(c->theta_sink) ||
      !std::isfinite(c->theta_dummy) || !std::isfinite(c->theta_spatial) ||
      !std::isfinite(c->theta_score))
    return HC_E_INVAL;
  return HC_OK;
}

const char *hc_status_string(hc_status s) {
  switch (s) {
    case HC_OK: return "ok";
    case HC_E_INVAL: return "invalid argument";
    case HC_E_STATE: return "invalid state";
    case HC_E_ORDER: return "block out of order";
    case HC_E_NOMEM: return "out of device memory";
    case HC_E_DEVICE: return "device error";
  }
  return "unknown status";
}

const char *hc_last_error(const hc_ctx *ctx) { return ctx ? ctx->err.c_str() : ""; }

int32_t hc_ring_slot(int64_t block, int32_t W) {
  if (block < 0 || W < 2) return -1;
  if (block == 0) return 0;
  return (int32_t)(1 + (block - 1) % (W - 1));
}

hc_status hc_create(const hc_config *cfg, int device, hc_ctx **out) try {
  if (!out) return HC_E_INVAL;
  *out = nullptr;
  if (hc_validate_config(cfg) != HC_OK) return HC_E_INVAL;
  int ndev = 0;
  void *scratch = nullptr;
  auto ok = [](hipError_t e) { return e == hipSuccess || ((void)hipGetLastError(), false); };
  if (!ok(hipGetDeviceCount(&ndev)) || device < 0 || device >= ndev) return HC_E_DEVICE;
  if (!ok(hipSetDevice(device)) || !ok(static_scratch(device, &scratch))) return HC_E_DEVICE;
  std::unique_ptr<hc_ctx, void (*)(hc_ctx *)> owner(new hc_ctx, hc_destroy);
  hc_ctx *c = owner.get();
  c->cfg = *cfg;
  c->device = device;
  c->scratch = scratch;
  c->scale = cfg->softmax_scale > 0.f ? cfg->softmax_scale : 1.0f / std::sqrt((float)cfg->head_dim);
  c->P = cfg->grid_h * cfg->grid_w;
  c->L = cfg->frames_per_block * c->P;
  c->geo = spatial_geometry(*cfg);
  // each head's part ends with a spare tile for the reads of a unit's last tile
  c->sd_keys = sd_buffer_keys(cfg->sd_blocks, c->L);
  c->g_keys = global_buffer_keys(cfg->window_blocks, c->L);
  c->sp_keys = (int64_t)cfg->window_blocks * cfg->frames_per_block * c->geo.rows * c->geo.pitch;
  if (!ok(hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, device))) c->n_cu = 0;
  c->layers.resize(cfg->n_layers);
  if (cfg->spatial_cell > 0) {
    c->cells = build_cell_tables(cfg->grid_h, cfg->grid_w, cfg->frames_per_block,
                                 cfg->window_blocks, cfg->spatial_cell);
    hc_status st = upload(c, c->cell_off_d, c->cells.off);
    if (st == HC_OK) st = upload(c, c->qmap_d, c->cells.qmap);
    if (st != HC_OK) return st;
  }
  *out = owner.release();
  return HC_OK;
} HC_NO_HOST_MEMORY(nullptr)

void hc_destroy(hc_ctx *c) {
  if (!c) return;
  (void)hipSetDevice(c->device);
  (void)hipDeviceSynchronize();
  for (auto &l : c->layers) free_layer(l);
  free_buf(c->part);
  free_buf(c->sp_part);
  free_buf(c->sp_ml);
  free_buf(c->cell_off_d);
  free_buf(c->qmap_d);
  for (DevBuf *b : {&c->cls_k, &c->cls_v, &c->cls_pk, &c->cls_pv, &c->cls_o[0], &c->cls_o[1],
                    &c->cls_o[2], &c->cls_o[3], &c->cls_part, &c->cls_units, &c->cls_comb,
                    &c->cls_tok})
    free_buf(*b);
  for (int k = 0; k < HC_K_COUNT; ++k)
    for (auto &e : c->pending[k]) c->pool.push_back(e);
  for (auto &e : c->pool) {
    (void)hipEventDestroy(e.a);
    (void)hipEventDestroy(e.b);
  }
  delete c;
}

hc_status hc_set_head_types(hc_ctx *c, int layer, const uint8_t *types, int64_t cur_block,
                            const void *k_win, const void *v_win, hc_stream stream) try {
  hc_status st = check_layer(c, layer);
  if (st != HC_OK) return st;
  if ((st = check_types(c, types)) != HC_OK) return st;
  if (cur_block < 0) return fail(c, HC_E_INVAL, "cur_block %lld < 0", (long long)cur_block);
  if (!k_win || !v_win) return fail(c, HC_E_INVAL, "window pointers must not be NULL");
  if (!aligned16(k_win) || !aligned16(v_win))
    return fail(c, HC_E_INVAL, "window pointers must be 16-byte aligned");
  HC_HIP(c, hipSetDevice(c->device));
  Layer &l = c->layers[layer];
  hipStream_t s = (hipStream_t)stream;
  if ((st = install_types(c, l, types, s)) != HC_OK) {
    free_layer(l);
    l.has_types = false;
    return st;
  }
  if ((st = split_window(c, l, cur_block, k_win, v_win, s)) != HC_OK) return st;
  l.cur_block = cur_block;
  return HC_OK;
} HC_NO_HOST_MEMORY(c)

hc_status hc_get_layout(const hc_ctx *cc, int layer, int32_t *head_slot, int32_t *ring) {
  hc_ctx *c = const_cast<hc_ctx *>(cc);
  hc_status st = check_layer(c, layer);
  if (st != HC_OK) return st;
  const Layer &l = c->layers[layer];
  if (!l.has_types) return fail(c, HC_E_STATE, "layer %d has no head table", layer);
  const int W = c->cfg.window_blocks;
  if (head_slot)
    for (int h = 0; h < c->cfg.n_heads; ++h) head_slot[h] = l.slot[h];
  if (ring) {
    const int n = n_valid_blocks(c, l.cur_block);
    for (int i = 0; i < W; ++i)
      ring[i] = i < n ? hc_ring_slot(logical_block(l.cur_block, W, i), W) : -1;
  }
  return HC_OK;
}

hc_status hc_append_block(hc_ctx *c, int layer, int64_t block, const void *k_blk,
                          const void *v_blk, hc_stream stream) try {
  hc_status st = check_layer(c, layer);
  if (st != HC_OK) return st;
  if (!k_blk || !v_blk) return fail(c, HC_E_INVAL, "block pointers must not be NULL");
  if (!aligned16(k_blk) || !aligned16(v_blk))
    return fail(c, HC_E_INVAL, "block pointers must be 16-byte aligned");
  Layer &l = c->layers[layer];
  if (!l.has_types) return fail(c, HC_E_STATE, "layer %d has no head table", layer);
  if (block != l.cur_block && block != l.cur_block + 1)
    return fail(c, HC_E_ORDER, "block %lld after current block %lld", (long long)block,
                (long long)l.cur_block);
  HC_HIP(c, hipSetDevice(c->device));
  ScatterArgs a = scatter_args(c, l);
  a.src_k = (const uint16_t *)k_blk;
  a.src_v = (const uint16_t *)v_blk;
  a.n_src = 1;
  a.src_slot[0] = (int8_t)hc_ring_slot(block, c->cfg.window_blocks);
  a.sink_slot[0] = (int8_t)sd_slot(c, HC_SINK, block, block);
  a.dummy_slot[0] = (int8_t)sd_slot(c, HC_DUMMY, block, block);
  hipStream_t s = (hipStream_t)stream;
  l.kv_stream = s;
  st = timed_launch(c, s, HC_K_SCATTER, [&] { return launch_scatter(a, c->cfg.n_heads, s); });
  if (st != HC_OK) return st;
  l.cur_block = block;
  return HC_OK;
} HC_NO_HOST_MEMORY(c)

hc_status hc_attention(hc_ctx *c, int layer, const void *q, const uint8_t *head_types, float *o,
                       hc_stream stream) try {
  hc_status st = check_attention(c, layer, q, head_types, o);
  if (st != HC_OK) return st;
  Layer &l = c->layers[layer];
  HC_HIP(c, hipSetDevice(c->device));
  const int nv = n_valid_blocks(c, l.cur_block);
  if ((st = ensure_plan(c, l, nv, (hipStream_t)stream)) != HC_OK) return st;
  if ((st = need_part(c, l.plan_slots, (hipStream_t)stream)) != HC_OK) return st;
  if ((st = need_sp_part(c, sp_split_rows(c, l), (hipStream_t)stream)) != HC_OK) return st;
  LayerWork wk;
  wk.units = l.units;
  wk.n_units = l.n_units;
  wk.wide_waves = l.plan_wide;
  wk.comb = l.comb;
  wk.n_comb = l.n_comb;
  wk.part = (float *)c->part.p;
  wk.sp_split = l.sp_split;
  wk.sp_part = (float *)c->sp_part.p;
  wk.sp_ml = (float *)c->sp_ml.p;
  return run_layer(c, l, nv, q, o, wk, (hipStream_t)stream);
} HC_NO_HOST_MEMORY(c)

hc_status hc_attention_static(hc_ctx *c, int layer, const void *q, const uint8_t *head_types,
                              float *o, hc_stream stream) try {
  hc_status st = check_attention(c, layer, q, head_types, o);
  if (st != HC_OK) return st;
  if (c->cfg.spatial_cell > 0)
    return fail(c, HC_E_INVAL, "hc_attention_static: the cell variant (spatial_cell > 0) is not "
                "supported");
  Layer &l = c->layers[layer];
  const int nv = n_valid_blocks(c, l.cur_block);
  const int D = c->cfg.head_dim, F = c->cfg.frames_per_block;
  StaticPlan p{};
  p.k_g = (const uint16_t *)l.k_g.p; p.v_g = (const uint16_t *)l.v_g.p;
  p.k_sd = (const uint16_t *)l.k_sd.p; p.v_sd = (const uint16_t *)l.v_sd.p;
  p.g_keys = c->g_keys; p.sd_keys = c->sd_keys;
  p.d = D; p.L = c->L; p.nv = nv; p.nqt = (c->L + kQTile - 1) / kQTile;
  p.sd_parts = (c->cfg.sd_blocks == 2 && nv >= 2) ? 2 : 1;
  p.n_g = (int)l.g_heads.size(); p.n_sd = (int)l.sd_heads.size();
  for (int i = 0; i < p.n_g; ++i) p.g_head[i] = (int8_t)l.g_heads[i];
  for (int i = 0; i < p.n_sd; ++i) p.sd_head[i] = (int8_t)l.sd_heads[i];
  // layout of the scratch: work list, merge items, dense partials, Spatial split
  // partials and their (max, sum) pairs, each 256-byte aligned.  Where not all of
  // them fit, the Spatial partials are merged before the dense units run, in the
  // place that the dense ones then take.
  const size_t need = static_dense_bytes(p);
  if (need > kStaticScratchBytes)
    return fail(c, HC_E_INVAL, "hc_attention_static: layer %d needs %zu bytes of scratch, the "
                "static buffer holds %zu", layer, need, (size_t)kStaticScratchBytes);
  if (l.static_nv != nv) {
    l.chosen = static_choice_shared(c, p, merged_anyway(c, l, nv));
    l.static_nv = nv;
  }
  p.g_parts = l.chosen.parts;
  const size_t n_units = (size_t)static_n_units(p), n_comb = (size_t)static_n_comb(p);
  const size_t b_units = align256(n_units * sizeof(DenseUnit)), b_lists = static_list_bytes(p);
  const int n_sp = (int)l.sp_heads.size();
  int split = std::min(l.sp_split, nv * F);
  auto sp_rows = [&](int sp) { return sp > 1 ? (size_t)sp * n_sp * c->L : 0; };
  auto sp_bytes = [&](int sp) { return align256(sp_rows(sp) * D * sizeof(float)) + sp_rows(sp) * 2 * sizeof(float); };
  size_t sp_at = static_dense_bytes(p);
  const bool shared = sp_at + sp_bytes(split) > kStaticScratchBytes;
  if (shared) {
    sp_at = b_lists;
    while (split > 1 && sp_at + sp_bytes(split) > kStaticScratchBytes) --split;
  }
  HC_HIP(c, hipSetDevice(c->device));
  hipStream_t s = (hipStream_t)stream;
  unsigned char *base = (unsigned char *)c->scratch;
  LayerWork wk;
  wk.units = (const DenseUnit *)base;
  wk.n_units = (int)n_units;
  wk.wide_waves = l.chosen.wide;
  wk.comb = (const CombineItem *)(base + b_units);
  wk.n_comb = (int)n_comb;
  wk.part = (float *)(base + b_lists);
  wk.sp_split = split;
  wk.sp_part = (float *)(base + sp_at);
  wk.sp_ml = (float *)(base + sp_at + align256(sp_rows(split) * D * sizeof(float)));
  wk.shared_part = shared;
  HC_HIP(c, launch_static_plan(p, (DenseUnit *)wk.units, (CombineItem *)wk.comb, s));
  return run_layer(c, l, nv, q, o, wk, s);
} HC_NO_HOST_MEMORY(c)

namespace {

// A classification buffer of at least `bytes`, kept by the context: allocated
// and zeroed the first time, reused as is afterwards.  Padding keys of the
// window copies stay zero because later calls only rewrite real keys.
hc_status keep(hc_ctx *c, DevBuf &b, size_t bytes, hipStream_t s) {
  if (b.p && b.bytes >= bytes) return HC_OK;
  HC_HIP(c, hipDeviceSynchronize());
  return alloc_zero(c, b, bytes, s);
}

// Eq. 5 on one head's statistics (HC_STAT_* order, float64): the first of Sink,
// Dummy, Spatial whose test passes, else Global.
uint8_t decide_label(const hc_config &cfg, const double *st) {
  if (st[HC_STAT_COS_SINK] >= (double)cfg.theta_sink) return HC_SINK;
  if (st[HC_STAT_COS_DUMMY] >= (double)cfg.theta_dummy) return HC_DUMMY;
  if (st[HC_STAT_COS_SPATIAL] >= (double)cfg.theta_spatial &&
      st[HC_STAT_SCORE] >= (double)cfg.theta_score)
    return HC_SPATIAL;
  return HC_GLOBAL;
}

}  // namespace

hc_status hc_classify_heads(hc_ctx *c, int layer, int64_t cur_block, const void *q,
                            const void *k_win, const void *v_win, uint8_t *types_out,
                            double *stats_out, hc_stream stream) try {
  hc_status st = check_layer(c, layer);
  if (st != HC_OK) return st;
  if (!q || !k_win || !v_win || !types_out)
    return fail(c, HC_E_INVAL, "q, k_win, v_win and types_out must not be NULL");
  if (!aligned16(q) || !aligned16(k_win) || !aligned16(v_win))
    return fail(c, HC_E_INVAL, "q, k_win and v_win must be 16-byte aligned");
  const int W = c->cfg.window_blocks, H = c->cfg.n_heads, D = c->cfg.head_dim, L = c->L;
  if (cur_block < W - 1)
    return fail(c, HC_E_STATE, "classification needs a full window (cur_block %lld < W-1 = %d)",
                (long long)cur_block, W - 1);
  HC_HIP(c, hipSetDevice(c->device));
  hipStream_t s = (hipStream_t)stream;
  c->cls_done = false;
  // 1. all heads in Global layout (logical order).  Where the Spatial frames
  //    have no padding columns (grid_w a multiple of 8) a block is stored alike
  //    in both layouts, so the Spatial proxy reads the same copy: the buffer
  //    then has the `lead` keys of zeros around it that halo reads reach.  With
  //    padding columns the proxy gets a copy of its own in the Spatial layout.
  //    (720P: one 464 MB copy, 165 us, instead of two.)
  Layer tmp;
  tmp.types.assign(H, HC_GLOBAL);
  tmp.slot.resize(H);
  for (int h = 0; h < H; ++h) tmp.slot[h] = h;
  const int64_t tkeys = global_buffer_keys(W, L);
  const int64_t lead = c->geo.lead;
  const size_t tbytes = ((size_t)H * tkeys + 2 * lead) * D * 2;
  if ((st = keep(c, c->cls_k, tbytes, s)) != HC_OK || (st = keep(c, c->cls_v, tbytes, s)) != HC_OK)
    return st;
  uint16_t *tk = (uint16_t *)c->cls_k.p + lead * D, *tv = (uint16_t *)c->cls_v.p + lead * D;
  auto copy_window = [&](uint8_t kind, uint16_t *k, uint16_t *v, int64_t keys) {
    Layer t = tmp;
    t.types.assign(H, kind);
    ScatterArgs a = scatter_args(c, t);
    a.cell = 0;                        // the proxy uses the centred-window layout
    a.g_keys = a.sp_keys = keys;
    a.k_g = a.k_sp = k; a.v_g = a.v_sp = v;
    a.src_k = (const uint16_t *)k_win; a.src_v = (const uint16_t *)v_win;
    a.n_src = W;
    for (int i = 0; i < W; ++i) { a.src_slot[i] = (int8_t)i; a.sink_slot[i] = a.dummy_slot[i] = -1; }
    return timed_launch(c, s, HC_K_SCATTER, [&] { return launch_scatter(a, H, s); });
  };
  if ((st = copy_window(HC_GLOBAL, tk, tv, tkeys)) != HC_OK) return st;
  const uint16_t *sk = tk, *sv = tv;
  int64_t sp_stride = tkeys * D;
  if (c->geo.pitch != c->cfg.grid_w) {
    const size_t pbytes = ((size_t)H * c->sp_keys + 2 * lead) * D * 2;
    if ((st = keep(c, c->cls_pk, pbytes, s)) != HC_OK || (st = keep(c, c->cls_pv, pbytes, s)) != HC_OK)
      return st;
    uint16_t *pk = (uint16_t *)c->cls_pk.p + lead * D, *pv = (uint16_t *)c->cls_pv.p + lead * D;
    if ((st = copy_window(HC_SPATIAL, pk, pv, c->sp_keys)) != HC_OK) return st;
    sk = pk; sv = pv;
    sp_stride = c->sp_keys * D;
  }
  // 2. O_ref, O_sink, O_dummy (Eq. 2 and the temporal proxies) in one sweep, O_spatial (r_p)
  const size_t obytes = (size_t)H * L * D * 4;
  for (int i = 0; i < 4; ++i)
    if ((st = keep(c, c->cls_o[i], obytes, s)) != HC_OK) return st;
  float *o_ref = (float *)c->cls_o[0].p, *o_sink = (float *)c->cls_o[1].p;
  float *o_dum = (float *)c->cls_o[2].p, *o_sp = (float *)c->cls_o[3].p;
  {
    const int nqt = (L + kQTile - 1) / kQTile;
    // One sweep: O_ref is the merge of one partial per window block; the
    // temporal proxies are the partials of block 0 (O_sink) and of the
    // current block (O_dummy) normalised on their own, so their keys are not
    // read a second time.
    if ((st = keep(c, c->cls_part, (size_t)H * nqt * W * partial_floats(D) * 4, s)) != HC_OK)
      return st;
    float *part = (float *)c->cls_part.p;
    // the work lists depend on the configuration only: built and uploaded once
    if (c->cls_n_units == 0) {
      std::vector<HeadKV> heads;
      for (int h = 0; h < H; ++h)
        heads.push_back(HeadKV{h, tk + (size_t)h * tkeys * D, tv + (size_t)h * tkeys * D});
      std::vector<DenseUnit> units;
      std::vector<CombineItem> comb;
      plan_classify_units(L, W, heads, units, comb);
      const std::vector<KeyRegion> regions = {{tk, (int64_t)H, tkeys}};
      if (first_unit_outside(units, regions, D) >= 0)
        return fail(c, HC_E_STATE, "internal: a classification unit reads past its head");
      if ((st = upload(c, c->cls_units, units)) != HC_OK || (st = upload(c, c->cls_comb, comb)) != HC_OK)
        return st;
      c->cls_wide = D == 128 && dense_wide_waves(units, c->n_cu, false);
      c->cls_n_units = (int)units.size();
      c->cls_n_comb = (int)comb.size();
    }
    void *d_units = c->cls_units.p, *d_comb = c->cls_comb.p;
    DenseArgs a{};
    a.units = (const DenseUnit *)d_units;
    a.q = (const uint16_t *)q;
    a.o[0] = o_ref; a.o[1] = o_sink; a.o[2] = o_dum;
    a.part = part;
    a.n_units = c->cls_n_units;
    a.L = L;
    a.scale_log2 = c->scale * 1.4426950408889634f;
    a.wide_waves = c->cls_wide;
    st = timed_launch(c, s, HC_K_DENSE,
                      [&] { return launch_dense(a, D, DenseRole::kClassify, s); });
    if (st != HC_OK) return st;
    CombineArgs ca{};
    ca.items = (const CombineItem *)d_comb;
    ca.part = part;
    ca.o[0] = o_ref; ca.o[1] = o_sink; ca.o[2] = o_dum;
    ca.n_items = c->cls_n_comb;
    ca.L = L; ca.D = D;
    SpatialArgs no_splits{};
    no_splits.n_split = 1;
    st = timed_launch(c, s, HC_K_COMBINE, [&] { return launch_merge(ca, no_splits, D, s); });
    if (st != HC_OK) return st;
  }
  {
    SpatialArgs a = spatial_args(c, c->cfg.proxy_radius, W);
    a.q = (const uint16_t *)q;
    a.o = o_sp;
    a.k = sk; a.v = sv;
    a.head_stride = sp_stride;
    a.n_sp = H;
    for (int h = 0; h < H; ++h) a.heads[h] = (int8_t)h;
    st = timed_launch(c, s, HC_K_SPATIAL,
                      [&] { return launch_spatial(a, D, SpatialRole::kClassify, s); });
    if (st != HC_OK) return st;
  }
  // 3. per-token and then per-head statistics on the device (float64), the
  // decision on the host
  const int groups = cls_stat_groups(L);
  if ((st = keep(c, c->cls_tok, (size_t)H * (L + groups * 4 + HC_N_STATS) * sizeof(double), s)) != HC_OK)
    return st;
  double *cos_sp = (double *)c->cls_tok.p;
  double *sums = cos_sp + (size_t)H * L;
  double *head_stats = sums + (size_t)H * groups * 4;
  {
    StatsArgs a{};
    a.o_ref = o_ref; a.o_sink = o_sink; a.o_dummy = o_dum; a.o_sp = o_sp;
    a.cos_sp = cos_sp; a.sums = sums; a.n_heads = H; a.L = L; a.D = D;
    st = timed_launch(c, s, HC_K_STATS, [&] { return launch_stats(a, s); });
    if (st != HC_OK) return st;
    ClsReduceArgs r{};
    r.cos_sp = cos_sp; r.sums = sums; r.out = head_stats;
    r.n_heads = H; r.n_groups = groups; r.L = L; r.D = D;
    r.gamma = (double)c->cfg.gamma;
    st = timed_launch(c, s, HC_K_STATS, [&] { return launch_cls_reduce(r, s); });
    if (st != HC_OK) return st;
  }
  static_assert(HC_N_STATS == 6 && HC_STAT_COS_SINK == 0 && HC_STAT_SCORE == 5,
                "the reduction kernel writes the statistics in HC_STAT order");
  std::vector<double> hstats((size_t)H * HC_N_STATS);
  HC_HIP(c, hipMemcpyAsync(hstats.data(), head_stats, hstats.size() * sizeof(double),
                           hipMemcpyDeviceToHost, s));
  HC_HIP(c, hipStreamSynchronize(s));
  std::vector<uint8_t> labels(H);
  for (int h = 0; h < H; ++h) labels[h] = decide_label(c->cfg, &hstats[(size_t)h * HC_N_STATS]);
  if (stats_out) std::memcpy(stats_out, hstats.data(), hstats.size() * sizeof(double));
  // 4. head table + cache split (Sec. 4.3)
  st = hc_set_head_types(c, layer, labels.data(), cur_block, k_win, v_win, stream);
  if (st != HC_OK) return st;
  // the routed work list is built while the split runs (without memory for it, that
  // is left to the layer's first hc_attention)
  st = ensure_plan(c, c->layers[layer], W, s);
  if (st == HC_E_NOMEM) c->err.clear();
  else if (st != HC_OK) return st;
  HC_HIP(c, hipStreamSynchronize(s));
  std::memcpy(types_out, labels.data(), H);
  c->cls_done = true;
  return HC_OK;
} HC_NO_HOST_MEMORY(c)

hc_status hc_classify_outputs(hc_ctx *c, int which, float *dst, hc_stream stream) {
  if (!c) return HC_E_INVAL;
  if (which < HC_CLS_O_REF || which > HC_CLS_O_SPATIAL)
    return fail(c, HC_E_INVAL, "which = %d is not one of the four classification outputs", which);
  if (!dst || !aligned16(dst)) return fail(c, HC_E_INVAL, "dst must be a 16-byte aligned device pointer");
  if (!c->cls_done)
    return fail(c, HC_E_STATE, "no classification has completed on this context");
  const size_t bytes = (size_t)c->cfg.n_heads * c->L * c->cfg.head_dim * sizeof(float);
  HC_HIP(c, hipSetDevice(c->device));
  HC_HIP(c, hipMemcpyAsync(dst, c->cls_o[which].p, bytes, hipMemcpyDeviceToDevice,
                           (hipStream_t)stream));
  return HC_OK;
}

hc_status hc_memory_bytes(const hc_ctx *c, int64_t *bytes) {
  if (!c || !bytes) return HC_E_INVAL;
  int64_t t = 0;
  for (const auto &l : c->layers)
    t += l.k_sd.bytes + l.v_sd.bytes + l.k_g.bytes + l.v_g.bytes + l.k_sp.bytes + l.v_sp.bytes +
         l.plan.bytes;
  t += c->part.bytes + c->sp_part.bytes + c->sp_ml.bytes + c->cell_off_d.bytes + c->qmap_d.bytes;
  for (const DevBuf *b : {&c->cls_k, &c->cls_v, &c->cls_pk, &c->cls_pv, &c->cls_o[0], &c->cls_o[1],
                          &c->cls_o[2], &c->cls_o[3], &c->cls_part, &c->cls_units, &c->cls_comb,
                          &c->cls_tok})
    t += b->bytes;
  *bytes = t;
  return HC_OK;
}

hc_status hc_profile_enable(hc_ctx *c, int on) {
  if (!c) return HC_E_INVAL;
  c->profile = on != 0;
  return HC_OK;
}

hc_status hc_profile_read(hc_ctx *c, int kind, double *total_ms, int64_t *launches) try {
  if (!c || kind < 0 || kind >= HC_K_COUNT || !total_ms || !launches) return HC_E_INVAL;
  HC_HIP(c, hipSetDevice(c->device));
  for (int k = 0; k < HC_K_COUNT; ++k) {
    // pairs are taken off the pending list as they are read, so a failure
    // leaves each pair in exactly one of the two lists
    auto &pend = c->pending[k];
    while (!pend.empty()) {
      const EventPair e = pend.front();
      HC_HIP(c, hipEventSynchronize(e.b));
      float ms = 0.f;
      HC_HIP(c, hipEventElapsedTime(&ms, e.a, e.b));
      c->prof_ms[k] += ms;
      c->prof_n[k] += 1;
      pend.erase(pend.begin());
      c->pool.push_back(e);
    }
  }
  *total_ms = c->prof_ms[kind];
  *launches = c->prof_n[kind];
  c->prof_ms[kind] = 0;
  c->prof_n[kind] = 0;
  return HC_OK;
} HC_NO_HOST_MEMORY(c)

}  // extern "C"

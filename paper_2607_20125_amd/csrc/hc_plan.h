// Host-side planning of the dense launches (plain C++, no HIP): the keys per
// head of the buffers the dense kernel reads (Sec. 4.3 buffers), the cell
// tables of the cell variant, the work lists of the routed step (Sec. 4.4) and
// of the classification sweep (Sec. 4.2), the check that every unit stays
// inside its head's part of a buffer, and the tail balancing of the unit runs
// the 8 XCDs execute.  Used by the runtime; compiled on its own by the CPU tests.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "hc_units.h"

namespace hc {

inline int64_t round_up_tiles(int64_t keys) { return (keys + kKTile - 1) / kKTile * kKTile; }

// key tiles of a unit (0: padding)
inline int unit_tiles(const DenseUnit &u) { return (u.kv1 - u.kv0 + kKTile - 1) / kKTile; }

// ---------------------------------------------------------------------------
// Keys per head of the buffers the dense kernel reads.  A unit's DMA moves
// whole kKTile-key tiles from kv0, so it reads up to kKTile - 1 keys past kv1:
// with two Sink-Dummy slots the second slot's unit starts at key L and its
// tiles end as late as L + round_up(L) > round_up(2 L) whenever L is not a
// multiple of kKTile.  Every buffer therefore ends each head with one spare tile.
// ---------------------------------------------------------------------------
inline int64_t sd_buffer_keys(int sd_blocks, int64_t L) {
  return round_up_tiles((int64_t)sd_blocks * L) + kKTile;
}
inline int64_t global_buffer_keys(int n_blocks, int64_t L) {
  return round_up_tiles((int64_t)n_blocks * L) + kKTile;
}

// ---------------------------------------------------------------------------
// Cell variant of the Spatial path: round(N / c) cells per axis (halves
// rounded up, at least one); all cells are c wide except the last, which ends
// at N.  A cell's keys are stored slot-major and padded to whole tiles; the
// query map lists the block's tokens cell by cell (frame-major inside a cell).
// ---------------------------------------------------------------------------
inline int n_cells(int N, int c) { return std::max(1, (2 * N + c) / (2 * c)); }

struct CellTables {
  int ncy = 0, ncx = 0;              // cells per column / per row
  std::vector<int64_t> off;          // first key of each cell (row-major cells)
  std::vector<int32_t> q0;           // first entry of each cell in qmap
  std::vector<int32_t> qmap;         // tokens cell by cell
  int64_t keys = 0;                  // keys per head of the cell-major buffer
  int cell_h(int cy, int Hg, int cs) const { return cy == ncy - 1 ? Hg - cy * cs : cs; }
  int cell_w(int cx, int Wg, int cs) const { return cx == ncx - 1 ? Wg - cx * cs : cs; }
};

inline CellTables build_cell_tables(int Hg, int Wg, int F, int W, int cs) {
  CellTables t;
  t.ncy = n_cells(Hg, cs);
  t.ncx = n_cells(Wg, cs);
  int64_t off = 0;
  for (int cy = 0; cy < t.ncy; ++cy)
    for (int cx = 0; cx < t.ncx; ++cx) {
      const int y0 = cy * cs, y1 = y0 + t.cell_h(cy, Hg, cs);
      const int x0 = cx * cs, x1 = x0 + t.cell_w(cx, Wg, cs);
      t.off.push_back(off);
      off += round_up_tiles((int64_t)W * F * (y1 - y0) * (x1 - x0));
      t.q0.push_back((int32_t)t.qmap.size());
      for (int f = 0; f < F; ++f)
        for (int y = y0; y < y1; ++y)
          for (int x = x0; x < x1; ++x) t.qmap.push_back(f * Hg * Wg + y * Wg + x);
    }
  t.keys = off + kKTile;   // the spare tile, as in the other buffers
  return t;
}

// ---------------------------------------------------------------------------
// Work lists.  A head's part of a buffer is given by its K and V bases.
// ---------------------------------------------------------------------------
struct HeadKV {
  int head;
  const uint16_t *k, *v;
};

struct DensePlanShape {
  int d = 128;               // head dimension
  int L = 0;                 // tokens per block
  int nv = 0;                // valid window blocks
  int g_parts = 0;           // key ranges per Global head (0: one per window block)
  int sd_blocks = 1;         // Sink-Dummy slots per head (1 or 2)
  int F = 1, grid_h = 0, grid_w = 0, cell = 0;   // cell variant (cell > 0)
  const CellTables *cells = nullptr;
};

// Keys [*kv0, *kv1) of part p of a Global head's nv L keys: window block p when
// there are as many parts as blocks (or parts is 0), else equal runs of tiles.
inline HC_HD void global_part(int L, int nv, int parts, int p, int32_t *kv0, int32_t *kv1) {
  if (parts == 0 || parts == nv) {
    *kv0 = p * L;
    *kv1 = *kv0 + L;
    return;
  }
  const int64_t keys = (int64_t)nv * L, tiles = (keys + kKTile - 1) / kKTile;
  const int64_t end = kKTile * (tiles * (p + 1) / parts);
  *kv0 = (int32_t)(kKTile * (tiles * p / parts));
  *kv1 = (int32_t)(end < keys ? end : keys);
}

// Dense work of one routed layer: Global heads get one unit per window block
// (or other part of the window) and 128-query tile (partials merged per tile), Sink/Dummy heads one unit per
// tile over their block (per block slot in the two-block variant once a second
// block exists, merged like a Global head), cells one query-mapped unit per
// 128 queries of a cell.  Units are ordered (head, key block, query tile) so
// that neighbouring units read the same K/V.  Then tail-balanced for n_cu CUs.
inline void balance_units(int n_cu, std::vector<DenseUnit> &units, std::vector<CombineItem> &comb,
                          int groups_per_cu = 2);

// Work groups per CU that the balancing counts on.  128-dim heads: the two that are
// resident.  The three of 64-dim heads share the CU's rate, one alone nearly reaching
// it, so what ends a launch is the work per CU, not per group: with one slot per CU 90
// drawn layers took 0.978 of the time with three (0.985 with two), and the layers of
// two to three units per CU that three had made 4-5% slower than two are faster again
// (7552 tokens, 531 units of 118 tiles: 177 us with two, 186 with three, 168 now).
// A launch of fewer units than CUs keeps three, so that its units are cut at all: 234
// units of 78 tiles take 76 us so and 83 uncut.
inline int balance_groups(int d, int n_units, int n_cu) {
  if (d != 64) return dense_groups_per_cu(d);
  return n_units > n_cu ? 1 : dense_groups_per_cu(d);
}

inline void plan_dense_units(const DensePlanShape &s, const std::vector<HeadKV> &global,
                             const std::vector<HeadKV> &sink_dummy,
                             const std::vector<HeadKV> &cell_heads, int n_cu,
                             std::vector<DenseUnit> &units, std::vector<CombineItem> &comb) {
  const int L = s.L, nv = s.nv;
  const int nqt = (L + kQTile - 1) / kQTile;
  units.clear();
  comb.clear();
  const int gp = s.g_parts > 0 ? s.g_parts : nv;
  int slot = 0;
  for (const HeadKV &h : global) {
    for (int part = 0; part < gp; ++part)
      for (int qt = 0; qt < nqt; ++qt) {
        DenseUnit u{};
        u.k = h.k; u.v = h.v; u.head = h.head; u.q0 = qt * kQTile;
        global_part(L, nv, gp, part, &u.kv0, &u.kv1);
        u.slot = gp > 1 ? slot + qt * gp + part : -1;
        units.push_back(u);
      }
    if (gp > 1) {
      for (int qt = 0; qt < nqt; ++qt)
        comb.push_back(CombineItem{h.head, qt * kQTile, slot + qt * gp, gp, 0, 0});
      slot += nqt * gp;
    }
  }
  const int sd_parts = (s.sd_blocks == 2 && nv >= 2) ? 2 : 1;
  for (const HeadKV &h : sink_dummy) {
    for (int part = 0; part < sd_parts; ++part)
      for (int qt = 0; qt < nqt; ++qt) {
        DenseUnit u{};
        u.k = h.k; u.v = h.v; u.head = h.head; u.q0 = qt * kQTile;
        u.kv0 = part * L; u.kv1 = (part + 1) * L;
        u.slot = sd_parts > 1 ? slot + qt * sd_parts + part : -1;
        units.push_back(u);
      }
    if (sd_parts > 1) {
      for (int qt = 0; qt < nqt; ++qt)
        comb.push_back(CombineItem{h.head, qt * kQTile, slot + qt * sd_parts, sd_parts, 0, 0});
      slot += nqt * sd_parts;
    }
  }
  if (s.cell > 0 && s.cells) {
    const CellTables &t = *s.cells;
    for (const HeadKV &h : cell_heads)
      for (int cy = 0; cy < t.ncy; ++cy)
        for (int cx = 0; cx < t.ncx; ++cx) {
          const int id = cy * t.ncx + cx;
          const int area = t.cell_h(cy, s.grid_h, s.cell) * t.cell_w(cx, s.grid_w, s.cell);
          const int nq = s.F * area;
          for (int q = 0; q < nq; q += kQTile) {
            DenseUnit u{};
            u.k = h.k; u.v = h.v; u.head = h.head; u.q0 = t.q0[id] + q;
            u.kv0 = (int32_t)t.off[id];
            u.kv1 = u.kv0 + nv * s.F * area;
            u.slot = -1;
            u.qn = std::min(kQTile, nq - q);
            units.push_back(u);
          }
        }
  }
  balance_units(n_cu, units, comb, balance_groups(s.d, (int)units.size(), n_cu));
}

// ---------------------------------------------------------------------------
// The same routed work list (before tail balancing) as a closed form of the
// unit index, for plans built on the device (hc_attention_static): unit i and
// merge item i of a layer from the head lists and buffer bases alone.  The
// order is plan_dense_units' (Global heads, then Sink/Dummy heads).
// ---------------------------------------------------------------------------
struct StaticPlan {
  const uint16_t *k_g, *v_g, *k_sd, *v_sd;   // buffer bases; head slot s at s * keys * d
  int64_t g_keys, sd_keys;
  int32_t d, L, nv, nqt, sd_parts, n_g, n_sd;
  int32_t g_parts;                           // key ranges per Global head (0: one per block)
  int8_t g_head[64], sd_head[64];            // head id of each buffer slot
};

inline HC_HD int static_g_parts(const StaticPlan &p) { return p.g_parts > 0 ? p.g_parts : p.nv; }
inline HC_HD int static_n_units(const StaticPlan &p) {
  return (p.n_g * static_g_parts(p) + p.n_sd * p.sd_parts) * p.nqt;
}
inline HC_HD int static_n_comb(const StaticPlan &p) {
  return ((static_g_parts(p) > 1 ? p.n_g : 0) + (p.sd_parts > 1 ? p.n_sd : 0)) * p.nqt;
}
inline HC_HD int static_n_slots(const StaticPlan &p) {
  const int gp = static_g_parts(p);
  return ((gp > 1 ? p.n_g * gp : 0) + (p.sd_parts > 1 ? p.n_sd * p.sd_parts : 0)) * p.nqt;
}

// Its place in the scratch: units, merge items and partial slots, each 256-byte aligned.
inline size_t align256(size_t b) { return (b + 255) / 256 * 256; }
inline size_t static_list_bytes(const StaticPlan &p) {
  return align256((size_t)static_n_units(p) * sizeof(DenseUnit)) +
         align256((size_t)static_n_comb(p) * sizeof(CombineItem));
}
inline size_t static_dense_bytes(const StaticPlan &p) {
  return static_list_bytes(p) + align256((size_t)static_n_slots(p) * partial_floats(p.d) * sizeof(float));
}
// Slots that fit beside the longest list, of kMaxSrcBlocks ranges per Global head.
inline int64_t static_max_slots(StaticPlan p, size_t scratch) {
  p.g_parts = kMaxSrcBlocks;
  const size_t list = static_list_bytes(p) + 256;
  return list < scratch ? (int64_t)((scratch - list) / ((size_t)partial_floats(p.d) * sizeof(float))) : 0;
}

inline HC_HD DenseUnit static_dense_unit(const StaticPlan &p, int i) {
  DenseUnit u{};
  const int gp = static_g_parts(p);
  const int ng_units = p.n_g * gp * p.nqt;
  const int g_slots = gp > 1 ? ng_units : 0;
  if (i < ng_units) {                         // Global: (head, part, query tile)
    const int qt = i % p.nqt, part = (i / p.nqt) % gp, gi = i / (p.nqt * gp);
    u.k = p.k_g + (int64_t)gi * p.g_keys * p.d;
    u.v = p.v_g + (int64_t)gi * p.g_keys * p.d;
    u.head = p.g_head[gi];
    global_part(p.L, p.nv, gp, part, &u.kv0, &u.kv1);
    u.slot = gp > 1 ? gi * p.nqt * gp + qt * gp + part : -1;
    u.q0 = qt * kQTile;
  } else {                                    // Sink/Dummy: (head, block slot, query tile)
    const int j = i - ng_units;
    const int qt = j % p.nqt, part = (j / p.nqt) % p.sd_parts, si = j / (p.nqt * p.sd_parts);
    u.k = p.k_sd + (int64_t)si * p.sd_keys * p.d;
    u.v = p.v_sd + (int64_t)si * p.sd_keys * p.d;
    u.head = p.sd_head[si];
    u.kv0 = part * p.L;
    u.kv1 = u.kv0 + p.L;
    u.slot = p.sd_parts > 1 ? g_slots + si * p.nqt * p.sd_parts + qt * p.sd_parts + part : -1;
    u.q0 = qt * kQTile;
  }
  return u;
}

inline HC_HD CombineItem static_comb_item(const StaticPlan &p, int i) {
  const int gp = static_g_parts(p);
  const int ng_items = gp > 1 ? p.n_g * p.nqt : 0;
  const int g_slots = gp > 1 ? p.n_g * gp * p.nqt : 0;
  CombineItem it{};
  if (i < ng_items) {
    const int qt = i % p.nqt, gi = i / p.nqt;
    it.head = p.g_head[gi];
    it.q0 = qt * kQTile;
    it.slot0 = gi * p.nqt * gp + qt * gp;
    it.n_slots = gp;
  } else {
    const int j = i - ng_items;
    const int qt = j % p.nqt, si = j / p.nqt;
    it.head = p.sd_head[si];
    it.q0 = qt * kQTile;
    it.slot0 = g_slots + si * p.nqt * p.sd_parts + qt * p.sd_parts;
    it.n_slots = p.sd_parts;
  }
  return it;
}

// Key ranges per Global head: one for windows of at most 12 key tiles (24 with
// 64-dim heads), else one per window block.  Up to there the merge launch of the
// ranges' partials takes longer than the tiles it saves: append and attention of
// six Global and six Sink/Dummy heads, one range against one per block, take 19.5
// against 22.0 us at 8 tiles, 20.0 against 22.0 at 12 and 23.6 against 22.4 at 16;
// 64-dim heads 19.5 against 22.4 at 16 and 22.4 both at 32.  (Not asked where split
// Spatial heads or two-block Sink/Dummy heads bring the merge launch anyway: with
// three blocks of 256 tokens and two-block heads one range took 25.8 us, one per
// block 22.2.)
inline int global_parts(int d, int L, int nv) {
  return ((int64_t)nv * L + kKTile - 1) / kKTile <= (d == 64 ? 24 : 12) ? 1 : nv;
}

// The classification sweep (Sec. 4.2): per head one unit per window block and
// query tile over the window in Global layout; O_ref is the merge of all W
// partials of a tile (output 0), O_sink the block-0 partial (output 1) and
// O_dummy the current-block partial (output 2), each normalised on its own.
inline void plan_classify_units(int L, int W, const std::vector<HeadKV> &heads,
                                std::vector<DenseUnit> &units, std::vector<CombineItem> &comb) {
  const int nqt = (L + kQTile - 1) / kQTile;
  units.clear();
  comb.clear();
  for (int hi = 0; hi < (int)heads.size(); ++hi) {
    const HeadKV &h = heads[hi];
    for (int blk = 0; blk < W; ++blk)
      for (int qt = 0; qt < nqt; ++qt) {
        DenseUnit u{};
        u.k = h.k; u.v = h.v; u.head = h.head; u.q0 = qt * kQTile;
        u.kv0 = blk * L; u.kv1 = (blk + 1) * L;
        u.slot = (hi * nqt + qt) * W + blk;
        units.push_back(u);
      }
    for (int qt = 0; qt < nqt; ++qt) {
      const int s0 = (hi * nqt + qt) * W;
      comb.push_back(CombineItem{h.head, qt * kQTile, s0, W, 0, 0});
      comb.push_back(CombineItem{h.head, qt * kQTile, s0, 1, 1, 0});
      comb.push_back(CombineItem{h.head, qt * kQTile, s0 + W - 1, 1, 2, 0});
    }
  }
}

// ---------------------------------------------------------------------------
// Every tile a unit's DMA reads (whole kKTile-key tiles from kv0) must lie
// inside its head's part of a buffer.  A buffer is n_heads parts of `keys`
// keys of d elements from `base`; a unit's k must be the base of one part.
// Addresses are compared as integers (no buffer is dereferenced).
// ---------------------------------------------------------------------------
struct KeyRegion {
  const uint16_t *base;
  int64_t n_heads, keys;
};

// keys of the part u.k starts, or -1 when u.k is no part's base
inline int64_t unit_region_keys(const DenseUnit &u, const std::vector<KeyRegion> &regions, int d) {
  const uintptr_t k = reinterpret_cast<uintptr_t>(u.k);
  for (const KeyRegion &r : regions) {
    const uintptr_t b = reinterpret_cast<uintptr_t>(r.base);
    const uintptr_t part = (uintptr_t)r.keys * d * sizeof(uint16_t);
    if (!r.base || part == 0 || k < b || k >= b + part * r.n_heads) continue;
    if ((k - b) % part == 0) return r.keys;
  }
  return -1;
}

// one past the last key a unit's DMA reads
inline int64_t unit_read_end(const DenseUnit &u) {
  return u.kv0 + round_up_tiles((int64_t)u.kv1 - u.kv0);
}

// index of the first unit (padding units aside) that reads outside its head's
// part, or -1 when all stay inside
inline int first_unit_outside(const std::vector<DenseUnit> &units,
                              const std::vector<KeyRegion> &regions, int d) {
  for (size_t i = 0; i < units.size(); ++i) {
    const DenseUnit &u = units[i];
    if (u.head < 0) continue;
    const int64_t keys = unit_region_keys(u, regions, d);
    if (keys < 0 || u.kv0 < 0 || u.kv1 < u.kv0 || unit_read_end(u) > keys) return (int)i;
  }
  return -1;
}

// ---------------------------------------------------------------------------
// Tail balancing of a dense launch.  Work groups are dealt round-robin to the
// 8 XCDs and the kernel maps them so that XCD x runs a contiguous run of the
// unit list in order, `groups_per_cu` per CU at a time (balance_groups).  With equal units the
// last round of a run is partly empty.  For each run, the tail (its last
// partial round, or that plus one full round) is cut into pieces of whole key
// tiles when a list-scheduling simulation says the run then ends earlier; each
// piece writes a partial slot and the pieces are merged by the combine kernel
// like the per-block partials of a Global head.  Runs are padded with no-op
// units (head < 0) to one length so the mapping stays run x -> XCD x.
// ---------------------------------------------------------------------------
namespace plan_detail {

constexpr double kUnitOverheadTiles = 4.0;   // fixed cost of a unit (Q load, fill, store)
constexpr int kMinPieceTiles = 12;
constexpr int kMaxPieces = 8;

// Free times of an XCD's work-group slots: each added unit goes to the slot that
// is free first.  A copy continues from the same state.
struct SlotClock {
  std::vector<double> free_at;   // min-heap
  double end = 0.0;              // when the last unit ends
  explicit SlotClock(int slots) : free_at(slots, 0.0) {}
  void add(double cost) {
    const double t = free_at[0] + cost;
    const size_t n = free_at.size();
    size_t i = 0;
    for (size_t c = 1; c < n; c = 2 * i + 1) {   // sift the new time down from the root
      if (c + 1 < n && free_at[c + 1] < free_at[c]) ++c;
      if (free_at[c] >= t) break;
      free_at[i] = free_at[c];
      i = c;
    }
    free_at[i] = t;
    end = std::max(end, t);
  }
};

// Pieces a unit of a cut suffix is cut into when k are asked for: none if they
// would have fewer than kMinPieceTiles tiles each.
inline int unit_pieces(const DenseUnit &u, int k) {
  return u.qn == 0 && unit_tiles(u) >= k * kMinPieceTiles ? k : 1;
}

// How the run [b, e) of the unit list is cut: the suffix length *best_j and the
// pieces *best_k per unit of it that end the run earliest by at least 1%, else
// 0 and 1.  The uncut units before a suffix are simulated once: the clock is
// copied where a suffix starts and each number of pieces continues from the
// copy, until it is past the best end so far.  `most` (or null): the pieces each
// unit may have.
inline void best_cut(const std::vector<DenseUnit> &units, const int *most, int b, int e, int slots,
                     int *best_j, int *best_k) {
  const int tail = (e - b) % slots;
  SlotClock clock(slots), at_long = clock, at_short = clock;
  for (int i = b; i < e; ++i) {
    if (e - i == tail + slots) at_long = clock;
    if (e - i == tail) at_short = clock;
    clock.add(unit_tiles(units[i]) + kUnitOverheadTiles);
  }
  double best = clock.end;
  *best_j = 0;
  *best_k = 1;
  for (int j : {tail, tail + slots}) {
    if (j <= 0 || j > e - b) continue;
    for (int k = 2; k <= kMaxPieces; ++k) {
      SlotClock cl = j == tail ? at_short : at_long;
      for (int i = e - j; i < e && cl.end < best * 0.99; ++i) {
        const int nt = unit_tiles(units[i]);
        const int kk = unit_pieces(units[i], most ? std::min(k, most[i]) : k);
        for (int p = 0; p < kk; ++p)
          cl.add((nt * (p + 1) / kk - nt * p / kk) + kUnitOverheadTiles);
      }
      if (cl.end < best * 0.99) { best = cl.end; *best_j = j; *best_k = k; }
    }
  }
}

}  // namespace plan_detail

// n_cu: compute units of the device (a multiple of 8; otherwise the list is left as is).
inline void balance_units(int n_cu, std::vector<DenseUnit> &units, std::vector<CombineItem> &comb,
                          int groups_per_cu) {
  using namespace plan_detail;
  const int n = (int)units.size();
  if (n_cu <= 0 || n_cu % 8 != 0 || n == 0) return;
  const int slots = groups_per_cu * n_cu / 8;
  // item of every unit: the combine item holding its slot, or -1 (writes o)
  std::vector<int> item(n, -1);
  {
    std::vector<int> of_slot;
    for (int i = 0; i < (int)comb.size(); ++i)
      for (int j = 0; j < comb[i].n_slots; ++j) {
        const int sl = comb[i].slot0 + j;
        if (sl >= (int)of_slot.size()) of_slot.resize(sl + 1, -1);
        of_slot[sl] = i;
      }
    for (int i = 0; i < n; ++i)
      if (units[i].slot >= 0) item[i] = of_slot[units[i].slot];
  }
  std::vector<int> item_n(comb.size());
  for (size_t i = 0; i < comb.size(); ++i) item_n[i] = comb[i].n_slots;
  // pieces per unit that an item of at most kMaxSrcBlocks slots has room for when
  // all its units are cut
  std::vector<int> most(n);
  for (int i = 0; i < n; ++i) most[i] = item[i] < 0 ? kMaxSrcBlocks : kMaxSrcBlocks / item_n[item[i]];

  struct Piece { DenseUnit u; int item; };
  std::vector<std::vector<Piece>> runs(8);
  const int per = n / 8, rem = n % 8;
  size_t longest = 0;
  int prev_b = 0, prev_e = -1, best_j = 0, best_k = 1;
  for (int x = 0; x < 8; ++x) {
    const int b = x * per + std::min(x, rem), e = b + per + (x < rem ? 1 : 0);
    const int m = e - b;
    // best (suffix length j, pieces k) by simulated end time; a run with the
    // same units as the one before (most runs of a layer) takes its answer.
    // A list of 2040 units is planned in 0.20 ms, of 976 in 0.12 ms (0.75 and
    // 0.43 ms with every run and suffix simulated from its first unit).
    auto same = [&](int i, int o) {
      return unit_tiles(units[i]) == unit_tiles(units[o]) && (units[i].qn == 0) == (units[o].qn == 0);
    };
    bool again = m == prev_e - prev_b;
    for (int i = 0; again && i < m; ++i) again = same(b + i, prev_b + i);
    if (!again) best_cut(units, nullptr, b, e, slots, &best_j, &best_k);
    prev_b = b;
    prev_e = e;
    // where an item has no room for its units' pieces, the run is cut again with
    // the room shared out evenly: giving it out first come first served left
    // single units whole at the end of a run (up to 1.9x the run's uncut time)
    int cut_j = best_j, cut_k = best_k;
    const int *limit = nullptr;
    auto grow = [&](int sign) {
      bool fits = true;
      for (int i = e - cut_j; i < e; ++i)
        if (item[i] >= 0) {
          item_n[item[i]] += sign * (unit_pieces(units[i], cut_k) - 1);
          fits = fits && item_n[item[i]] <= kMaxSrcBlocks;
        }
      return fits;
    };
    const bool fits = grow(1);
    grow(-1);
    if (!fits) {
      limit = most.data();
      best_cut(units, limit, b, e, slots, &cut_j, &cut_k);
    }
    std::vector<Piece> &r = runs[x];
    for (int i = b; i < e; ++i) {
      const DenseUnit &u = units[i];
      const int nt = unit_tiles(u);
      int k = i >= e - cut_j ? unit_pieces(u, limit ? std::min(cut_k, limit[i]) : cut_k) : 1;
      if (k > 1 && item[i] >= 0 && item_n[item[i]] + k - 1 > kMaxSrcBlocks) k = 1;
      if (k == 1) { r.push_back({u, item[i]}); continue; }
      int it = item[i];
      if (it < 0) {               // a unit writing o directly gets an item of its own
        it = (int)comb.size();
        comb.push_back(CombineItem{u.head, u.q0, 0, 0, u.out_sel, 0});
        item_n.push_back(1);
      }
      item_n[it] += k - 1;
      for (int p = 0; p < k; ++p) {
        DenseUnit q = u;
        q.kv0 = u.kv0 + kKTile * (nt * p / k);
        q.kv1 = std::min(u.kv1, u.kv0 + kKTile * (nt * (p + 1) / k));
        r.push_back({q, it});
      }
    }
    longest = std::max(longest, r.size());
  }
  // slots: consecutive per item
  std::vector<int> next(comb.size());
  int slot = 0;
  for (size_t i = 0; i < comb.size(); ++i) {
    comb[i].slot0 = slot;
    comb[i].n_slots = item_n[i];
    next[i] = slot;
    slot += item_n[i];
  }
  units.clear();
  for (int x = 0; x < 8; ++x) {
    for (Piece &p : runs[x]) {
      p.u.slot = p.item >= 0 ? next[p.item]++ : -1;
      units.push_back(p.u);
    }
    DenseUnit none{};
    none.head = -1;
    for (size_t i = runs[x].size(); i < longest; ++i) units.push_back(none);
  }
}

// ---------------------------------------------------------------------------
// How long a dense launch takes, from its work list: every XCD runs its part of the
// list in order on its CUs, and work groups that share a CU share its rate, so the
// time follows the end with one slot per CU.  Where the last groups are alone on
// their CUs they do not reach the full rate, by which it leans towards the end with
// two slots (`lone`; the kernel with one wave per SIMD gets half the rate alone, so
// for it two slots are the whole answer).  A unit costs its key tiles and a fixed
// number of tiles on top.  Fitted to forced key ranges on both 128-dim kernels and
// the 64-dim one (45 layers of 440 to 10800 tokens, 1 to 8 blocks, 1 to 16 Global
// heads, 1 to 16 ranges: some 700 times, 3-4% rms).
// ---------------------------------------------------------------------------
struct DenseCost {
  double tile_us;      // a key tile of 128 queries on a CU
  double unit_tiles;   // fixed cost of a unit in tiles
  double lone;
};
inline constexpr DenseCost kCost64 = {0.369, 4.0, 0.2};
inline constexpr DenseCost kCost128 = {0.619, 2.0, 0.3};        // 32 queries per wave
inline constexpr DenseCost kCostWide128 = {0.564, 5.0, 1.0};    // 64 queries per wave

// A merge launch, and one slot's way through memory (33 and 66 KB), in us.
inline constexpr double merge_launch_us(int d) { return d == 64 ? 4.0 : 5.3; }
inline constexpr double merge_slot_us(int d) { return d == 64 ? 0.0070 : 0.0202; }

// When the slots of an XCD are free, as groups of slots with the same time: `count`
// units of one cost go to the slots that are free first, a group at a time.
struct SlotGroups {
  static constexpr int kMax = 256;
  double at[kMax];     // ascending
  int n[kMax];
  int groups = 1;
  double end = 0.0;
  explicit SlotGroups(int slots) { at[0] = 0.0; n[0] = slots; }
  void add(double cost, int64_t count) {
    while (count > 0) {
      const int k = (int)std::min<int64_t>(count, n[0]);
      const double t = at[0] + cost;
      if (k < n[0]) {
        n[0] -= k;
      } else {
        --groups;
        std::copy(at + 1, at + 1 + groups, at);
        std::copy(n + 1, n + 1 + groups, n);
      }
      int i = groups;
      while (i > 0 && at[i - 1] > t) --i;
      if (i > 0 && at[i - 1] == t) {
        n[i - 1] += k;
      } else {
        std::copy_backward(at + i, at + groups, at + groups + 1);
        std::copy_backward(n + i, n + groups, n + groups + 1);
        at[i] = t;
        n[i] = k;
        ++groups;
      }
      end = std::max(end, t);
      count -= k;
    }
  }
};

// Time of a launch of n_units units in list order.  tiles(i, e, &same): the key tiles
// of unit i (0: padding) and how many units from i on have as many, counted as far as
// e at least.
template <class Tiles>
inline double dense_us(const DenseCost &c, int n_units, int n_cu, Tiles &&tiles) {
  const int cus = n_cu / 8, per = n_units / 8, rem = n_units % 8;
  double one = 0.0, two = 0.0;
  for (int x = 0; x < 8; ++x) {
    const int b = x * per + std::min(x, rem), e = b + per + (x < rem ? 1 : 0);
    SlotGroups g1(cus), g2(2 * cus);
    bool alike = true;
    for (int i = b, same = 0; i < e; i += same) {
      const int nt = tiles(i, e, &same);
      alike = alike && i == b && same >= n_units - b;
      same = std::min(same, e - i);
      if (nt == 0) continue;
      if (c.lone < 1.0) g1.add(nt + c.unit_tiles, same);
      g2.add(nt + c.unit_tiles, same);
    }
    one = std::max(one, g1.end);
    two = std::max(two, g2.end);
    if (alike) break;            // the runs after this one hold the same units, and no more
  }
  return c.tile_us * ((1.0 - c.lone) * one + c.lone * 2.0 * two);
}

// Device counts that the estimates cover.
inline bool dense_us_covers(int n_cu) {
  return n_cu > 0 && n_cu % 8 == 0 && n_cu / 4 <= SlotGroups::kMax;
}

// Whether a dense launch of 128-dim heads may run on waves of 64 queries, by its key
// tiles (over all units): from 96 per resident work group (two per CU) on.  There the
// estimate decides.  On a full GPU it is the faster kernel (less energy per product:
// 115 tiles per group 0.95 of the time of 32-query waves, 16 heads, L = 4680; 600 and
// more 0.93), but it has one wave per SIMD and two per work group, so a CU left with one
// group uses half its SIMDs, and a unit's start and end weigh more: below the line 5
// tiles per group took 1.27 (12 heads, L = 1320), 48 1.07 (4 Global heads, L = 2688, 7
// blocks), 75 1.06 (2 Global heads, L = 4680); above it lists whose last rounds are not
// full 1.03-1.19.
inline bool dense_wide_waves(int64_t tiles, int n_cu) {
  return tiles >= (int64_t)96 * dense_groups_per_cu(128) * n_cu;
}

// The same for a list as it is launched: 200 against 208 us for 8 Global heads of six
// blocks of 2856 tokens, whose cut tails end unevenly.  Tail-balanced lists of 120 tiles
// per group or more are not estimated (3-20 us, which a classification waits for): all
// 39 drawn ones ran in 0.94-1.01 of the time.
inline bool dense_wide_waves(const std::vector<DenseUnit> &units, int n_cu, bool balanced) {
  int64_t tiles = 0;
  for (const DenseUnit &u : units) tiles += unit_tiles(u);
  if (!dense_wide_waves(tiles, n_cu)) return false;
  if (!dense_us_covers(n_cu) || (balanced && tiles >= (int64_t)120 * dense_groups_per_cu(128) * n_cu))
    return true;
  auto tiles_of = [&](int i, int e, int *same) {
    const int nt = unit_tiles(units[i]);
    int j = i + 1;
    while (j < e && unit_tiles(units[j]) == nt) ++j;
    *same = j - i;
    return nt;
  };
  return dense_us(kCostWide128, (int)units.size(), n_cu, tiles_of) <=
         dense_us(kCost128, (int)units.size(), n_cu, tiles_of);
}

// The device-built work list of the no-allocation call: its key ranges per Global head
// and the kernel it runs on.
struct StaticChoice {
  int parts;
  bool wide;
};

inline double static_dense_us(const StaticPlan &p, const DenseCost &c, int n_cu) {
  const int gp = static_g_parts(p), ng = p.n_g * gp * p.nqt, n = static_n_units(p);
  const bool equal = gp == 1 || gp == p.nv;
  return dense_us(c, n, n_cu, [&](int i, int, int *same) {
    if (i >= ng) {
      *same = n - i;
      return (p.L + kKTile - 1) / kKTile;
    }
    *same = equal ? ng - i : p.nqt - i % p.nqt;
    int32_t kv0, kv1;
    global_part(p.L, p.nv, gp, (i / p.nqt) % gp, &kv0, &kv1);
    const int nt = (kv1 - kv0 + kKTile - 1) / kKTile;
    if (equal && nt == (p.L + kKTile - 1) / kKTile) *same = n - i;
    return nt;
  });
}

// This list is not tail-balanced, so its last round may be nearly empty; other ranges
// than one per block then end earlier (480P, three Global, seven Sink/Dummy and two
// Spatial heads: 1036 units in three rounds of 512 take 373 us, six ranges 350, and
// 334 with 64 queries per wave), and so may waves of 32 queries (four Global and eight
// Sink/Dummy heads of two 480P blocks: 203 against 231 us).  The estimate decides
// both, with at most max_slots partial slots.  One range per block stays unless
// another count is 2% faster, and 9% where that is fewer, longer ranges with 64
// queries per wave: those are estimated up to 6% too fast (6912 tokens, four blocks,
// three ranges 473 us against 469).  15 us stand for the rest of the call.  Windows
// that hc_attention leaves uncut are left uncut here.  Counts whose perfectly packed
// list would not be faster are passed over unsimulated: 0-50 us a choice on one CPU
// (30-420 us with every count simulated unit by unit).
inline StaticChoice static_choice(StaticPlan p, int n_cu, int64_t max_slots, bool merged_anyway) {
  constexpr double kGain = 0.02, kWideLongGain = 0.09, kRest = 15.0;
  const int small = merged_anyway ? p.nv : global_parts(p.d, p.L, p.nv);
  const int64_t l_tiles = (p.L + kKTile - 1) / kKTile, w_tiles = ((int64_t)p.nv * p.L + kKTile - 1) / kKTile;
  const int64_t tiles = (p.n_g * w_tiles + (int64_t)p.n_sd * p.sd_parts * l_tiles) * p.nqt;
  const bool may_wide = p.d == 128 && dense_wide_waves(tiles, n_cu);
  if (!dense_us_covers(n_cu) || static_n_units(p) == 0) return {small, may_wide};
  const DenseCost &cost = p.d == 64 ? kCost64 : kCost128;
  auto merge_us = [&] {
    const int ns = static_n_slots(p);
    return (ns > 0 || merged_anyway ? merge_launch_us(p.d) : 0.0) + ns * merge_slot_us(p.d);
  };
  auto packed_us = [&](const DenseCost &c) {
    return c.tile_us * (tiles + c.unit_tiles * static_n_units(p)) / n_cu;
  };
  StaticChoice best = {small, false};
  double best_us = 1e30;
  auto take = [&](const DenseCost &c, bool wide, double at_most) {   // p.g_parts on this kernel
    if (packed_us(c) + merge_us() >= at_most) return;
    const double t = static_dense_us(p, c, n_cu) + merge_us();
    if (t < at_most) { best = {p.g_parts, wide}; best_us = t; }
  };
  p.g_parts = small;
  take(cost, false, best_us);
  if (may_wide) take(kCostWide128, true, best_us);
  if (p.n_g == 0 || small < p.nv) return best;
  const double base_us = best_us;
  for (int parts = 1; parts <= std::min<int64_t>(kMaxSrcBlocks, w_tiles); ++parts) {
    p.g_parts = parts;
    if (parts == p.nv || static_n_slots(p) > max_slots) continue;
    const double at_most = best_us - kGain * (best_us + kRest);
    take(cost, false, at_most);
    if (may_wide)
      take(kCostWide128, true,
           std::min(best.parts == parts ? best_us : at_most,
                    parts < p.nv ? base_us - kWideLongGain * (base_us + kRest) : 1e30));
  }
  return best;
}

}  // namespace hc

// Dense softmax attention of 128-query tiles over a contiguous key range for
// 128-dim heads: Global path (the whole window), Sink/Dummy paths (one block),
// cells, and the classification proxies O_ref, O_sink, O_dummy (Sec. 4.4, Eq. 2).
#include "hc_device.h"

namespace hc {
namespace {
using namespace dev;

// ---------------------------------------------------------------------------
// One work group = kQTile (128) queries of one unit on two waves of 64; two
// work groups share a CU (2 x 80 KB of LDS), one wave per SIMD.
//
// What bounds it: the matrix cores run at the clock that the board's power
// allows (1.6-1.8 GHz under this load against 2.4), so energy counts as much as
// idle cycles.  With 32 queries per wave every K and V operand read from LDS
// fed one product, four waves read the same tiles, and the full-window 720P
// layer kept its matrix cores busy 76% of the time at 1.61 GHz.  With 64 queries
// per wave each read feeds two products: half the LDS traffic, and 75% at 1.71
// GHz.  720P full-window layer 4.31 -> 4.09 ms (1.23 PFLOP/s on that box), routed
// layer 1.21 -> 1.12 ms, fill phase at 480P 408 -> 394 us.
//
// Registers: 128 accumulators and the 64 of Q live in AGPRs, two score sets of
// 64 and the probabilities in VGPRs.  The compiler puts the results of all MFMA
// builtins into one file or the other (AGPRs for this source, whose build leaves
// out the VGPR form the others use), and with scores in AGPRs every one is
// copied out; so the score products are inline assembly with the file in the
// constraint.  The compiler knows nothing of their latency: the source has no vector
// instruction touch a score before ten more slots are issued or `settle` has
// waited, and packs a probability at least one slot before the product that
// reads it.  The compiler may still copy scores ahead of `settle` (it does, behind
// the last products of a partial step, 20 wait states after the nearest), so
// tests/test_dense128_scores.py walks the built instructions from every such product.
//
// One wave per SIMD has nobody to hide behind, so the order is written out: a
// step is 32 slots of two products each (16 of S(t+1) = K(t+1) Q^T, 16 of O +=
// V(t) P(t)), each with one pair of probabilities (two multiplies, two exp2, one
// pack of the pair before) and one operand read three slots ahead; scheduling
// fences keep it.  The softmax of tile t+1 begins in the last slots of PV(t), so
// every slot has the same vector work.  Both exp2 between the two products
// measured best: one between and one after 5% slower, both after 6%.  The only
// barrier of a step sits between its two halves; the first operand reads of the
// second half are issued before it, but it waits for them too (__syncthreads drains
// the LDS counter).  The DMA of K(t+3) and V(t+2) follows
// it four instructions at a time (all at once, two or one at a time: 0.5-2% slower).
// ---------------------------------------------------------------------------
constexpr int kPre = 6;      // pairs of the next tile formed during PV: 5 would leave the
                             // last pair's pack right before the product that reads it
constexpr int kAhead = 3;    // operand reads in flight
constexpr int kCheckTile = 8;   // units of 4 kCheckTile tiles or more look at their row sums here

__device__ __forceinline__ void mfma_score(f32x16 &c, bf16x8 a, const bf16x8 &q, bool first) {
  if (first) asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "a"(q));
  else asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "a"(q));
}
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }

// kRole only separates the symbols of the callers in profiles: 0 routed step,
// 1 full-window step (all heads Global), 2 classification, 3 routed step of a
// context with the cell or two-block variant, 4 a table of Sink and Dummy heads only.
template <int kRole>
__global__ __launch_bounds__(128, 1) void attn_dense128_kernel(DenseArgs a) {
  constexpr int D = 128, NW = 2, NQB = 2, KT = kKTile, NKK = D / 16, NDB = D / 32;
  constexpr int CPR = D / 8;                 // 16-byte chunks per K row
  constexpr int RPI = 64 / CPR;              // K rows per 1 KB wave instruction
  constexpr int TILE = KT * D;               // elements per tile
  constexpr int LPW = TILE / 512 / NW;       // 1 KB instructions per wave per tensor
  constexpr int RK = 2, RV = 3;              // ring buffers
  static_assert(kQTile == 32 * NW * NQB && LPW == 8, "unit shape");
  static_assert((RK + RV) * TILE * 2 * dense_groups_per_cu(D) <= 160 * 1024, "LDS of a CU");
  __shared__ __attribute__((aligned(1024))) uint16_t sK[RK][TILE];
  __shared__ __attribute__((aligned(1024))) uint16_t sV[RV][TILE];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, g = lane >> 5;
  const DenseUnit u = a.units[xcd_unit(blockIdx.x, a.n_units)];
  if (u.head < 0) return;                    // padding of the unit list: no work
  const int L = a.L;

  // this lane's queries: rows wave 64 + 32 qb + n of the unit
  bool rvalid[NQB];
  int row[NQB];
  bf16x8 qf[NQB][NKK];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int lrow = wave * 64 + qb * 32 + n;
    if (u.qn > 0) {
      rvalid[qb] = lrow < u.qn;
      row[qb] = a.qmap[u.q0 + (rvalid[qb] ? lrow : 0)];
    } else {
      row[qb] = u.q0 + lrow;
      rvalid[qb] = row[qb] < L;
    }
    const uint16_t *qp = a.q + ((size_t)u.head * L + (rvalid[qb] ? row[qb] : L - 1)) * D;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) qf[qb][kk] = ld_g16(qp + 16 * kk + 8 * g);
  }
  // Q in its registers before any DMA is issued (the compiler cannot count the DMAs)
  wait_vmcnt<0>();
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) asm volatile("" : "+a"(qf[qb][kk]));
  const float sl2 = a.scale_log2;             // logits in log2 units: s * scale * log2(e)

  const int nkeys = u.kv1 - u.kv0;
  const int nt = (nkeys + KT - 1) / KT;       // at least 1: no unit is empty
  const int rem_last = nkeys - (nt - 1) * KT; // keys in the last tile
  const uint16_t *kbase = u.k + (size_t)u.kv0 * D;
  const uint16_t *vbase = u.v + (size_t)u.kv0 * D;

  // DMA sources of this wave's LPW instructions per tensor, in bytes: K rows
  // permuted and swizzled (kperm, kswz), the V tile in order.  Instruction j
  // also adds 1024 j through its immediate offset or base, so it is taken off
  // here; the K base is taken 8 KB lower (and added back here) so that no offset
  // goes below zero.
  uint32_t ka[LPW], va[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int ins = wave * LPW + j;
    const int r = ins * RPI + lane / CPR;
    const int key = (r & ~31) | kperm(r & 31);
    const int c = kswz<D>(r, lane % CPR);
    ka[j] = (uint32_t)((key * D + c * 8) * 2 + 8192 - 1024 * j);
    va[j] = (uint32_t)(wave * LPW * 1024 + lane * 16);
  }
  const uint32_t k_dst = lds_addr(&sK[0][wave * LPW * 512]);
  const uint32_t v_dst = lds_addr(&sV[0][wave * LPW * 512]);
  auto k_src = [&](int t) { return kbase + (size_t)t * TILE - 4096; };
  auto v_src = [&](int t) { return vbase + (size_t)t * TILE; };
  auto k_to = [&](int t) { return k_dst + (uint32_t)((t % RK) * TILE * 2); };
  auto v_to = [&](int t) { return v_dst + (uint32_t)((t % RV) * TILE * 2); };
  auto issue_k = [&](int t) { lds_dma16_runs<LPW>(k_src(t), ka, k_to(t)); };
  auto issue_v = [&](int t) { lds_dma16_runs<LPW>(v_src(t), va, v_to(t)); };

  f32x16 acc[NQB][NDB];
  float m_run[NQB], l_run[NQB];
  // Row sums of the fixed-offset pass on the matrix cores: a 16x16x32 product of
  // a 0/1 selector with the P operand.  Lane l of P holds query l % 32 and key
  // half l / 32, so B column n gathers queries n (k-groups 0, 2) and n + 16
  // (k-groups 1, 3); selector row 0 takes groups 0 and 2, row 1 groups 1 and 3.
  // Lane n < 16 then holds the sum of query n in lacc[.][0], of n + 16 in lacc[.][1].
  f32x4 lacc[NQB];
  bf16x8 sel;
  {
    const int i = lane & 15, kg = lane >> 4;
    const float v = (i == 0 && (kg & 1) == 0) || (i == 1 && (kg & 1) == 1) ? 1.f : 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) sel[e] = (__bf16)v;
  }

  using Scores = f32x16[2][NQB];   // [32-key block][query block]
  using Probs = u32x4[4][NQB];     // [16-key chunk][query block]: 8 probabilities in bf16
  // operand reads: this lane's K chunks 2kk+g in ring slot 0, and its V row; a
  // tile adds its slot, the rest are constants of the read instructions
  using lds8 = const __attribute__((address_space(3))) bf16x8 *;
  uint32_t k_at[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk)
    k_at[kk] = (uint32_t)(uintptr_t)(lvoid)&sK[0][n * D] +
               ((uint32_t)(kswz<D>(n, g) * 16) ^ (uint32_t)(32 * kk));
  const uint32_t v_lane = (uint32_t)(uintptr_t)(lvoid)&sV[0][(g * D + n) * 8];
  auto k_slot = [&](int t) { return (uint32_t)((t % RK) * TILE * 2); };
  auto ldk = [&](uint32_t slot, int i) -> bf16x8 {   // read i: 16 dims i / 2, key block i % 2
    return *(lds8)(uintptr_t)(k_at[i / 2] + slot + (uint32_t)(64 * D * (i % 2)));
  };
  auto v_base = [&](int t) {
    uint32_t b = v_lane + (uint32_t)((t % RV) * TILE * 2);
    asm volatile("" : "+v"(b));   // opaque, so that the constants below stay offsets
    return b;
  };
  auto ldv = [&](uint32_t b, int i) -> bf16x8 {      // read i: key chunk i / 4, 32 dims i % 4
    return *(lds8)(uintptr_t)(b + (uint32_t)((2 * (i / 4) * D + 32 * (i % 4)) * 16));
  };
  // matrix results in their registers before vector instructions use them: a
  // 32x32x16 product needs at most 18 wait states
  auto settle = [&](Scores &s) {
    asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s[0][0]), "+v"(s[0][1]), "+v"(s[1][0]), "+v"(s[1][1]));
  };
  auto qk = [&](int t, Scores &s) {
#pragma unroll
    for (int i = 0; i < 2 * NKK; ++i) {
      const bf16x8 kf = ldk(k_slot(t), i);
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) mfma_score(s[i % 2][qb], kf, qf[qb][i / 2], i < 2);
    }
    settle(s);
  };
  // keys at or past `rem` of this tile get no weight
  auto mask = [&](Scores &s, int rem) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (32 * kb + kperm(8 * (r >> 2) + 4 * g + (r & 3)) >= rem)
          s[kb][0][r] = s[kb][1][r] = -INFINITY;
  };
  // pair p of a tile's probabilities: key chunk p / 8, query block (p / 4) % 2,
  // elements 2 (p % 4) and the next
  auto score = [](const Scores &s, int p, int e) {
    return s[p / 16][(p / 4) % 2][8 * ((p / 8) % 2) + 2 * (p % 4) + e];
  };
  auto pack = [&](Probs &pf, int p, float x0, float x1) {
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(x0), "v"(x1));
    pf[p / 8][(p / 4) % 2][p % 4] = r;
  };
  auto probs = [](const Probs &pf, int chunk, int qb) { return __builtin_bit_cast(bf16x8, pf[chunk][qb]); };
  auto row_sums = [&](const Probs &pf, int chunk) {
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
      lacc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sel, probs(pf, chunk, qb), lacc[qb], 0, 0, 0);
  };

  // --- fixed-offset pass: each probability is 2^x for the logit x in log2 units,
  // with no row max, no subtraction and no rescale.  That is exact softmax
  // arithmetic as long as nothing overflows or underflows (checked below).
  float px0, px1;                 // the last pair, not yet packed
  bf16x8 kf[kAhead + 1];
  auto prob = [&](const Scores &s, int p, int e) {
    return __builtin_amdgcn_exp2f(score(s, p, e) * sl2);
  };
  // S(t+1), then PV(t), with the probabilities of tile t from pair kPre on and the
  // first kPre pairs of tile t+1 beside the products.  STEADY: tiles t+3 (K) and
  // t+2 (V) exist, kslot is a constant, and kf holds the first reads of K(t+1).
  auto step = [&](auto steady, int t, uint32_t kslot, Scores &cur, Scores &nxt, Probs &pf) {
    constexpr bool STEADY = decltype(steady)::value;
    const uint32_t vb = v_base(t);
    if constexpr (!STEADY) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i) kf[i] = ldk(kslot, i);
    }
    fence();
    auto slot = [&](int i, auto &&product) {
      const int p = kPre + i;
      product(0);
      fence();
      const float y0 = p < 32 ? prob(cur, p, 0) : prob(nxt, p - 32, 0);
      const float y1 = p < 32 ? prob(cur, p, 1) : prob(nxt, p - 32, 1);
      fence();
      product(1);
      fence();
      pack(pf, (p - 1) % 32, px0, px1);
      px0 = y0;
      px1 = y1;
      fence();
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i + kAhead < 16) kf[(i + kAhead) % 4] = ldk(kslot, i + kAhead);
      else kf[(i + kAhead) % 4] = ldv(vb, i + kAhead - 16);
      slot(i, [&](int qb) { mfma_score(nxt[i % 2][qb], kf[i % 4], qf[qb][i / 2], i < 2); });
    }
    wait_vmcnt<0>();              // K(t+2) and V(t+1) landed
    __syncthreads();              // ... for every wave; S(t+1) and PV(t-1) are over
    if constexpr (!STEADY) {
      settle(nxt);
      if (t + 1 == nt - 1 && rem_last < KT) mask(nxt, rem_last);
      if (t + 3 < nt) issue_k(t + 3);
      if (t + 2 < nt) issue_v(t + 2);
    }
    fence();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i + kAhead < 16) kf[(i + kAhead) % 4] = ldv(vb, i + kAhead);
      else if constexpr (STEADY) kf[(i + kAhead) % 4] = ldk(kslot ^ (uint32_t)(TILE * 2), i + kAhead - 16);
      if constexpr (STEADY) {
        if (i < 2) lds_dma16_run<4>(k_src(t + 3) + 2048 * i, ka + 4 * i, k_to(t + 3) + 4096 * i);
        else if (i < 4) lds_dma16_run<4>(v_src(t + 2) + 2048 * (i - 2), va + 4 * (i - 2), v_to(t + 2) + 4096 * (i - 2));
      }
      slot(16 + i, [&](int qb) { acc[qb][i % 4] = mfma32(kf[i % 4], probs(pf, i / 4, qb), acc[qb][i % 4]); });
      if (i % 4 == 3) {
        row_sums(pf, i / 4);
        fence();
      }
    }
  };
  // Returns false as soon as it cannot stand any more: row sums only grow, so one
  // above the bound after kCheckTile tiles (NaN included) stays above it, and the
  // rest of the pass would be for nothing.
  auto run_fixed = [&]() -> bool {
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
#pragma unroll
      for (int db = 0; db < NDB; ++db) acc[qb][db] = f32x16{};
      m_run[qb] = 0.f;
      lacc[qb] = f32x4{};
    }
    issue_k(0);
    if (nt > 1) issue_k(1);
    issue_v(0);
    if (nt > 1) wait_vmcnt<2 * LPW>();        // K(0) landed
    else wait_vmcnt<LPW>();
    __syncthreads();
    Scores sa, sb;
    Probs pf;
    qk(0, sa);
    if (nt == 1 && rem_last < KT) mask(sa, rem_last);
    wait_vmcnt<0>();              // K(1) and V(0) landed
    __syncthreads();              // ... for every wave; S(0) is over
    if (nt > 2) issue_k(2);
    if (nt > 1) issue_v(1);
    // a pair with its pack (an exp2 result needs one wait state before the pack)
    auto pair = [&](int p) {
      px0 = prob(sa, p, 0);
      px1 = prob(sa, p, 1);
      asm volatile("s_nop 1" : "+v"(px0), "+v"(px1));
    };
#pragma unroll
    for (int p = 0; p < kPre; ++p) {
      if (p) pack(pf, p - 1, px0, px1);
      pair(p);
    }
    int t = 0;
    if (t + 4 < nt) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i) kf[i] = ldk(TILE * 2, i);
      for (int stop = nt >= 4 * kCheckTile ? kCheckTile : nt;; stop = nt) {
        for (; t + 4 < nt && t < stop; t += 2) {   // two steps, so that the score sets swap roles
          step(std::true_type{}, t, TILE * 2, sa, sb, pf);
          step(std::true_type{}, t + 1, 0, sb, sa, pf);
        }
        if (stop == nt) break;
        bool over = false;
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)
          over = over || max(__float_as_uint(lacc[qb][0]), __float_as_uint(lacc[qb][1])) >
                             __builtin_bit_cast(uint32_t, 0x1p96f);
        over = __any(lane < 16 && over);
        // the waves agree through the V slot of tile t - 1: read by both, and
        // refilled only after the next step's barrier
        int *flag = reinterpret_cast<int *>(&sV[(t - 1) % RV][0]);
        __syncthreads();
        if (lane == 0) flag[wave] = over ? 1 : 0;
        __syncthreads();
        if ((flag[0] | flag[1]) != 0) return false;
      }
    }
    while (t + 1 < nt) {
      step(std::false_type{}, t, k_slot(t + 1), sa, sb, pf);
      ++t;
      if (t + 1 < nt) {
        step(std::false_type{}, t, k_slot(t + 1), sb, sa, pf);
        ++t;
      } else {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) sa[kb][qb] = sb[kb][qb];
      }
    }
    // last tile: the rest of its probabilities, PV(nt - 1)
#pragma unroll
    for (int p = kPre; p < 32; ++p) {
      pack(pf, p - 1, px0, px1);
      pair(p);
    }
    pack(pf, 31, px0, px1);
    const uint32_t vb = v_base(t);
    fence();
    asm volatile("s_nop 1");      // the last pack before the products
    fence();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const bf16x8 vf = ldv(vb, i);
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) acc[qb][i % 4] = mfma32(vf, probs(pf, i / 4, qb), acc[qb][i % 4]);
      if (i % 4 == 3) row_sums(pf, i / 4);
    }
    return true;
  };

  // --- running-max pass: the online softmax with lazy rescaling, for the units
  // whose fixed-offset pass does not stand.  The softmax of tile t goes beside
  // S(t+1), the row max of S(t+1) beside PV(t).
  auto run_max = [&] {
    const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
    float mx[NQB];
    auto tile_max = [&](const Scores &s, int qb) {
      float m = fmaxf(s[0][qb][0], s[1][qb][0]);
#pragma unroll
      for (int r = 1; r < 16; ++r) m = fmaxf(m, fmaxf(s[0][qb][r], s[1][qb][r]));
      return max_xor32(m) * sl2;
    };
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
#pragma unroll
      for (int db = 0; db < NDB; ++db) acc[qb][db] = f32x16{};
      m_run[qb] = kMInit;
      l_run[qb] = 0.f;
    }
    auto rescale = [&] {
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb)
        if (__any(mx[qb] > m_run[qb] + kRescale)) {
          const float m_new = fmaxf(m_run[qb], mx[qb]);
          const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
          m_run[qb] = m_new;
          l_run[qb] *= alpha;
#pragma unroll
          for (int db = 0; db < NDB; ++db) acc[qb][db] *= alpha;
        }
    };
    // probabilities of pair p, and the row sum of the rounded values
    auto pair = [&](const Scores &s, Probs &pf, int p) {
      const int qb = (p / 4) % 2;
      const bf16x2 r = {(__bf16)__builtin_amdgcn_exp2f(fmaf(score(s, p, 0), sl2, -m_run[qb])),
                        (__bf16)__builtin_amdgcn_exp2f(fmaf(score(s, p, 1), sl2, -m_run[qb]))};
      l_run[qb] = __builtin_amdgcn_fdot2_f32_bf16(r, one, l_run[qb], false);
      pf[p / 8][qb][p % 4] = __builtin_bit_cast(uint32_t, r);
    };
    // PV(t), with its first kAhead operand reads in kf; leaves there the first reads
    // of the K tile in ring slot `kslot`
    auto pv = [&](uint32_t vb, uint32_t kslot, Probs &pf, auto &&beside) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        kf[(i + kAhead) % 4] = i + kAhead < 16 ? ldv(vb, i + kAhead) : ldk(kslot, i + kAhead - 16);
        acc[0][i % 4] = mfma32(kf[i % 4], probs(pf, i / 4, 0), acc[0][i % 4]);
        fence();
        beside(i);
        fence();
        acc[1][i % 4] = mfma32(kf[i % 4], probs(pf, i / 4, 1), acc[1][i % 4]);
        fence();
      }
    };
    issue_k(0);
    if (nt > 1) issue_k(1);
    issue_v(0);
    if (nt > 1) wait_vmcnt<2 * LPW>();
    else wait_vmcnt<LPW>();
    __syncthreads();
    Scores sa, sb;
    Probs pf;
    qk(0, sa);
    if (nt == 1 && rem_last < KT) mask(sa, rem_last);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) mx[qb] = tile_max(sa, qb);
    wait_vmcnt<0>();
    __syncthreads();
    if (nt > 2) issue_k(2);
    if (nt > 1) issue_v(1);
#pragma unroll
    for (int i = 0; i < kAhead; ++i) kf[i] = ldk(k_slot(1), i);
    auto step_max = [&](int t, Scores &cur, Scores &nxt) {
      const uint32_t kslot = k_slot(t + 1), vb = v_base(t);
      rescale();
      fence();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (i + kAhead < 16) kf[(i + kAhead) % 4] = ldk(kslot, i + kAhead);
        else kf[(i + kAhead) % 4] = ldv(vb, i + kAhead - 16);
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          mfma_score(nxt[i % 2][qb], kf[i % 4], qf[qb][i / 2], i < 2);
          fence();
          // three pairs in two slots here, the last eight beside PV(t)
          if (qb == 0)
#pragma unroll
            for (int p = 3 * i / 2; p < 3 * (i + 1) / 2; ++p) pair(cur, pf, p);
          fence();
        }
      }
      wait_vmcnt<0>();
      __syncthreads();
      settle(nxt);
      if (t + 1 == nt - 1 && rem_last < KT) mask(nxt, rem_last);
      if (t + 3 < nt) issue_k(t + 3);
      if (t + 2 < nt) issue_v(t + 2);
      float m[NQB] = {-INFINITY, -INFINITY};
      auto take = [&](int r) {
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)      // (fmaxf would first quiet each score)
          asm("v_max3_f32 %0, %1, %2, %0" : "+v"(m[qb]) : "v"(nxt[0][qb][r]), "v"(nxt[1][qb][r]));
      };
      pv(vb, k_slot(t + 2), pf, [&](int i) {
        if (i < 8) {
          pair(cur, pf, 24 + i);
        } else {
          take(2 * (i - 8));
          take(2 * (i - 8) + 1);
        }
      });
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) mx[qb] = max_xor32(m[qb]) * sl2;
    };
    int t = 0;
    while (t + 1 < nt) {
      step_max(t, sa, sb);
      ++t;
      if (t + 1 < nt) {
        step_max(t, sb, sa);
        ++t;
      } else {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) sa[kb][qb] = sb[kb][qb];
      }
    }
    rescale();
#pragma unroll
    for (int p = 0; p < 32; ++p) pair(sa, pf, p);
    const uint32_t vb = v_base(t);
#pragma unroll
    for (int i = 0; i < kAhead; ++i) kf[i] = ldv(vb, i);
    pv(vb, 0, pf, [](int) {});
  };

  // Fixed-offset pass first.  Its result stands when every row sum of the work
  // group lies in [2^-60, 2^96] and every accumulator is finite and below 2^121:
  // then no probability overflowed (each is at most 2^96), and the N keys that
  // underflowed to 0 (logit < -126 in log2 units) weigh at most N 2^-126 against
  // a sum of at least 2^-60: less than 2^-36 of it for any N below 2^30 (the
  // most the configuration allows).  The accumulator bound leaves room for the
  // merge kernel's fp32 sum of up to 32 such partials (2^121 * 32 = 2^126).
  // Otherwise the group runs the running-max pass over the same keys (at once
  // when the row sums of the first tiles already say so: a 720P layer with queries
  // 40 times as large, where every group does: 2.28 -> 1.51 ms).  The
  // flags go through K ring slot 0, which no DMA targets once the pass is over.
  bool any_fallback = !run_fixed();
  if (any_fallback) {
    wait_vmcnt<0>();              // nothing of the abandoned pass is in flight
    __syncthreads();
  } else {
    bool bad = false;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const int q = lane & 31;
      const float s0 = __shfl(lacc[qb][0], q & 15), s1 = __shfl(lacc[qb][1], q & 15);
      l_run[qb] = q < 16 ? s0 : s1;    // the full row sum, in both lanes of the query
      uint32_t amax = 0;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) amax = max(amax, abs_bits(acc[qb][db][r]));
      bad = bad || !fixed_offset_ok(l_run[qb], amax);
    }
    bad = __any(bad);
    int *flag = reinterpret_cast<int *>(&sK[0][0]);
    __syncthreads();
    if (lane == 0) flag[wave] = bad ? 1 : 0;
    __syncthreads();
    any_fallback = (flag[0] | flag[1]) != 0;
    __syncthreads();              // every wave has read the flags
  }
  if (any_fallback) run_max();

#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int lrow = wave * 64 + qb * 32 + n;
    // l_run: the row sum of this lane's query (the fixed-offset pass), or this
    // lane's half of it (the running-max pass)
    const float l_tot = any_fallback ? sum_xor32(l_run[qb]) : l_run[qb];
    if (u.slot < 0) {
      if (rvalid[qb]) {
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        float *obase = u.out_sel == 0 ? a.o[0] : (u.out_sel == 1 ? a.o[1] : a.o[2]);
        float *op = obase + ((size_t)u.head * L + row[qb]) * D;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int rq = 0; rq < 4; ++rq) {
            f32x4 v4 = {acc[qb][db][4 * rq + 0] * inv, acc[qb][db][4 * rq + 1] * inv,
                        acc[qb][db][4 * rq + 2] * inv, acc[qb][db][4 * rq + 3] * inv};
            *reinterpret_cast<f32x4 *>(op + 32 * db + 8 * rq + 4 * g) = v4;
          }
      }
    } else {
      float *pp = a.part + (size_t)u.slot * partial_floats(D);
      float *op = pp + (size_t)lrow * D;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          f32x4 v4 = {acc[qb][db][4 * rq + 0], acc[qb][db][4 * rq + 1], acc[qb][db][4 * rq + 2],
                      acc[qb][db][4 * rq + 3]};
          *reinterpret_cast<f32x4 *>(op + 32 * db + 8 * rq + 4 * g) = v4;
        }
      if (g == 0) {
        pp[(size_t)kQTile * D + lrow] = m_run[qb];
        pp[(size_t)kQTile * D + kQTile + lrow] = l_tot;
      }
    }
  }
}

}  // namespace

hipError_t launch_dense128(const DenseArgs &a, DenseRole role, hipStream_t s) {
  dim3 grid(a.n_units), block(128);
#define HC_DENSE(RR) hipLaunchKernelGGL((attn_dense128_kernel<RR>), grid, block, 0, s, a)
  if (role == DenseRole::kRouted) HC_DENSE(0);
  else if (role == DenseRole::kFullWindow) HC_DENSE(1);
  else if (role == DenseRole::kClassify) HC_DENSE(2);
  else if (role == DenseRole::kVariant) HC_DENSE(3);
  else HC_DENSE(4);
#undef HC_DENSE
  return hipGetLastError();
}

}  // namespace hc

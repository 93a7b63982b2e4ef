// Cache split and block append into the per-archetype buffers (Sec. 4.3), and
// the per-token statistics of the classification rule (Eq. 3 and Eq. 4).
#include "hc_device.h"

namespace hc {
namespace {
using namespace dev;

// ---------------------------------------------------------------------------
// Scatter: one work group = 64 rows of one (head, source block), 64 tokens or,
// for the frames of a Spatial buffer, 64 storage keys.
// K rows are copied as 16-byte chunks; V goes through LDS and is written in the
// 8-key-grouped layout, 16 bytes per (8 keys, dim) when the 8 rows are one
// aligned group, else element by element.  A Spatial frame is walked by its
// storage (rows of `pitch` keys) and not by its tokens, because then every
// group of eight is aligned also where grid_w is not a multiple of 8: the
// padding columns of a row are read as zeros and written as such.  By tokens,
// three of four groups of a 52-wide grid went out as single elements: all-head
// split of a 480P window 95 -> 78 us, append of a routed
// 480P layer with three Spatial heads 16.4 -> 15.0 us.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void kv_scatter_kernel(ScatterArgs a) {
  constexpr int TT = 64;
  constexpr int VS = D + 8;
  __shared__ __attribute__((aligned(16))) uint16_t sV[TT * VS];
  // source token (-1: none) and destination key (-1: past the end) of every row,
  // computed once (the Spatial layouts need integer divisions)
  __shared__ int64_t skey[TT];
  __shared__ int stok[TT];
  int bid = blockIdx.x;
  const int tt = bid % a.n_tiles;
  bid /= a.n_tiles;
  const int i = bid % a.n_src;
  const int h = bid / a.n_src;

  const uint8_t kind = a.head_kind[h];
  uint16_t *kd, *vd;
  int64_t kph;      // keys per head of the destination buffer
  int mode;         // 0 dense rows, 1 Spatial frames, 2 cells
  int64_t kbase = 0;
  if (kind == 0 /*sink*/ || kind == 1 /*dummy*/) {
    const int sd = kind == 0 ? a.sink_slot[i] : a.dummy_slot[i];
    if (sd < 0) return;
    kd = a.k_sd; vd = a.v_sd; kph = a.sd_keys; mode = 0;
    kbase = (int64_t)sd * a.L;
  } else if (kind == 3 /*global*/) {
    kd = a.k_g; vd = a.v_g; kph = a.g_keys; mode = 0;
    kbase = (int64_t)a.src_slot[i] * a.L;
  } else {
    kd = a.k_sp; vd = a.v_sp; kph = a.sp_keys; mode = a.cell > 0 ? 2 : 1;
  }
  const int slot = a.src_slot[i];
  const int t0 = tt * TT;
  const int frame_keys = a.geo.rows * a.geo.pitch;
  const int n_rows = mode == 1 ? a.F * frame_keys : a.L;
  if (t0 >= n_rows) return;
  const int64_t hoff = (int64_t)a.head_slot[h] * kph * D;
  kd += hoff;
  vd += hoff;
  if (threadIdx.x < TT) {
    const int row = t0 + threadIdx.x;
    const int P = a.Hg * a.Wg;
    int tok = row < n_rows ? row : -1;
    int64_t key = -1;
    if (tok >= 0) {
      if (mode == 0) {
        key = kbase + tok;
      } else if (mode == 1) {
        const int fr = row / frame_keys, p = row % frame_keys;
        const int yy = p / a.geo.pitch, xx = p % a.geo.pitch;
        key = (int64_t)slot * a.F * frame_keys + row;
        tok = xx < a.Wg ? fr * P + yy * a.Wg + xx : -1;
      } else {
        const int fr = tok / P, p = tok % P;
        const int yy = p / a.Wg, xx = p % a.Wg;
        const int cy = min(yy / a.cell, a.ncy - 1), cx = min(xx / a.cell, a.ncx - 1);
        const int ch = cy == a.ncy - 1 ? a.Hg - cy * a.cell : a.cell;
        const int cw = cx == a.ncx - 1 ? a.Wg - cx * a.cell : a.cell;
        key = a.cell_off[cy * a.ncx + cx] + ((int64_t)slot * a.F + fr) * ch * cw +
              (yy - cy * a.cell) * cw + (xx - cx * a.cell);
      }
    }
    stok[threadIdx.x] = tok;
    skey[threadIdx.x] = key;
  }

  const uint16_t *sk = a.src_k + ((size_t)(h * a.n_src + i) * a.L) * D;
  const uint16_t *sv = a.src_v + ((size_t)(h * a.n_src + i) * a.L) * D;
  __syncthreads();
  constexpr int CPR = D / 8;
  for (int c = threadIdx.x; c < TT * CPR; c += 256) {
    const int lt = c / CPR, col = c % CPR;
    const int tok = stok[lt];
    u32x4 vv = {0, 0, 0, 0};
    if (tok >= 0) {
      const u32x4 kv = *reinterpret_cast<const u32x4 *>(sk + (size_t)tok * D + col * 8);
      *reinterpret_cast<u32x4 *>(kd + skey[lt] * D + col * 8) = kv;
      vv = *reinterpret_cast<const u32x4 *>(sv + (size_t)tok * D + col * 8);
    }
    *reinterpret_cast<u32x4 *>(&sV[lt * VS + col * 8]) = vv;
  }
  __syncthreads();
  for (int w = threadIdx.x; w < D * (TT / 8); w += 256) {
    const int d = w % D, j = w / D;
    const int64_t kA = skey[8 * j];
    if (kA < 0) continue;
    const bool full = (kA & 7) == 0 && skey[8 * j + 7] == kA + 7;
    if (full) {
      uint16_t vals[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) vals[e] = sV[(8 * j + e) * VS + d];
      u32x4 pk;
#pragma unroll
      for (int e = 0; e < 4; ++e) pk[e] = (uint32_t)vals[2 * e] | ((uint32_t)vals[2 * e + 1] << 16);
      *reinterpret_cast<u32x4 *>(vd + ((kA >> 3) * D + d) * 8) = pk;
    } else {
      for (int e = 0; e < 8 && skey[8 * j + e] >= 0; ++e) {
        const int64_t ke = skey[8 * j + e];
        vd[((ke >> 3) * D + d) * 8 + (ke & 7)] = sV[(8 * j + e) * VS + d];
      }
    }
  }
}


// ---------------------------------------------------------------------------
// Classification statistics (Eq. 3, Eq. 4), fp64 accumulation.  One work group
// takes kClsStatRows token rows of one head; D/4 lanes share a row (four dims
// each).  The eight sums of a row are reduced by halving: in three steps a lane
// trades half of its sums for the other half of its partner's, so a row costs
// 7 + log2(D/32) lane exchanges instead of 8 log2(D/4); the cosines (fp64
// square roots and divisions) are then formed once per row, one row per lane,
// instead of once per wave.  Only the Spatial cosine is stored per token (the
// percentile needs it); the sums over the group's rows go out once.  Measured
// with 12 heads, d = 128: 720P (L = 10800) 160 -> 66 us, 4.0 TB/s of the four
// outputs read; 480P 62 -> 31 us, against one wave per row with 48 exchanges and
// the divisions in every lane.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void cls_stats_kernel(StatsArgs a) {
  constexpr int LPR = D / 4;                    // lanes per row
  constexpr int RPS = 256 / LPR;                // rows per step of the work group
  static_assert(LPR >= 8 && kClsStatRows == 64 && kClsStatRows % RPS == 0, "row split");
  __shared__ double row_s[kClsStatRows][9];     // 9: rows start in different banks
  const int tid = threadIdx.x, lane = tid & 63, j = tid % LPR;
  const int nb = (a.L + kClsStatRows - 1) / kClsStatRows;
  const int h = blockIdx.x / nb, b = blockIdx.x % nb;
#pragma unroll 2
  for (int i = 0; i < kClsStatRows / RPS; ++i) {
    const int lr = i * RPS + tid / LPR;
    const size_t at = ((size_t)h * a.L + min(b * kClsStatRows + lr, a.L - 1)) * D + 4 * j;
    const f32x4 r4 = *reinterpret_cast<const f32x4 *>(a.o_ref + at);
    const f32x4 s4 = *reinterpret_cast<const f32x4 *>(a.o_sink + at);
    const f32x4 u4 = *reinterpret_cast<const f32x4 *>(a.o_dummy + at);
    const f32x4 p4 = *reinterpret_cast<const f32x4 *>(a.o_sp + at);
    // ref.ref, sink.sink, dummy.dummy, sp.sp, sink.ref, dummy.ref, sp.ref, |sp - ref|^2
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double r = r4[e], s = s4[e], u = u4[e], p = p4[e];
      v[0] += r * r; v[1] += s * s; v[2] += u * u; v[3] += p * p;
      v[4] += s * r; v[5] += u * r; v[6] += p * r; v[7] += (p - r) * (p - r);
    }
#pragma unroll
    for (int step = 0; step < 3; ++step) {
      const int m = 4 >> step, bit = 1 << step;
      const bool up = (lane & bit) != 0;
#pragma unroll
      for (int k = 0; k < m; ++k) {
        const double send = up ? v[k] : v[k + m];
        v[k] = (up ? v[k + m] : v[k]) + __shfl_xor(send, bit, 64);
      }
    }
    double t = v[0];
#pragma unroll
    for (int bit = 8; bit < LPR; bit <<= 1) t += __shfl_xor(t, bit, 64);
    // lane j < 8 holds sum number 4 (j & 1) + (j & 2) + (j >> 2)
    if (j < 8) row_s[lr][4 * (j & 1) + (j & 2) + (j >> 2)] = t;
  }
  __syncthreads();
  if (tid >= 64) return;
  const int tok = b * kClsStatRows + tid;
  const double *v = row_s[tid];
  double out[4] = {0, 0, 0, 0};
  if (tok < a.L) {
    const double nr = sqrt(v[0]);
    out[0] = v[4] / fmax(sqrt(v[1]) * nr, 1e-30);
    out[1] = v[5] / fmax(sqrt(v[2]) * nr, 1e-30);
    out[2] = v[6] / fmax(sqrt(v[3]) * nr, 1e-30);
    out[3] = v[7];
    a.cos_sp[(size_t)h * a.L + tok] = out[2];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) out[k] += __shfl_xor(out[k], off, 64);
    if (lane == 0) a.sums[((size_t)h * nb + b) * 4 + k] = out[k];
  }
}


// ---------------------------------------------------------------------------
// Per-head reduction of the statistics, one work group per head: the sums of
// the row groups in float64, and the 5th percentile of the Spatial cosines by
// radix selection of its lower order statistic.  The cosines become 64-bit keys
// in the same order; a first pass finds the bits that all keys share, and each
// further pass counts the next 11 bits of the keys that match the prefix so far
// and narrows the prefix to the bin of the k-th smallest, until one key is left
// in it (or no bits are).  The upper order statistic is the same key again, or
// the smallest one above it.  Bound by the latency of the passes (a few loads
// per thread each, all from L2): the shared bits are skipped because every key
// would fall into one bin there and its LDS atomics would queue up, and usually
// two counting passes settle the rest.  Measured with 12 heads: L = 10800 in 340
// -> 38 us, L = 4680 in 235 -> 26 us, against 16 passes of 8-bit digits by 256
// threads over cosines 32 bytes apart.  1024 threads leave 128 registers each, so 44
// values (the sums above all, which only the last lines use) are kept in scratch
// memory meanwhile.
// ---------------------------------------------------------------------------
constexpr int kRedThreads = 1024;
constexpr int kDigit = 11, kBins = 1 << kDigit;

__device__ __forceinline__ uint64_t order_key(double x) {
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double key_double(uint64_t k) {
  return __longlong_as_double((long long)((k >> 63) ? (k & 0x7FFFFFFFFFFFFFFFull) : ~k));
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  return (uint64_t)__shfl_xor((unsigned long long)v, m, 64);
}

__global__ __launch_bounds__(kRedThreads) void cls_reduce_kernel(ClsReduceArgs a) {
  constexpr int NW = kRedThreads / 64;
  constexpr int BPT = kBins / kRedThreads;       // bins per thread of the scan
  __shared__ double sum_s[4][NW];
  __shared__ uint64_t lo_s[NW], hi_s[NW], above_s[NW], found_s;
  __shared__ int wave_s[NW], cnt_s[NW];
  __shared__ unsigned hist[kBins];
  __shared__ int bin_s, below_s, in_bin_s;
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int L = a.L;
  const double *cosv = a.cos_sp + (size_t)h * L;

  // the row groups' sums; the smallest and the largest key
  double sum[4] = {0, 0, 0, 0};
  for (int b = tid; b < a.n_groups; b += kRedThreads)
#pragma unroll
    for (int k = 0; k < 4; ++k) sum[k] += a.sums[((size_t)h * a.n_groups + b) * 4 + k];
  uint64_t lo = ~0ull, hi = 0;
  for (int t = tid; t < L; t += kRedThreads) {
    const uint64_t key = order_key(cosv[t]);
    lo = min(lo, key);
    hi = max(hi, key);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sum[k] += __shfl_xor(sum[k], off, 64);
    lo = min(lo, shfl_xor_u64(lo, off));
    hi = max(hi, shfl_xor_u64(hi, off));
  }
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sum_s[k][w] = sum[k];
    lo_s[w] = lo;
    hi_s[w] = hi;
  }
  __syncthreads();
  double tot[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < NW; ++i) {
#pragma unroll
    for (int k = 0; k < 4; ++k) tot[k] += sum_s[k][i];
    lo = min(lo, lo_s[i]);
    hi = max(hi, hi_s[i]);
  }

  // the k-th smallest key (0-based): bits at and above `shift` of it are `prefix`
  const double rank = 0.05 * (L - 1);
  int k = (int)floor(rank);
  const int klo = k;
  int shift = lo == hi ? 0 : 64 - __clzll((long long)(lo ^ hi));
  uint64_t prefix = shift == 64 ? 0 : lo >> shift << shift;
  int in_bin = L;
  while (shift > 0 && in_bin > 1) {
    const int width = min(shift, kDigit);
    const uint64_t mask = shift == 64 ? 0 : ~0ull << shift;
    shift -= width;
    for (int i = tid; i < kBins; i += kRedThreads) hist[i] = 0;
    __syncthreads();
    for (int t = tid; t < L; t += kRedThreads) {
      const uint64_t key = order_key(cosv[t]);
      if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & (uint64_t)((1 << width) - 1)], 1u);
    }
    __syncthreads();
    // scan of the bins: thread tid holds bins BPT tid .. BPT tid + BPT - 1
    int own[BPT], s = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) { own[i] = (int)hist[BPT * tid + i]; s += own[i]; }
    int incl = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int up = __shfl_up(incl, off, 64);
      if (lane >= off) incl += up;
    }
    if (lane == 63) wave_s[w] = incl;
    __syncthreads();
    int before = incl - s;
    for (int i = 0; i < w; ++i) before += wave_s[i];
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      if (k >= before && k < before + own[i]) {   // exactly one thread and bin
        bin_s = BPT * tid + i;
        below_s = before;
        in_bin_s = own[i];
      }
      before += own[i];
    }
    __syncthreads();
    prefix |= (uint64_t)bin_s << shift;
    k -= below_s;
    in_bin = in_bin_s;
    __syncthreads();
  }
  // the whole key: one match is left unless all bits are known
  uint64_t v = prefix;
  if (shift > 0) {
    for (int t = tid; t < L; t += kRedThreads) {
      const uint64_t key = order_key(cosv[t]);
      if (key >> shift == prefix >> shift) found_s = key;
    }
    __syncthreads();
    v = found_s;
  }
  // the next order statistic: v again when more than klo + 1 keys are at most v,
  // else the smallest key above v
  int le = 0;
  uint64_t above = ~0ull;
  for (int t = tid; t < L; t += kRedThreads) {
    const uint64_t key = order_key(cosv[t]);
    if (key <= v) ++le;
    else above = min(above, key);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    le += __shfl_xor(le, off, 64);
    above = min(above, shfl_xor_u64(above, off));
  }
  if (lane == 0) { cnt_s[w] = le; above_s[w] = above; }
  __syncthreads();
  if (tid != 0) return;
  le = 0;
  above = ~0ull;
  for (int i = 0; i < NW; ++i) { le += cnt_s[i]; above = min(above, above_s[i]); }
  const double v_lo = key_double(v);
  const double v_hi = (klo + 1 >= L || le > klo + 1) ? v_lo : key_double(above);
  const double p5 = v_lo + (rank - klo) * (v_hi - v_lo);
  const double mse = tot[3] / ((double)L * a.D);
  double *o = a.out + (size_t)h * 6;
  o[0] = tot[0] / L;
  o[1] = tot[1] / L;
  o[2] = tot[2] / L;
  o[3] = p5;
  o[4] = mse;
  o[5] = p5 - a.gamma * mse;
}


}  // namespace

hipError_t launch_cls_reduce(const ClsReduceArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(cls_reduce_kernel, dim3(a.n_heads), dim3(kRedThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_scatter(ScatterArgs a, int n_heads, hipStream_t s) {
  // tiles of 64 rows per (head, block): a Spatial frame's storage has at least
  // as many rows as tokens
  bool frames = false;
  for (int h = 0; h < n_heads; ++h) frames |= a.head_kind[h] == HC_SPATIAL;
  const int rows = frames && a.cell == 0 ? a.F * a.geo.rows * a.geo.pitch : a.L;
  a.n_tiles = (rows + 63) / 64;
  dim3 grid((unsigned)(n_heads * a.n_src * a.n_tiles)), block(256);
  if (a.D == 128)
    hipLaunchKernelGGL((kv_scatter_kernel<128>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((kv_scatter_kernel<64>), grid, block, 0, s, a);
  return hipGetLastError();
}


hipError_t launch_stats(const StatsArgs &a, hipStream_t s) {
  const dim3 grid((unsigned)(a.n_heads * cls_stat_groups(a.L)));
  if (a.D == 128) hipLaunchKernelGGL((cls_stats_kernel<128>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((cls_stats_kernel<64>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}


}  // namespace hc

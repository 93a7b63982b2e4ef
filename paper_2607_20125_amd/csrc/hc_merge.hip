// The merge of partial results: per-range partials of the dense units
// (Global heads, two-block Sink/Dummy heads, tail pieces) and key-frame splits
// of the Spatial heads, in one launch.
#include "hc_device.h"

#include <algorithm>

namespace hc {
namespace {
using namespace dev;

// ---------------------------------------------------------------------------
// Combine: O = sum_i 2^(m_i - M) acc_i / sum_i 2^(m_i - M) l_i over the partial
// slots of one (head, query tile).  One work group takes kCombRows rows of an
// item, so even a few Global heads spread over the whole GPU.
// ---------------------------------------------------------------------------
constexpr int kCombRows = 32;

__device__ __forceinline__ void combine_rows(const CombineArgs &a, int block) {
  constexpr int kGroups = 256 / kCombRows;               // slot groups of the weight phase
  constexpr int kPerGroup = kMaxSrcBlocks / kGroups;
  __shared__ float w_s[kMaxSrcBlocks][kCombRows];
  __shared__ float red_s[kGroups][kCombRows];
  __shared__ float inv_s[kCombRows];
  constexpr int kParts = kQTile / kCombRows;
  const CombineItem it = a.items[block / kParts];
  const int r0 = (block % kParts) * kCombRows;     // first row of this group in the tile
  const int D = a.D, ns = it.n_slots;
  const int64_t pf = (int64_t)kQTile * (D + 2);
  const float *part = a.part + (int64_t)it.slot0 * pf;

  // weights: thread (sg, lr) loads the max and sum of row r0 + lr in slots
  // sg, sg + 8, ...; all loads of the group are in flight together
  const int lr = threadIdx.x % kCombRows, sg = threadIdx.x / kCombRows;
  float mv[kPerGroup], lv[kPerGroup];
#pragma unroll
  for (int j = 0; j < kPerGroup; ++j) {
    const int i = sg + kGroups * j;
    const float *ml = part + i * pf + (int64_t)kQTile * D + r0 + lr;
    mv[j] = i < ns ? ml[0] : kMInit;
    lv[j] = i < ns ? ml[kQTile] : 0.f;
  }
  float m = mv[0];
#pragma unroll
  for (int j = 1; j < kPerGroup; ++j) m = fmaxf(m, mv[j]);
  red_s[sg][lr] = m;
  __syncthreads();
  float M = red_s[0][lr];
#pragma unroll
  for (int k = 1; k < kGroups; ++k) M = fmaxf(M, red_s[k][lr]);
  __syncthreads();                                       // every thread has read red_s
  float den = 0.f;
#pragma unroll
  for (int j = 0; j < kPerGroup; ++j) {
    const int i = sg + kGroups * j;
    if (i < ns) {
      const float wgt = __builtin_amdgcn_exp2f(mv[j] - M);
      w_s[i][lr] = wgt;
      den += wgt * lv[j];
    }
  }
  red_s[sg][lr] = den;
  __syncthreads();
  if (sg == 0) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < kGroups; ++k) t += red_s[k][lr];
    inv_s[lr] = t > 0.f ? 1.f / t : 0.f;
  }
  __syncthreads();

  // outputs: 16-byte columns of the group's rows, slots read eight at a time
  float *obase = it.out_sel == 0 ? a.o[0] : (it.out_sel == 1 ? a.o[1] : a.o[2]);
  const int nq = D / 4;
  for (int e = threadIdx.x; e < kCombRows * nq; e += 256) {
    const int er = e / nq, c4 = e % nq, row = r0 + er;
    if (it.q0 + row >= a.L) continue;
    const float *src = part + (int64_t)row * D + 4 * c4;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0; i0 < ns; i0 += 8) {
      f32x4 v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (i0 + j < ns) v[j] = *reinterpret_cast<const f32x4 *>(src + (i0 + j) * pf);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (i0 + j < ns) sum += v[j] * w_s[i0 + j][er];
    }
    *reinterpret_cast<f32x4 *>(obase + ((size_t)it.head * a.L + it.q0 + row) * D + 4 * c4) =
        sum * inv_s[er];
  }
}

// ---------------------------------------------------------------------------
// The per-split partial results of the Spatial heads: for each (head, query)
// O = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s, M = max_s m_s.  One thread
// per 4 output dims; with the number of splits known to the compiler the loads of
// all of them are in flight together.
// ---------------------------------------------------------------------------
template <int N>
__device__ __forceinline__ void merge_splits(const SpatialArgs &a, int D, int block, int blocks) {
  const uint32_t nq = (uint32_t)D / 4;
  const int64_t plane = (int64_t)a.n_sp * a.L;        // rows per split
  const int64_t total = plane * nq;
  for (int64_t e = (int64_t)block * 256 + threadIdx.x; e < total; e += (int64_t)blocks * 256) {
    const uint32_t row = (uint32_t)(e / nq), c4 = (uint32_t)(e % nq);   // hs * L + token
    f32x2 ml[N];
    f32x4 v[N];
#pragma unroll
    for (int s = 0; s < N; ++s) ml[s] = reinterpret_cast<const f32x2 *>(a.part_ml)[s * plane + row];
#pragma unroll
    for (int s = 0; s < N; ++s)
      v[s] = *reinterpret_cast<const f32x4 *>(a.part + (s * plane + row) * D + 4 * c4);
    float M = ml[0][0];
#pragma unroll
    for (int s = 1; s < N; ++s) M = fmaxf(M, ml[s][0]);
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
#pragma unroll
    for (int s = 0; s < N; ++s) {
      const float w = __builtin_amdgcn_exp2f(ml[s][0] - M);
      den += w * ml[s][1];
      sum += w * v[s];
    }
    const uint32_t hs = row / (uint32_t)a.L, tok = row % (uint32_t)a.L;
    const float inv = den > 0.f ? 1.f / den : 0.f;
    *reinterpret_cast<f32x4 *>(a.o + ((size_t)a.heads[hs] * a.L + tok) * D + 4 * c4) = sum * inv;
  }
}

// Dense items alone, in a kernel of its own: a grid that also holds the code and the
// arguments of the Spatial rows takes 0.3-0.7 us longer for them (96 items of five
// 128-dim slots 6.1 against 6.5 us), which a two-block layer of 20 us notices.
__global__ __launch_bounds__(256) void combine_kernel(CombineArgs c) { combine_rows(c, blockIdx.x); }

// Both kinds of partials in one grid: the first `combine_blocks` work groups take
// the dense items, the others the Spatial rows.
__global__ __launch_bounds__(256) void merge_kernel(CombineArgs c, SpatialArgs s, int D,
                                                    int combine_blocks) {
  if ((int)blockIdx.x < combine_blocks) combine_rows(c, blockIdx.x);
  else {
    const int b = blockIdx.x - combine_blocks, n = gridDim.x - combine_blocks;
    switch (s.n_split) {
      case 2: merge_splits<2>(s, D, b, n); break;
      case 3: merge_splits<3>(s, D, b, n); break;
      case 4: merge_splits<4>(s, D, b, n); break;
      case 5: merge_splits<5>(s, D, b, n); break;
      case 6: merge_splits<6>(s, D, b, n); break;
      case 7: merge_splits<7>(s, D, b, n); break;
      default: merge_splits<8>(s, D, b, n); break;
    }
  }
}

}  // namespace

hipError_t launch_merge(const CombineArgs &c, const SpatialArgs &s, int head_dim, hipStream_t st) {
  const int combine_blocks = std::max(c.n_items, 0) * (kQTile / kCombRows);
  int64_t split_blocks = 0;
  if (s.n_split > 1) {
    if (s.n_split > 8 || !s.part || !s.part_ml) return hipErrorInvalidValue;
    split_blocks = std::min<int64_t>(((int64_t)s.n_sp * s.L * (head_dim / 4) + 255) / 256, 8192);
  }
  if (combine_blocks + split_blocks == 0) return hipSuccess;
  if (split_blocks == 0) {
    hipLaunchKernelGGL(combine_kernel, dim3((unsigned)combine_blocks), dim3(256), 0, st, c);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(merge_kernel, dim3((unsigned)(combine_blocks + split_blocks)), dim3(256), 0, st,
                     c, s, head_dim, combine_blocks);
  return hipGetLastError();
}

}  // namespace hc

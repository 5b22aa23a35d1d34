// Log-sum-exp merge of partial attentions over disjoint key parts:
// LSE = log sum_s exp(lse_s), O = sum_s exp(lse_s - LSE) O_s.  The parts together
// are the single softmax over Concat(C, X) of Section 3.1.
//
// One thread per (row, 16 bytes of partial row): 8 dims of a scaled-fp16 partial
// (bfloat16 inputs; value * 2^exp[row] restores the row) or 4 dims of a float32
// one.  A thread takes all parts, CH at a time (CH = the part count, or 8), every load
// of those issued before the first use.  More than 8 parts of few rows (decoding), at
// least half as many as a workgroup has groups: a workgroup per row, its threads split into groups that take every GR-th part and are
// joined in LDS -- the parts are then the only parallelism (25 parts of 32 rows: 6.8 us
// one thread per piece, 4.3 split; 16 parts of 2,048 rows: 3.7 and 6.5).
#include "launch.h"

namespace infllm {
namespace {

// One piece of one part's row: its values in float, and its lse.
template <bool HALF>
__device__ __forceinline__ void load_piece(const MergeArgs& a, int64_t pr, int c, float (&o)[HALF ? 8 : 4], float& l) {
  l = a.part_lse[pr];
  if constexpr (HALF) {
    const uint4 w = *(const uint4*)((const uint16_t*)a.part_o + pr * a.head_dim + 8 * c);
    const float sc = exp2_int(a.part_exp[pr]);
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      o[2 * q] = f16_lo(ww[q]) * sc;
      o[2 * q + 1] = f16_hi(ww[q]) * sc;
    }
  } else {
    const float4 w = *(const float4*)((const float*)a.part_o + pr * a.head_dim + 4 * c);
    o[0] = w.x;
    o[1] = w.y;
    o[2] = w.z;
    o[3] = w.w;
  }
}
// Joins parts first, first + step, ... (every load of CH of them issued before the
// first use) into a running maximum, weight sum and weighted row.  ONCE: there are at
// most CH of them.
template <bool HALF, int CH, bool ONCE>
__device__ __forceinline__ void join_parts(const MergeArgs& a, int row, int c, int first, int step, float& M, float& tot,
                                           float (&acc)[HALF ? 8 : 4]) {
  constexpr int DPT = HALF ? 8 : 4;
  M = -__builtin_inff();
  tot = 0.f;
#pragma unroll
  for (int e = 0; e < DPT; ++e) acc[e] = 0.f;
  for (int p0 = first; p0 < a.parts; p0 += CH * step) {
    float l[CH], o[CH][DPT];
#pragma unroll
    for (int j = 0; j < CH; ++j)
      load_piece<HALF>(a, (int64_t)min(p0 + j * step, a.parts - 1) * a.rows + row, c, o[j], l[j]);
    float m_new = M;
#pragma unroll
    for (int j = 0; j < CH; ++j)
      if (p0 + j * step < a.parts) m_new = fmaxf(m_new, l[j]);
    if (m_new == -__builtin_inff()) continue;  // nothing visible yet
    if constexpr (!ONCE) {
      const float r = M == -__builtin_inff() ? 0.f : expf(M - m_new);
      tot *= r;
#pragma unroll
      for (int e = 0; e < DPT; ++e) acc[e] *= r;
    }
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const float w = (p0 + j * step < a.parts && l[j] != -__builtin_inff()) ? expf(l[j] - m_new) : 0.f;
      tot += w;
#pragma unroll
      for (int e = 0; e < DPT; ++e) acc[e] += w * o[j][e];
    }
    M = m_new;
    if (ONCE) break;
  }
}
template <typename T, int DPT>
__device__ __forceinline__ void store_piece(const MergeArgs& a, int row, int c, float M, float tot, const float (&acc)[DPT]) {
  const float inv = tot > 0.f ? 1.f / tot : 0.f;
  const int bh = row / a.n_q, i = row - bh * a.n_q;
  T* op = (T*)a.out + (int64_t)bh * a.out_head_stride + (int64_t)i * a.head_dim + DPT * c;
  if constexpr (sizeof(T) == 2) {
    uint32_t w[DPT / 2];
#pragma unroll
    for (int q = 0; q < DPT / 2; ++q)
      w[q] = (uint32_t)f32_to_bf16(acc[2 * q] * inv) | ((uint32_t)f32_to_bf16(acc[2 * q + 1] * inv) << 16);
    if constexpr (DPT == 8) *(uint4*)op = make_uint4(w[0], w[1], w[2], w[3]);
    else *(uint2*)op = make_uint2(w[0], w[1]);
  } else {
#pragma unroll
    for (int e = 0; e < DPT; ++e) op[e] = acc[e] * inv;
  }
  if (a.lse != nullptr && c == 0) a.lse[row] = tot > 0.f ? M + logf(tot) : -__builtin_inff();
}

template <typename T, bool HALF, int CH>
__global__ void __launch_bounds__(256) merge_kernel(MergeArgs a) {
  constexpr int DPT = HALF ? 8 : 4;  // dims per thread
  const int tpr = a.head_dim / DPT;
  const int rows_per_wg = 256 / tpr;
  // Workgroups in the attention's XCD order (reversed, consecutive ids on one
  // XCD): where a kv head's parts were written by the workgroups of one XCD, the
  // rows of that kv head are merged on the same XCD and read its L2.
  const int wg = (int)gridDim.x - 1 - xcd_logical_block(blockIdx.x, gridDim.x);
  const int row = wg * rows_per_wg + threadIdx.x / tpr;
  const int c = threadIdx.x % tpr;
  if (row >= a.rows) return;
  float M, tot, acc[DPT];
  join_parts<HALF, CH, (CH < 8)>(a, row, c, 0, 1, M, tot, acc);
  store_piece<T, DPT>(a, row, c, M, tot, acc);
}

// More than 8 parts: one workgroup per row.
template <typename T, bool HALF>
__global__ void __launch_bounds__(256) merge_many_kernel(MergeArgs a) {
  constexpr int DPT = HALF ? 8 : 4, CH = 4;
  const int row = blockIdx.x;
  const int tpr = a.head_dim / DPT, groups = 256 / tpr;  // 8 to 32 groups
  const int c = threadIdx.x % tpr, grp = threadIdx.x / tpr;
  __shared__ float sM[32], sT[32], sO[256 * DPT];
  float M, tot, acc[DPT];
  if (a.parts <= CH * groups) join_parts<HALF, CH, true>(a, row, c, grp, groups, M, tot, acc);
  else join_parts<HALF, CH, false>(a, row, c, grp, groups, M, tot, acc);
  if (c == 0) {
    sM[grp] = M;
    sT[grp] = tot;
  }
#pragma unroll
  for (int e = 0; e < DPT; ++e) sO[threadIdx.x * DPT + e] = acc[e];
  __syncthreads();
  if (grp != 0) return;
  for (int g = 0; g < groups; ++g) M = fmaxf(M, sM[g]);
  tot = 0.f;
#pragma unroll
  for (int e = 0; e < DPT; ++e) acc[e] = 0.f;
  if (M != -__builtin_inff()) {
    for (int g = 0; g < groups; ++g) {
      const float w = sM[g] == -__builtin_inff() ? 0.f : expf(sM[g] - M);
      tot += w * sT[g];
#pragma unroll
      for (int e = 0; e < DPT; ++e) acc[e] += w * sO[(g * tpr + c) * DPT + e];
    }
  }
  store_piece<T, DPT>(a, row, c, M, tot, acc);
}

constexpr int kManyRows = 1024;  // most rows whose many parts are split over threads

template <typename T, bool HALF>
hipError_t launch_merge_t(const MergeArgs& a, hipStream_t s) {
  constexpr int DPT = HALF ? 8 : 4;
  const int rows_per_wg = 256 / (a.head_dim / DPT);
  const dim3 grid((a.rows + rows_per_wg - 1) / rows_per_wg), block(256);
  // (at least half of a workgroup's groups with a part, or the join of the others' shares
  // shows: 10 parts of 320 rows of 64 dims, 32 groups, 7.6 us split and 5.0 not)
  const int groups = 256 / (a.head_dim / DPT);
  if (a.parts > max(8, groups / 2) && a.rows <= kManyRows) {
    hipLaunchKernelGGL((merge_many_kernel<T, HALF>), dim3(a.rows), block, 0, s, a);
    return hipGetLastError();
  }
  switch (a.parts) {
    case 2: hipLaunchKernelGGL((merge_kernel<T, HALF, 2>), grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL((merge_kernel<T, HALF, 3>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((merge_kernel<T, HALF, 4>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((merge_kernel<T, HALF, 8>), grid, block, 0, s, a); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_merge(const MergeArgs& a, hipStream_t s) {
  if (a.rows == 0) return hipSuccess;
  return a.bf16 ? launch_merge_t<bf16_t, true>(a, s) : launch_merge_t<float, false>(a, s);
}

}  // namespace infllm

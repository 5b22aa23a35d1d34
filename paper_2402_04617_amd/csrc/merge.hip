// Log-sum-exp merge of partial attentions over disjoint key parts:
// LSE = log sum_s exp(lse_s), O = sum_s exp(lse_s - LSE) O_s.  The parts together
// are the single softmax over Concat(C, X) of Section 3.1.
//
// One thread per (row, 16 bytes of partial row): 8 dims of a scaled-fp16 partial
// (bfloat16 inputs; value * 2^exp[row] restores the row) or 4 dims of a float32
// one.  Up to 8 parts: one thread takes them all (CH = the part count, or 8), every
// load issued before the first use.  More parts (decoding): a workgroup per row, its
// threads split into groups that take every GR-th part and are joined in LDS -- with
// few rows the parts are the only parallelism (25 parts of 32 rows, one thread per
// piece and 8 parts at a time: 6.8 us; split: 4.3).
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
// The softmax join of CH parts: running maximum, weight sum and weighted rows.
template <int CH, int DPT>
__device__ __forceinline__ void join(const float (&l)[CH], const float (&o)[CH][DPT], int n, float& M, float& tot,
                                     float (&acc)[DPT]) {
  M = -__builtin_inff();
#pragma unroll
  for (int j = 0; j < CH; ++j)
    if (j < n) M = fmaxf(M, l[j]);
  tot = 0.f;
#pragma unroll
  for (int e = 0; e < DPT; ++e) acc[e] = 0.f;
  if (M == -__builtin_inff()) return;  // nothing visible
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const float w = (j < n && l[j] != -__builtin_inff()) ? expf(l[j] - M) : 0.f;
    tot += w;
#pragma unroll
    for (int e = 0; e < DPT; ++e) acc[e] += w * o[j][e];
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
  float l[CH], o[CH][DPT], M, tot, acc[DPT];
#pragma unroll
  for (int j = 0; j < CH; ++j) load_piece<HALF>(a, (int64_t)min(j, a.parts - 1) * a.rows + row, c, o[j], l[j]);
  join<CH, DPT>(l, o, a.parts, M, tot, acc);
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
  float M = -__builtin_inff(), tot = 0.f, acc[DPT];
#pragma unroll
  for (int e = 0; e < DPT; ++e) acc[e] = 0.f;
  for (int p0 = grp; p0 < a.parts; p0 += CH * groups) {
    float l[CH], o[CH][DPT], m, t, x[DPT];
    const int n = (a.parts - p0 + groups - 1) / groups;  // parts left to this group
#pragma unroll
    for (int j = 0; j < CH; ++j)
      load_piece<HALF>(a, (int64_t)min(p0 + j * groups, a.parts - 1) * a.rows + row, c, o[j], l[j]);
    join<CH, DPT>(l, o, n, m, t, x);
    const float mn = fmaxf(M, m);
    if (mn == -__builtin_inff()) continue;
    const float w0 = M == -__builtin_inff() ? 0.f : expf(M - mn), w1 = m == -__builtin_inff() ? 0.f : expf(m - mn);
    tot = tot * w0 + t * w1;
#pragma unroll
    for (int e = 0; e < DPT; ++e) acc[e] = acc[e] * w0 + x[e] * w1;
    M = mn;
  }
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

template <typename T, bool HALF>
hipError_t launch_merge_t(const MergeArgs& a, hipStream_t s) {
  constexpr int DPT = HALF ? 8 : 4;
  const int rows_per_wg = 256 / (a.head_dim / DPT);
  const dim3 grid((a.rows + rows_per_wg - 1) / rows_per_wg), block(256);
  if (a.parts > 8) {
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

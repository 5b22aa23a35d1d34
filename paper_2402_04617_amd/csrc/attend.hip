// Attention dispatch (bfloat16 chunks: matrix-core kernel; bfloat16 decoding:
// the bandwidth kernel of attend_decode.hip), plus the float32 kernel:
//  - attend_f32_kernel: float32 inputs (any n_q), float32 matrix cores, expf online
//    softmax; the float32 accuracy path.  It reads keys through the same
//    virtual key axis as the other kernels.
#include <algorithm>

#include "launch.h"

namespace infllm {

hipError_t launch_attend_mfma(const AttendArgs& a, hipStream_t s);
hipError_t launch_attend_decode(const AttendArgs& a, hipStream_t s);

namespace {

// ---------------------------------------------------------------- float32 path
// Direct global->LDS load of 16 bytes per lane (lane i lands at lds + 16*i), waited
// for by the kernel itself.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_load_lane(uint32_t lds, const void* p) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds), "v"(p) : "m0", "memory");
}
#pragma clang diagnostic pop
#define INFLLM_LDS __attribute__((address_space(3)))

constexpr int kF32Keys = 32;  // keys per tile
constexpr int kF32Sel = 2048;  // lookup entries kept in LDS

// Float32 attention on the matrix cores (v_mfma_f32_32x32x2_f32: float32 products
// and sums).  NW waves of 32 query rows each; the workgroup's keys come in tiles of
// 32 through two LDS buffers, loaded directly one tile ahead.
//  S^T = K Q^T: A = K rows from LDS, B = the wave's Q rows in registers.  The
//    contraction may take the dims in any order: a lane's half of k-steps 4i..4i+3
//    is dims 8i + 4*gsel .. +4, so that one 16-byte read feeds four k-steps.
//    Sums of 16 products are joined by additions (see scores).
//  O^T += V^T P^T: B = the probabilities as S^T leaves them (k-step (a, b) pairs
//    keys 8a + b and 8a + 4 + b, one per lane half), A = V rows from LDS; output
//    block db holds dims DBLK*m + db, so that one read feeds all DBLK blocks.
// In tiles of units the first wave's search for the keys of the tile after next waits for
// the tile just requested (a lookup entry lies in LDS or in memory and is read through one
// pointer), so only the other waves run ahead there.
// Rows of an LDS tile are XOR-swizzled by granule, which makes both reads
// conflict-free.  What bounds it: the matrix cores' float32 rate (64 cycles per
// instruction); with one wave per SIMD the softmax (expf, 16 scores per lane and
// tile) is exposed.  With one vector-ALU dot product and a shuffle reduction per
// (row, key) instead, a step of 256 queries of 8 heads (D 64) over 2,400 keys took
// 228 us against 43 now (D 128 287 and 63, remapped 290 and 75), with an error against
// 64 bits of 5.4 to 6.3e-7 against 4.3 to 4.4e-7 (three seeds).
// With the positional remap (ROPE) a wave holds both forms of its query rows; a tile
// of memory keys takes the one at distance l_L, a tile of local keys the other, and
// the tile that holds both kinds takes both and picks per key.
template <int D, int NW, bool ROPE>
__global__ void __launch_bounds__(64 * NW, 1) attend_f32_kernel(AttendArgs a) {
  constexpr int KT = kF32Keys, RW = 32 * NW;
  constexpr int QL = D / 2;             // query dims per lane
  constexpr int DBLK = D / 32;          // 32-wide output blocks
  constexpr int GPR = D / 4;            // 16-byte granules per row
  constexpr int RPI = 64 / GPR;         // rows per load instruction
  constexpr int NI = KT / (RPI * NW);   // load instructions per wave and tile (K or V)
  __shared__ __attribute__((aligned(256))) float ks[2][KT * D];
  __shared__ __attribute__((aligned(256))) float vs[2][KT * D];
  __shared__ int64_t spos[3][KT];  // store positions of a tile's keys (0 where there is none)
  __shared__ __attribute__((aligned(4))) uint8_t sval[3][KT];
  __shared__ int32_t sidx[kF32Sel];

  const int G = a.n_q_heads / a.n_kv_heads;
  const int R = G * a.geom.n_q;
  const int n_row_tiles = (R + RW - 1) / RW;
  const int L = (int)gridDim.x - 1 - xcd_logical_block(blockIdx.x, gridDim.x);
  const int rt = L % n_row_tiles;
  const int tmp = L / n_row_tiles;
  const int part = tmp % a.parts;
  const int bg = tmp / a.parts;
  const int b = bg / a.n_kv_heads, g = bg - b * a.n_kv_heads;
  // this sequence's step (its own past length in a variable-length batch)
  const SeqStep sq = seq_step(a, b);
  const StepGeom& geo = sq.geom;
  const int mem_len = sq.mem_len;

  // the tiles the row tile's queries see, split evenly over the parts
  const int v_x0 = geo.n_virtual - geo.n_q;
  const int n_tiles = (v_x0 + (min(R, (rt + 1) * RW) - 1) / G) / KT + 1;
  const int t_begin = (int)((int64_t)n_tiles * part / a.parts), t_end = (int)((int64_t)n_tiles * (part + 1) / a.parts);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, gsel = lane >> 5;
  const int row = rt * RW + wave * 32 + n;
  const bool row_ok = row < R;
  const bool active = rt * RW + wave * 32 < R;  // whether the wave has rows at all
  const int qi = row_ok ? row / G : 0;
  const int qh = g * G + (row_ok ? row - qi * G : 0);
  const int vlim = v_x0 + qi;  // last visible key
  const int32_t* idx_row = a.idx + (int64_t)bg * geo.idx_stride;
  const float* kbase = (const float*)a.k_store + (int64_t)bg * a.capacity * D;
  const float* vbase = (const float*)a.v_store + (int64_t)bg * a.capacity * D;
  const float* krot = ROPE ? (const float*)a.k_rot + (int64_t)bg * a.capacity * D : nullptr;

  for (int u = tid; u < min(geo.n_sel, kF32Sel); u += 64 * NW) sidx[u] = idx_row[u];

  // Query pieces: qv as given; under the remap qv is the query at its own position
  // (L and X) and qm the query turned by R(l_L) (I and the units, keys unrotated).
  float qv[QL], qm[ROPE ? QL : 1];
  const float* qp = (const float*)a.q + (int64_t)(b * a.n_q_heads + qh) * a.q_head_stride + (int64_t)qi * D;
#pragma unroll
  for (int i = 0; i < QL / 4; ++i) {
    const f32x4 x = row_ok ? *(const f32x4*)(qp + 8 * i + 4 * gsel) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e) qv[4 * i + e] = x[e];
  }
  if constexpr (ROPE) {
#pragma unroll
    for (int j = 0; j < QL / 2; ++j) {
      const int pr = 4 * (j >> 1) + 2 * gsel + (j & 1);  // the pair held in qv[2j], qv[2j+1]
      const float x0 = qv[2 * j], x1 = qv[2 * j + 1];
      float c, sn;
      rope_cos_sin(a.rope, geo.past_len + qi, pr, c, sn);
      qv[2 * j] = x0 * c - x1 * sn;
      qv[2 * j + 1] = x0 * sn + x1 * c;
      qm[2 * j] = x0 * a.rope.mem_cos[pr] - x1 * a.rope.mem_sin[pr];
      qm[2 * j + 1] = x0 * a.rope.mem_sin[pr] + x1 * a.rope.mem_cos[pr];
    }
  }

  // positions of tile t's keys, by the first 32 threads
  auto find_keys = [&](int t) {
    if (tid >= KT) return;
    const int v = t * KT + tid;
    int64_t pos = -1;
    if (v < geo.n_virtual) {
      const int w = v - geo.n_init, sel_len = geo.n_sel * geo.block_size;
      if (v < geo.n_init) {
        pos = v;
      } else if (w >= sel_len) {
        pos = geo.local_begin + (w - sel_len);
      } else {
        const int u = w / geo.block_size;
        const int bu = u < kF32Sel ? sidx[u] : idx_row[u];
        if (bu >= 0 && bu < geo.n_units) pos = (int64_t)geo.unit_base + (int64_t)bu * geo.block_size + (w - u * geo.block_size);
      }
    }
    const int slot = (t - t_begin) % 3;
    spos[slot][tid] = pos >= 0 ? pos : 0;  // position 0 is always written; masked
    sval[slot][tid] = pos >= 0;
  };
  const uint32_t lds_k = (uint32_t)(uintptr_t)(INFLLM_LDS float*)ks[0] + NI * wave * 1024;
  const uint32_t lds_v = (uint32_t)(uintptr_t)(INFLLM_LDS float*)vs[0] + NI * wave * 1024;
  constexpr uint32_t kTileBytes = KT * D * 4;
  // Loads of tile t: granule slot c of tile row r holds the row's granule c ^ (r & 15).
  auto load_tile = [&](int t) {
    const int slot = (t - t_begin) % 3;
    const uint32_t buf = ((t - t_begin) & 1) * kTileBytes;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int r = (NI * wave + j) * RPI + lane / GPR;
      const int gran = (lane % GPR) ^ (r & 15);
      const int64_t off = spos[slot][r] * D + 4 * gran;
      const float* kp = ROPE && t * KT + r >= mem_len ? krot : kbase;
      lds_load_lane(lds_k + buf + j * 1024, kp + off);
      lds_load_lane(lds_v + buf + j * 1024, vbase + off);
    }
  };

  f32x16 o[DBLK];
#pragma unroll
  for (int db = 0; db < DBLK; ++db)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[db][j] = 0.f;
  float m = -__builtin_inff(), l = 0.f;

  // S^T of the tile in buffer `kt` against one form of the query rows
  auto scores = [&](const float* kt, const float* qx) {
    // Sums of 16 products, joined: chains of 32 (64 at D = 128) took 41 us where this
    // takes 43, but left rows of short parts further from 64 bits than the vector ALU's
    // sums had (40 queries of 2 heads: 5.1e-7, 4.3e-7 now, 4.5e-7 there).
    f32x16 sum;
#pragma unroll
    for (int i0 = 0; i0 < QL / 4; i0 += 4) {
      f32x16 s0 = {}, s1 = {};
#pragma unroll
      for (int i = i0; i < i0 + 4; ++i) {
        const f32x4 kf = *(const f32x4*)(kt + n * D + 4 * ((2 * i + gsel) ^ (n & 15)));
        s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[0], qx[4 * i], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[1], qx[4 * i + 1], s1, 0, 0, 0);
        s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[2], qx[4 * i + 2], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[3], qx[4 * i + 3], s1, 0, 0, 0);
      }
      sum = i0 == 0 ? s0 + s1 : sum + (s0 + s1);
      if (ROPE && D == 128) __builtin_amdgcn_sched_barrier(0);  // (the registers of one group at a time)
    }
    return sum;
  };

  if (t_begin < t_end) {
    __syncthreads();  // sidx
    find_keys(t_begin);
    find_keys(t_begin + 1);
    __syncthreads();
    load_tile(t_begin);
  }
  for (int t = t_begin; t < t_end; ++t) {
    asm volatile("s_waitcnt vmcnt(0)");  // this wave's part of tile t has landed
    __syncthreads();                     // every wave's has; the other buffer is free
    if (t + 1 < t_end) load_tile(t + 1);
    find_keys(t + 2);
    if (!active) continue;
    const int buf = (t - t_begin) & 1, slot = (t - t_begin) % 3;
    f32x16 s;
    if constexpr (ROPE) {
      if (t * KT >= mem_len) {
        s = scores(ks[buf], qv);
      } else if ((t + 1) * KT <= mem_len) {
        s = scores(ks[buf], qm);
      } else {
        const f32x16 sl = scores(ks[buf], qv);
        s = scores(ks[buf], qm);
        const int first_local = mem_len - t * KT - 4 * gsel;
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (8 * (j >> 2) + (j & 3) >= first_local) s[j] = sl[j];
      }
    } else {
      s = scores(ks[buf], qv);
    }
    // mask and the tile's maximum (both lane halves of a row)
    const int lim = vlim - t * KT - 4 * gsel;
    float mx = -__builtin_inff();
    uint32_t seen = 0;  // this lane's visible keys
#pragma unroll
    for (int j4 = 0; j4 < 4; ++j4) {
      const uint32_t kv = *(const uint32_t*)&sval[slot][8 * j4 + 4 * gsel];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 4 * j4 + e;
        const bool vis = 8 * j4 + e <= lim && ((kv >> (8 * e)) & 0xFFu) != 0;
        seen |= vis ? 1u << j : 0u;
        s[j] = vis ? s[j] * a.sm_scale : -__builtin_inff();
        mx = fmaxf(mx, s[j]);
      }
    }
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    if (__ballot(mx > m)) {  // some row's maximum grows (the first visible tile included)
      const float m_new = fmaxf(m, mx);
      const float corr = m_new == -__builtin_inff() ? 1.f : expf(m - m_new);
      m = m_new;
      l *= corr;
#pragma unroll
      for (int db = 0; db < DBLK; ++db)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[db][j] *= corr;
    }
    const float base = m == -__builtin_inff() ? 0.f : m;
    float ls[2] = {0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      s[j] = expf(s[j] - base);
      ls[j & 1] += s[j];
    }
    l += ls[0] + ls[1];
    typedef float vfrag_t __attribute__((ext_vector_type(DBLK)));
    auto value_row = [&](int r, int d0) {
      return *(const vfrag_t*)(vs[buf] + r * D + 4 * ((d0 >> 2) ^ (r & 15)) + (d0 & 3));
    };
    auto add_keys = [&](int j, const vfrag_t& vf) {
#pragma unroll
      for (int db = 0; db < DBLK; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[db], s[j], o[db], 0, 0, 0);
    };
    auto values = [&](int j) { return value_row(8 * (j >> 2) + 4 * gsel + (j & 3), DBLK * n); };  // this lane's dims
    if (__ballot(seen != 0xFFFFu) == 0) {
#pragma unroll
      for (int j = 0; j < 16; ++j) add_keys(j, values(j));
      continue;
    }
    // Values that are not finite must not reach rows that do not see their key (0 * inf):
    // in a tile with hidden keys such a pair of keys is added row by row.
    uint32_t apart = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const vfrag_t vf = values(j);
      float z = 0.f;
#pragma unroll
      for (int db = 0; db < DBLK; ++db) z += vf[db] * 0.f;
      if (__ballot(z != 0.f)) apart |= 1u << j;
      else add_keys(j, vf);
    }
    while (apart) {
      const int j = __builtin_ctz(apart);
      apart &= apart - 1;
      float pj = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) pj = i == j ? s[i] : pj;
      for (int h = 0; h < 2; ++h) {  // the pair's key of lane half h
        const float p = __shfl(pj, n + 32 * h);
        const bool vis = (__shfl((int)seen, n + 32 * h) >> j) & 1;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const vfrag_t vf = value_row(8 * (j >> 2) + 4 * h + (j & 3), DBLK * (8 * (i >> 2) + 4 * gsel + (i & 3)));
#pragma unroll
          for (int db = 0; db < DBLK; ++db) o[db][i] += vis ? p * vf[db] : 0.f;
        }
      }
    }
  }

  const auto lw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
  const float l_tot = __uint_as_float(lw[0]) + __uint_as_float(lw[1]);
  if (!row_ok) return;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const float lse_v = l_tot > 0.f ? m + logf(l_tot) : -__builtin_inff();
  const int64_t grow = (int64_t)(b * a.n_q_heads + qh) * geo.n_q + qi;
  const int64_t rows_total = (int64_t)a.batch * a.n_q_heads * geo.n_q;
  float* op = a.parts == 1 ? (float*)a.out + (int64_t)(b * a.n_q_heads + qh) * a.out_head_stride + (int64_t)qi * D
                           : (float*)a.part_o + ((int64_t)part * rows_total + grow) * D;
  typedef float orow_t __attribute__((ext_vector_type(DBLK)));
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    orow_t w;
#pragma unroll
    for (int db = 0; db < DBLK; ++db) w[db] = o[db][j] * inv;
    *(orow_t*)(op + DBLK * (8 * (j >> 2) + 4 * gsel + (j & 3))) = w;
  }
  if (gsel == 0) {
    if (a.parts > 1) a.part_lse[(int64_t)part * rows_total + grow] = lse_v;
    else if (a.lse != nullptr) a.lse[grow] = lse_v;
  }
}

// Waves (of 32 rows) per workgroup of the float32 kernel.
int f32_waves(int R) { return R > 64 ? 4 : R > 32 ? 2 : 1; }

template <int D, int NW>
void launch_f32(const AttendArgs& a, int blocks, hipStream_t s) {
  if (a.rope.on) hipLaunchKernelGGL((attend_f32_kernel<D, NW, true>), dim3(blocks), dim3(64 * NW), 0, s, a);
  else hipLaunchKernelGGL((attend_f32_kernel<D, NW, false>), dim3(blocks), dim3(64 * NW), 0, s, a);
}
template <int D>
void launch_f32_d(const AttendArgs& a, hipStream_t s) {
  const int R = a.n_q_heads / a.n_kv_heads * a.geom.n_q, nw = f32_waves(R);
  const int blocks = ((R + 32 * nw - 1) / (32 * nw)) * a.parts * a.batch * a.n_kv_heads;
  if (nw == 4) launch_f32<D, 4>(a, blocks, s);
  else if (nw == 2) launch_f32<D, 2>(a, blocks, s);
  else launch_f32<D, 1>(a, blocks, s);
}

bool decode_eligible(bool bf16, int n_q, int G, int n_sel) {
  return bf16 && n_q == 1 && (G == 1 || G == 2 || G == 4 || G == 8) && n_sel <= kDecodeMaxSel;
}

}  // namespace

// Most key parts of the decode kernel: of kDecodeMinWork keys * head_dim each.
static int decode_most_parts(int head_dim, int64_t n_virtual) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(kDecodeTargetWgs, n_virtual * head_dim / kDecodeMinWork));
}

// Key parts of the decode kernel: a short context whole, else the cheapest of the counts
// that just fit one or two workgroups per compute unit (and 8 and 16, which the merge joins
// in one and two passes).  In eighths of a tile: 3.5 tiles for each round of workgroups (their
// prologues and epilogues), half the tiles of a wave with and half without the padding of
// its buffers, and the merge.  Swept over 1 to 72 (sequence, kv head) pairs, groups of 1, 4
// and 8, 512 to 6,400 keys of 64 and 128 dims: within 1.5 % of the best count on average
// (parts of at least 256 keys for two workgroups per unit: 13 %; of 128: 8 %, and up to 40 %
// off where a few more workgroups than fit began a round of their own).
int attend_decode_parts(int bh, int G, int head_dim, int n_virtual) {
  if ((int64_t)n_virtual * head_dim * (G + 2) <= kDecodeWholeWork) return 1;
  const int most = decode_most_parts(head_dim, n_virtual);
  // many pairs: the count that just passes the target (where it leaves half the chip with one
  // workgroup fewer, only for long contexts: 200 pairs of 8,350 keys 186 us as 600 workgroups,
  // 200 as 400; of 1,100 keys 45 and 42)
  const int pass = (kDecodeTargetWgs + bh - 1) / bh;
  if (bh > kDecodeTargetWgs / 2 || (3 * bh > kDecodeTargetWgs && n_virtual >= 4096))
    return std::max(1, std::min(pass, n_virtual / 256));
  const int fit2 = kDecodeTargetWgs / bh, fit1 = kDecodeTargetWgs / 2 / bh;
  const int tile = decode_step_keys(head_dim);  // of all waves
  int best = 1, best_cost = 0;
  for (const int c : {1, 8, 16, fit1, fit2}) {
    int p = std::min(c, std::min(fit2, most));
    const int tiles = (n_virtual + p * tile - 1) / (p * tile);
    const bool few = tiles <= kDecodeShortTiles;
    // (no more for two workgroups per unit than fill the buffers of their waves)
    if (few && p > fit1) p = std::max(fit1, (n_virtual + kDecodeShortTiles * tile - 1) / (kDecodeShortTiles * tile));
    const int padded = few ? kDecodeShortTiles : (tiles + 2) / 3 * 3;
    const int rounds = (bh * p + kDecodeTargetWgs / 2 - 1) / (kDecodeTargetWgs / 2);
    const int cost = 28 * rounds + 4 * padded + (int)((int64_t)4 * n_virtual / (p * tile)) + (p > 1 ? 24 : 0) +
                     (p > 8 ? 16 : 0) + (p > 16 ? 4 : 0);
    if (best_cost == 0 || cost <= best_cost) {
      best = p;
      best_cost = cost;
    }
  }
  return best;
}

int attend_choose_parts(bool bf16, int batch, int n_q_heads, int n_kv_heads, int head_dim, int n_q, int n_sel,
                        int n_virtual, int max_parts, int* row_waves) {
  *row_waves = kMfmaWaves;
  const int G = n_q_heads / n_kv_heads;
  if (decode_eligible(bf16, n_q, G, n_sel))
    return std::min(attend_decode_parts(batch * n_kv_heads, G, head_dim, n_virtual), std::max(1, max_parts));
  const int R = G * n_q;
  const int key_tile = bf16 ? 64 : kF32Keys;
  const int n_tiles = (n_virtual + key_tile - 1) / key_tile;
  const int cap = std::min(bf16 ? 8 : 16, std::min(std::max(1, n_tiles / 2), std::max(1, max_parts)));
  // Both kernels put one wave on a SIMD's matrix core (float32) or eight on a compute
  // unit's (bf16) at a time, so a part count that starts a new round of workgroups for a few of
  // them is worse than a lower one.  A workgroup costs its tiles plus kPartCost (prologue and
  // epilogue), and any split the merge, kMergeCost tiles.  (56 row
  // tiles of 108 key tiles, a 389-query chunk: 5 parts, 280 workgroups, 84.5 us per
  // step; 4 parts, 224 workgroups, 63.8 us.  A 300-token prompt: 2 parts 25.4 us, 1
  // part and no merge 22.9 us.)
  // The row tiles of a chunk see the keys up to their last query, and the longest start
  // first, so that in several rounds long workgroups are followed by short ones: unsplit, r
  // rounds end after r workgroups of the size in their middle, or the longest.  (A prompt of
  // 1,500 tokens, 8 kv heads of group 8: 376 workgroups of 1 part 86 us, 752 of 2 parts 97.
  // Splits are charged their longest part each round: by their middle, a 1M chunk would run
  // as two rounds of half the keys, 333 us instead of 326.)
  constexpr int kPartCost = 5, kMergeCost = 3;
  int best = 1;
  int64_t best_cost = 0;
  // (costs in quarters of a tile of a full workgroup; a half-filled bf16 workgroup,
  // one wave per SIMD, takes about kHalfTile/4 of that tile's time: a 300-token
  // prompt as 80 half-filled workgroups 17.7 us per step, as 40 full ones 21)
  constexpr int kHalfTile = 3;
  for (int half = 0; half < (bf16 ? 2 : 1); ++half) {
    const int waves = bf16 ? (half ? kMfmaWaves / 2 : kMfmaWaves) : f32_waves(R);
    const int row_tiles = batch * n_kv_heads * ((R + 32 * waves - 1) / (32 * waves));
    const int per_round = bf16 ? kMfmaTargetWgs : kMfmaTargetWgs * 4 / waves;
    const int tile_cost = half || R <= 32 * kMfmaWaves / 2 ? kHalfTile : 4;
    for (int p = 1; p <= cap; ++p) {
      const int64_t wgs = (int64_t)row_tiles * p, rounds = (wgs + per_round - 1) / per_round;
      auto wg_cost = [&](int64_t tiles) { return 4 * kPartCost + (tile_cost * tiles + p - 1) / p; };
      int64_t cost = rounds * wg_cost(n_tiles) + (p > 1 ? 4 * kMergeCost : 0);
      if (p == 1 && rounds > 1) {
        const int64_t after = std::max((int64_t)0, wgs - rounds * per_round / 2);  // workgroups after the middle one
        const int64_t mid_tiles = (n_virtual - n_q + n_q * after / wgs) / key_tile + 1;
        cost = std::max(wg_cost(n_tiles), rounds * wg_cost(std::min((int64_t)n_tiles, mid_tiles)));
      }
      if ((half == 0 && p == 1) || cost < best_cost) {
        best = p;
        best_cost = cost;
        *row_waves = waves;
      }
    }
  }
  return best;
}

// (an upper bound, for any batch)
int attend_max_parts(bool bf16, int G, int head_dim, int n_q, int64_t max_virtual) {
  if (decode_eligible(bf16, n_q, G, 0)) return decode_most_parts(head_dim, max_virtual);
  return bf16 ? 8 : 16;
}

bool attend_uses_mfma(const AttendArgs& a) {
  const int G = a.n_q_heads / a.n_kv_heads;
  return a.geom.n_q > 0 && a.bf16 && !decode_eligible(a.bf16, a.geom.n_q, G, a.geom.n_sel);
}

int attend_select_max(const AttendArgs& a) {
  if (attend_uses_mfma(a)) return a.geom.idx_stride <= kFusedSelectMaxK ? kFusedSelectMax : -1;
  const int G = a.n_q_heads / a.n_kv_heads;
  if (a.geom.n_q == 0 || !decode_eligible(a.bf16, a.geom.n_q, G, a.geom.n_sel)) return -1;
  // (of a row of at most n_sel units every unit is looked up, and nothing is selected)
  return a.geom.n_sel <= kWaveSelMaxK ? kDecodeSelMax : a.geom.n_sel;
}

hipError_t launch_attend(const AttendArgs& a, hipStream_t s) {
  if (a.geom.n_q == 0) return hipSuccess;
  const int G = a.n_q_heads / a.n_kv_heads;
  if (decode_eligible(a.bf16, a.geom.n_q, G, a.geom.n_sel)) return launch_attend_decode(a, s);
  if (a.bf16) return launch_attend_mfma(a, s);
  if (a.head_dim == 128) launch_f32_d<128>(a, s);
  else launch_f32_d<64>(a, s);
  return hipGetLastError();
}

}  // namespace infllm

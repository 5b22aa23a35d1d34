// Chunk attention over Concat(I, selected units, L, X) (Section 3.1) in bf16 on
// CDNA4 matrix cores (v_mfma_f32_32x32x16_bf16), fp32 accumulation.
//
// Work decomposition
//   rows   : per (sequence, kv head) the G*n_q query rows (row r -> query i = r/G,
//            head g*G + r%G), so the G heads sharing a K/V tile are packed together;
//            256 rows per workgroup (one per compute unit), 32 per wave, so each
//            K/V tile crosses into LDS once for all 8 waves.
//   keys   : the virtual key axis (see StepGeom) in tiles of 64 keys, gathered
//            straight from the token-ordered store (a selected unit is contiguous)
//            into LDS by direct global->LDS loads (no staging registers) through
//            four buffers, a pair of tiles per barrier; optionally split into parts whose partial softmaxes
//            are merged afterwards by log-sum-exp.
// Per wave and key tile:
//   S^T = K Q^T  : A = K tile rows from LDS, B = the wave's Q rows held in VGPRs.
//                  The 32x32 accumulator gives each lane one query row and 16 keys.
//   online softmax in the exp2 domain, row max combined across the two lane halves.
//   O^T += V^T P^T: B = P^T taken directly from the S^T accumulator (no shuffle);
//                  A = V^T fragments read from the key-major V tile with the LDS
//                  transpose read (ds_read_b64_tr_b16), in the key order the
//                  accumulator layout gives P^T.
#include "launch.h"
#include "topk_select.h"

namespace infllm {
namespace {

constexpr int KB = 64;      // keys per tile
constexpr int NWAVE = kMfmaWaves;

typedef short i16x4 __attribute__((ext_vector_type(4)));
#define INFLLM_LDS __attribute__((address_space(3)))

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Direct global->LDS loads (16 bytes per lane; lane i lands at LDS byte
// lds + 16*i, lds taken from M0).  Written as inline assembly so that the
// compiler does not guard every later LDS read with a wait for these loads: the
// kernel waits for them itself (s_waitcnt before the barrier that publishes a
// tile).  No compiler-generated code in these kernels uses M0.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// Wave-uniform base address plus a per-lane 32-bit byte offset.
__device__ __forceinline__ void lds_load(uint32_t lds, const void* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(off), "s"(base) : "m0");
}
// A full per-lane address.
__device__ __forceinline__ void lds_load_lane(uint32_t lds, const void* p) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds), "v"(p) : "m0");
}
#pragma clang diagnostic pop

// Values the compiler must treat as produced here (keeps derived addresses from
// being hoisted out of the tile loop into long-lived registers).
__device__ __forceinline__ uint32_t opaque_v(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ uint32_t opaque_s(uint32_t x) {
  asm volatile("" : "+s"(x));
  return x;
}

// Both LDS tiles are key-major [64 keys][D], unpadded, with the 16-byte granules
// of row r XOR-swizzled (granule g stored at g ^ swz(r)), and a 1 KB direct-load
// instruction still writes one contiguous LDS range.  gfx950 LDS serves 256
// bytes per clock (64 banks); for D = 128 (256-byte rows) the 4-bit swizzle
// below makes both fragment reads conflict-free: the K reads (16 consecutive
// rows, one granule each, per clock) and the transposed V reads (per 32 lanes:
// 4 consecutive rows x 64 bytes).  For D = 64 the 3-bit swizzle r & 7.
template <int D>
__device__ __forceinline__ int swz(int r) {
  if constexpr (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  else return r & 7;
}
template <int D>
__device__ __forceinline__ int tile_off(int r, int g) { return r * D + 8 * (g ^ swz<D>(r)); }

constexpr int NBUF = 4;         // K and V tile buffers: a pair of tiles in use, the next pair in flight
constexpr float kMaskCost = 1.5f;  // cost of a masked tile, in plain tiles
// The in-prologue unit selection, in plain tiles.  Rows of at most 1,024 units: 0.5, 1, 1.5 and 2
// tiles make a 128K chunk 90.1, 89.3, 89.2 and 90.2 us, a 389-query chunk at 32K 62.1, 63.1,
// 62.0 and 62.0, four sequences of 24 tokens 44.4, 44.0, 44.7 and 44.7, 256 tokens at 64K 55.9,
// 56.0, 57.1 and 57.4; longer rows: 1, 2 and 3 tiles make 512 tokens at 1M 94.3, 95.5 and 96.9.
constexpr float kSelTiles = 1.f;
constexpr int kRowTable = 4096;  // key-group positions kept in LDS (512 tiles of 8-key groups, 64 of single keys)
constexpr int kSelLds = 1024;    // lookup entries kept in LDS
static_assert(kFusedSelectMaxK <= kSelLds, "a selected lookup row fits in LDS");

constexpr uint32_t kNoRow = 0xFFFFFFFFu;

template <int D>
struct Smem {
  bf16_t k[NBUF][KB * D];
  bf16_t v[NBUF][KB * D];
  uint32_t rows[kRowTable];  // store position of each key group of a window of tiles (kNoRow: skipped entry)
  int32_t sidx[kSelLds];    // the lookup row (its first kSelLds entries)
  int32_t sel_ok;           // whether the first wave's select wrote it
  uint8_t kvalid[NBUF][KB];
};

// Publish LDS tiles to the workgroup: wait until at most N of this wave's
// direct loads are still in flight (older loads -- the tiles about to be read
// -- have landed in LDS) and its own LDS traffic is done, then barrier.  Written
// out so that no wait for the younger loads is implied.
template <int N>
__device__ __forceinline__ void publish_barrier() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N));
  lds_barrier();
}

// SEL > 0: the workgroups select the lookup themselves from a.sel_scores (2: rows of
// at most kFusedSelectShort units, by one wave; 16: longer rows, 16 keys per thread
// of all waves) -- kernels of their own, so that the plain
// kernel's code is unaffected.  MASS (with SEL):
// for every tile of the looked-up units the kernel also stores, per query row,
// the tile's sum of P = exp2(S*c2 - m) and the running max m it was formed
// against, from which the attention mass of each unit follows once the final
// lse is known (mass_parts_kernel).
template <int D, int SEL, bool MASS>
__global__ void __launch_bounds__(64 * NWAVE, 1) attend_mfma_kernel(AttendArgs a) {
  constexpr int CH = D / 8;                   // 16-byte granules per row
  constexpr int KSTEPS = D / 16;              // MFMA k-steps over the head dim
  constexpr int DBLK = D / 32;                // 32-wide output blocks
  constexpr int RPI = 64 / CH;                // tile rows per 1 KB load instruction
  constexpr int NI = KB * D * 2 / (NWAVE * 1024);  // load instructions per wave per tile (K or V)
  static_assert(NI * NWAVE * RPI == KB, "tile rows covered exactly once");
  __shared__ __attribute__((aligned(256))) Smem<D> sm;

  // The prologue is latency: 10 us for a selecting workgroup and 6.7 for another of a
  // 128K step's 79, 7.4 and 4.7 since (arguments, divisions and the part bounds
  // 1.8 -> 0.9; selection 4.6 -> 2.9; the queries and K(t0) are requested before the
  // position table is filled).  In a workgroup whose tiles hold units the table does not
  // hide them: a lookup entry lies in LDS or in memory and is read through one pointer,
  // and that read waits for every load in flight.
  // Every argument the prologue reads, requested at once: read where they are used,
  // their cold cache lines were waited for one after another.
  asm volatile("" ::"s"(a.batch), "s"(a.capacity), "s"(a.q_head_stride), "s"(a.q), "s"(a.k_store), "s"(a.v_store),
               "s"(a.parts), "s"(a.row_waves), "s"(a.n_q_heads), "s"(a.n_kv_heads));
  asm volatile("" ::"s"(a.geom.n_init), "s"(a.geom.n_units), "s"(a.geom.n_sel), "s"(a.geom.block_size),
               "s"(a.geom.unit_base), "s"(a.geom.idx_stride), "s"(a.geom.local_begin), "s"(a.geom.past_len),
               "s"(a.geom.n_q), "s"(a.geom.n_virtual));
  asm volatile("" ::"s"(a.mem_len), "s"(a.parts_mem), "s"(a.rope.on), "s"(a.var.on), "s"(a.d_row_tiles.mul),
               "s"(a.d_parts.mul), "s"(a.d_kv.mul), "s"(a.d_group.mul), "s"(a.d_block.mul), "s"(a.sel_scores),
               "s"(a.sel_stride));
  const int G = (int)a.d_group.d;
  const int R = G * a.geom.n_q;
  const int n_row_tiles = (int)a.d_row_tiles.d;
  const int rows_wg = 32 * a.row_waves;
  // XCD-aware order, reversed so that the workgroups dispatched first are those
  // with the most work: the last key part (it holds the causal diagonal of X) and
  // the last row tiles (their queries see the most of X)
  const int L = (int)gridDim.x - 1 - xcd_logical_block(blockIdx.x, gridDim.x);
  const int tmp = div_by(L, a.d_row_tiles), rt = L - tmp * n_row_tiles;
  const int bg = div_by(tmp, a.d_parts), part = tmp - bg * a.parts;
  const int b = div_by(bg, a.d_kv), g = bg - b * a.n_kv_heads;
  // this sequence's step (its own past length in a variable-length batch)
  const SeqStep sq = seq_step(a, b);
  const StepGeom& geo = sq.geom;
  const int mem_len = sq.mem_len, parts_mem = sq.parts_mem;

  // This part's tiles.  Without the positional remap the parts split the tiles
  // evenly.  With it, parts [0, parts_mem) split the memory tiles [0,
  // ceil(mem_len/KB)) (I and the units: unrotated keys, queries turned by R(l_L))
  // and the other parts the local tiles [floor(mem_len/KB), n_tiles) (L and X:
  // rotated keys, queries at their own positions); a tile holding keys of both
  // kinds is taken by both sides, each masking the other's keys.
  const int n_tiles = (geo.n_virtual + KB - 1) / KB;
  const bool remap = a.rope.on != 0;
  const bool mem_part = part < parts_mem;
  int rt0 = 0, rt1 = n_tiles, rpart = part, rparts = a.parts;
  if (mem_part) {
    rt1 = (mem_len + KB - 1) / KB;
    rparts = parts_mem;
  } else if (parts_mem > 0) {
    rt0 = mem_len / KB;
    rpart = part - parts_mem;
    rparts = a.parts - parts_mem;
  }
  // The parts split the tiles this row tile's queries see by cost rather than by
  // count, so that they end together: a masked tile (the causal diagonal) costs
  // kMaskCost plain tiles, and with the selection inside (SEL) the parts that
  // read unit keys also select the units (see below), kSelTiles tiles of work
  // each: the tiles up to the end of the units are charged that work spread over
  // them, for the share of the parts expected to fall there.
  const int v_x0 = geo.n_virtual - geo.n_q;  // first current-token key
  const int qi_min = div_by(min(R - 1, rt * rows_wg), a.d_group);
  const int qi_max = div_by(min(R, (rt + 1) * rows_wg) - 1, a.d_group);
  const int vis_end = mem_part ? mem_len : v_x0 + qi_min + 1;  // every row of the tile sees the keys below
  rt1 = min(rt1, (v_x0 + qi_max) / KB + 1);                    // later tiles are fully causal-masked
  const int a_m = min(max(vis_end / KB, rt0), rt1);            // first masked tile
  int s_end = rt0;                                             // end of the tiles charged the selection
  float c_seltile = 1.f;
  if constexpr (SEL > 0) {
    if (geo.n_sel > 0 && geo.n_sel < geo.n_units) {
      const int u_end = (geo.n_init + geo.n_sel * geo.block_size + KB - 1) / KB;
      s_end = min(max(u_end, rt0), a_m);
      c_seltile += kSelTiles * (float)rparts * __builtin_amdgcn_rcpf((float)max(1, rt1 - rt0));
    }
  }
  const float c_sel = c_seltile * (float)(s_end - rt0), c_plain = c_sel + (float)(a_m - s_end);
  const float c_part = (c_plain + kMaskCost * (float)(rt1 - a_m)) * __builtin_amdgcn_rcpf((float)rparts);
  auto part_bound = [&](int pp) -> int {  // first tile of part pp of rparts (the same in every workgroup)
    if (pp == 0) return rt0;
    if (pp == rparts) return rt1;
    const float c = c_part * (float)pp;
    const int t = c <= c_sel     ? rt0 + (int)(c * __builtin_amdgcn_rcpf(c_seltile) + 0.5f)
                  : c <= c_plain ? s_end + (int)(c - c_sel + 0.5f)
                                 : a_m + (int)((c - c_plain) * (1.f / kMaskCost) + 0.5f);
    return min(max(t, rt0), rt1);
  };
  const int t_begin = part_bound(rpart);
  const int t_end = part_bound(rpart + 1);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, gsel = lane >> 5;
  const int row0 = rt * rows_wg + wave * 32;  // the wave's first row
  // A wave without rows (past the last query of a short or ragged chunk, or of the
  // unused half of a half-filled workgroup) computes nothing: it only loads its rows
  // of the tiles and keeps the barriers, which leaves its SIMD's matrix core and the
  // power budget to the others.
  const bool active = wave < a.row_waves && row0 < R;
  const int row = row0 + n;
  const bool row_ok = active && row < R;
  const int qi = row_ok ? div_by(row, a.d_group) : 0;
  // last virtual key this row may see: causal within X (which also excludes the
  // ragged end), or for a memory part of the remap the last memory key
  const int vlim = mem_part ? mem_len - 1 : v_x0 + qi;
  const int qh = g * G + (row_ok ? row - qi * G : 0);

  const int32_t* idx_row = a.idx + (int64_t)bg * geo.idx_stride;
  const bf16_t* kbase = (const bf16_t*)(remap && !mem_part ? a.k_rot : a.k_store) + (int64_t)bg * a.capacity * D;
  const bf16_t* vbase = (const bf16_t*)a.v_store + (int64_t)bg * a.capacity * D;

  // Whether a tile this workgroup loads (its own and those issued ahead, [t_begin,
  // t_end + 7)) may hold unit keys; only then does it need the lookup.
  const int u_t0 = geo.n_init / KB, u_t1 = (geo.n_init + geo.n_sel * geo.block_size + KB - 1) / KB;
  const bool units_here = t_begin < t_end && t_begin < u_t1 && t_end + 7 > u_t0;
  // Lookup inside the attention: such a workgroup selects the units itself; the
  // workgroup of row tile 0 and part 0 always does, and writes the row out (also
  // without units: it is then all -1).  Every entry is valid.
  static_assert(SEL == 0 || SEL == 2 || SEL == tk::kMaxPer, "select variants");
  static_assert(tk::kThreads == 64 * NWAVE && tk::kMaxPer * tk::kThreads >= kFusedSelectMax, "select layout");
  const bool sel_writer = SEL > 0 && rt == 0 && part == 0;
  const bool sel_here = SEL > 0 && (sel_writer || units_here);
  const bool sel_all = geo.n_sel == 0 || geo.n_sel == geo.n_units;  // every unit (or none) is looked up
  // by single waves, or by the radix select of all of them
  const bool sel_waves = SEL > 2 ? tk::long_select_fits<tk::kWavePer>(geo.n_units, geo.n_sel) : geo.n_sel <= tk::kWaveK;
  const float* srow = SEL > 0 ? a.sel_scores + (int64_t)bg * a.sel_stride : nullptr;
  // scores of the single-wave select: short rows in the first wave, 16 per lane; long
  // rows 16 per lane of every wave (loaded before the queries, whose latency overlaps)
  constexpr int WPER = tk::kWavePer;
  static_assert(tk::kWaveRow >= kFusedSelectShort, "a short row fits one wave");
  uint32_t wkey[WPER] = {};
  if (SEL > 0 && sel_here && !sel_all && sel_waves && (SEL > 2 || wave == 0)) {
#pragma unroll
    for (int j = 0; j < WPER; ++j)
      wkey[j] = __float_as_uint(srow[min(wave * tk::kWaveRow + 64 * j + lane, geo.n_units - 1)]);
  }
  uint32_t skey[SEL > 0 ? SEL : 1] = {};  // scores of the radix select, SEL per thread
  auto load_radix_keys = [&]() {
#pragma unroll
    for (int j = 0; j < SEL; ++j) skey[j] = tk::order_key(srow[min(tid + j * tk::kThreads, geo.n_units - 1)]);
  };
  if (SEL == 2 && sel_here && !sel_all && !sel_waves) load_radix_keys();

  // The wave's query rows go to LDS first, whole rows at a time, into the V buffers
  // (256 rows fill the four exactly; V loads start once they are read back), swizzled
  // like a K tile.  Loading them into registers directly made the compiler wait for
  // every tile load issued behind them.  A part without tiles loads none: nothing of it
  // waits for them, and the epilogue stages its rows over the V buffers.
  const uint32_t lds_k0 = (uint32_t)(uintptr_t)(INFLLM_LDS bf16_t*)sm.k[0];
  const uint32_t lds_v0 = (uint32_t)(uintptr_t)(INFLLM_LDS bf16_t*)sm.v[0];
  constexpr int NQ = 32 / RPI;  // load instructions for 32 rows
  const uint32_t lds_q = lds_v0 + wave * 32 * D * 2;
  // (query, head) of the rows this lane moves, here and in the epilogue: row0 + lane /
  // CH and every RPI-th after it, stepped without a division
  const int li0 = div_by(row0 + lane / CH, a.d_group), lh0 = row0 + lane / CH - li0 * G;
  const int step_i = div_by(RPI, a.d_group), step_h = RPI - step_i * G;
  auto next_row = [&](int& i, int& h) {
    i += step_i;
    h += step_h;
    const bool wrap = h >= G;
    h -= wrap ? G : 0;
    i += wrap ? 1 : 0;
  };
  if (active && t_begin < t_end) {
    // within the kv head's query rows 32-bit byte offsets do, unless the heads lie
    // very far apart
    const bf16_t* qg = (const bf16_t*)a.q + (int64_t)(b * a.n_q_heads + g * G) * a.q_head_stride;
    const bool near = (int64_t)G * a.q_head_stride < (1ll << 30);
    int i = li0, h = lh0;
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const int rr = RPI * j + lane / CH;
      const bool in = row0 + rr < R;
      const int ii = in ? i : 0, hh = in ? h : 0;
      const int gran = (lane % CH) ^ swz<D>(rr);
      if (near) {
        lds_load(lds_q + j * 1024, qg, 2u * ((uint32_t)hh * (uint32_t)a.q_head_stride + (uint32_t)ii * D + 8u * gran));
      } else {
        lds_load_lane(lds_q + j * 1024, qg + hh * a.q_head_stride + (int64_t)ii * D + 8 * gran);
      }
      next_row(i, h);
    }
  }
  // The lane's rotary table entries under the remap (granule lane % CH, four pairs)
  double rev[4];
  float mcos[4], msin[4];
  if (remap) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      rev[j] = a.rope.rev[4 * (lane % CH) + j];
      mcos[j] = a.rope.mem_cos[4 * (lane % CH) + j];
      msin[j] = a.rope.mem_sin[4 * (lane % CH) + j];
    }
  }

  bool has_invalid = false;
  if constexpr (SEL == 0) {
    // The lookup row goes to LDS; skipped (out-of-range) entries send every tile
    // through the validity mask.
    if (units_here) {
      bool bad = false;
      for (int u = tid; u < geo.n_sel; u += 64 * NWAVE) {
        const int x = idx_row[u];
        if (u < kSelLds) sm.sidx[u] = x;
        bad |= (x < 0 || x >= geo.n_units);
      }
      has_invalid = __syncthreads_or(bad) != 0;
    }
  } else if (sel_here) {
    // (the select's scratch lies in the position table, filled after it)
    static_assert(sizeof(tk::LongSelSmem) <= sizeof(sm.rows) && sizeof(tk::WaveSelSmem) <= sizeof(sm.rows), "scratch");
    bool done = sel_all, published = false;
    if (sel_all) {
      for (int u = tid; u < geo.n_sel; u += 64 * NWAVE) sm.sidx[u] = u;
    } else if (sel_waves) {
#pragma unroll
      for (int j = 0; j < WPER; ++j) wkey[j] = tk::order_key(__uint_as_float(wkey[j]));
      if constexpr (SEL > 2) {
        done = tk::long_select<WPER>(wkey, geo.n_units, geo.n_sel, sm.sidx, *(tk::LongSelSmem*)sm.rows);
      } else {
        if (wave == 0) {
          const bool ok = tk::wave_select<WPER, false>(wkey, geo.n_units, geo.n_sel, sm.sidx, *(tk::WaveSelSmem*)sm.rows);
          if (lane == 0) sm.sel_ok = ok;
        }
        lds_barrier();
        done = published = sm.sel_ok != 0;
      }
    }
    if constexpr (SEL > 0) if (__builtin_expect(!done, 0)) {
      // more units than the waves' select takes, or too many candidates: the radix select,
      // SEL keys per thread, long rows filtered first (the filter declines, uniformly, when
      // the bound it finds leaves more than a thread's worth of candidates)
      if (SEL > 2 || sel_waves) load_radix_keys();
      auto valid = [&](int j) { return tid + j * tk::kThreads < geo.n_units; };
      auto index = [&](int j) { return tid + j * tk::kThreads; };
      uint32_t thr;
      int rem;
      bool ge;
      if constexpr (SEL > 2)
        done = geo.n_sel <= tk::kThreads && tk::filtered_select<SEL>(skey, geo.n_units, geo.n_sel, sm.sidx);
      if (!done) {
        tk::radix_threshold<SEL>(skey, valid, geo.n_sel, thr, rem, ge);
        tk::write_selection<SEL>(skey, valid, index, thr, rem, ge, geo.n_sel, sm.sidx);
      }
    }
    if (!published) lds_barrier();
    if (sel_writer) {
      int32_t* orow = a.idx_out + (int64_t)bg * geo.idx_stride;
      for (int u = tid; u < geo.idx_stride; u += 64 * NWAVE) orow[u] = u < geo.n_sel ? sm.sidx[u] : -1;
    }
  }

  // Direct loads: instruction j of wave w fills LDS granules [(NI*w + j)*64, +64)
  // of the tile, lane l writing granule slot l; that slot belongs to tile row
  // r_j = r_0 + RPI*j, r_0 = 8*w + l / CH, and holds its global granule
  // (l % CH) ^ swz(r_j); a wave's loads cover the eight rows [8w, 8w + 8).
  static_assert(NI * RPI == 8, "a wave loads eight rows of a tile");
  const int lrow0 = 8 * wave + lane / CH;

  // Store positions of the keys.  The virtual axis is cut into groups of 8 keys
  // when no group crosses a boundary between I, the units and the local run
  // (l_I and l_bs multiples of 8), else into single keys; a table in LDS holds the
  // position of every group's first key for a window of tiles.  A lane's load
  // offset is then one table read and three integer operations whatever the
  // tile holds -- no branch, no division in the tile loop.  (With per-tile run
  // starts, a branch to a per-key path and 64-bit arithmetic the bookkeeping
  // between the matrix phases took 870 of an iteration's 3,600 cycles.)
  const int gshift = ((geo.n_init | geo.block_size) & 7) == 0 ? 3 : 0;
  const int tile_groups = KB >> gshift;
  const int window = kRowTable / tile_groups;  // tiles in the table
  // The last position of the axis is the store's last written row: an offset past
  // it (a ragged end, a tile past the axis) reads that row instead, which the
  // causal bound masks.
  const uint32_t last_row = (uint32_t)(geo.past_len + geo.n_q - 1);
  auto group_row = [&](int v) -> uint32_t {
    int64_t pos = v;
    if (v >= geo.n_init) {
      const int w = v - geo.n_init;
      const int sel_len = geo.n_sel * geo.block_size;
      if (w >= sel_len) {
        pos = geo.local_begin + (w - sel_len);
      } else {
        const int u = div_by(w, a.d_block);
        const int bu = u < kSelLds ? sm.sidx[u] : idx_row[u];
        if (bu < 0 || bu >= geo.n_units) return kNoRow;
        pos = (int64_t)geo.unit_base + (int64_t)bu * geo.block_size + (w - u * geo.block_size);
      }
    }
    return (uint32_t)min(pos, (int64_t)last_row);
  };
  int w0 = t_begin;  // first tile of the table's window
  auto fill_rows = [&](int first) {
    w0 = first;
    const int n = min(kRowTable, (t_end + 7 - first) * tile_groups);
    for (int i = tid; i < n; i += 64 * NWAVE) sm.rows[i] = group_row(first * KB + (i << gshift));
  };
  // this lane's table entry of a tile, and its row within the group
  const uint32_t lds_rows = (uint32_t)(uintptr_t)(INFLLM_LDS uint32_t*)sm.rows;
  const uint32_t gr_mask = (1u << gshift) - 1u;
  // Byte offsets (from the slice base) of this lane's loads of tile `tile`.  The
  // host guarantees that one (sequence, kv head) slice of the store spans less than
  // 4 GiB.  A skipped unit entry reads row 0 -- always written -- and is masked.
  struct TileOff {
    uint32_t o[NI];
  };
  auto row_read = [&](int tile, uint32_t (&e)[NI]) {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const uint32_t at = lds_rows + 4u * ((uint32_t)(lrow0 + RPI * j) >> gshift);
      e[j] = *(const INFLLM_LDS uint32_t*)(uintptr_t)(at + 4u * (uint32_t)((tile - w0) * tile_groups));
    }
  };
  auto row_off = [&](const uint32_t (&e)[NI], TileOff& f) {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const uint32_t r = (uint32_t)(lrow0 + RPI * j);
      const uint32_t gran = (uint32_t)(lane % CH) ^ (uint32_t)swz<D>(lrow0 + RPI * j);
      const uint32_t base = has_invalid && e[j] == kNoRow ? 0u : e[j];
      f.o[j] = (min(base + (r & gr_mask), last_row) * (2u * D)) | (16u * gran);
    }
  };

  // Byte offsets of this wave's 1 KB slices in the LDS tiles.
  const uint32_t lds_k = lds_k0 + NI * wave * 1024;
  const uint32_t lds_v = lds_v0 + NI * wave * 1024;
  constexpr uint32_t kTileBytes = KB * D * 2;
  // load j of a tile into buffer `buf` of K or V
  auto load_k = [&](int buf, const TileOff& f, int j) { lds_load(lds_k + buf * kTileBytes + j * 1024, kbase, f.o[j]); };
  auto load_v = [&](int buf, const TileOff& f, int j) { lds_load(lds_v + buf * kTileBytes + j * 1024, vbase, f.o[j]); };
  // with skipped unit entries: the validity of the keys this wave loads into K buffer `buf`
  auto note_valid = [&](int buf, const uint32_t (&e)[NI]) {
    if (has_invalid) {
#pragma unroll
      for (int j = 0; j < NI; ++j)
        if (lane % CH == 0) sm.kvalid[buf][lrow0 + RPI * j] = e[j] != kNoRow;
    }
  };

  // Loop-invariant per-lane LDS offsets (elements); the swizzle depends on the
  // row only through r & 15, so +16 and +32 rows keep it.
  //  K fragment (S^T A operand) of k-step s: lane (n, gsel) reads row n (+32 for
  //  the second key block), granule 2s + gsel.
  //  V^T fragment (O^T A operand) of output block db: a transposed read by lane
  //  (h = lane/16, q = (lane%16)/4, m = lane%4) addresses key row
  //  16*j + 4*(h/2) + 8*e + q and dims 32*db + 16*(h%2) + 4*m .. +4; each lane then
  //  holds dim 32*db + lane%32 of keys 16*j + 4*gsel + 8*e + 0..3 -- the key order
  //  of the P^T operand taken from the S^T accumulator.
  // Under the swizzle these offsets are XOR-related (buffers start at multiples
  // of 256 bytes, so the XOR commutes with adding the buffer address):
  //   K, k-step s          : koff0 ^ 32*s                         (bytes)
  //   V^T, block db, half e: (voff0 ^ 64*db ^ VX*e) + e*16*D      (bytes)
  // so only two bases stay in registers and each tile derives its addresses.
  constexpr uint32_t VX = D == 128 ? 32 : 0;
  const uint32_t koff0 = 2u * tile_off<D>(n, gsel);
  uint32_t voff0;
  {
    const int h = lane >> 4, q = (lane & 15) >> 2, m = lane & 3;
    const int vr = 4 * (h >> 1) + q, d0 = 16 * (h & 1) + 4 * m;
    voff0 = 2u * (tile_off<D>(vr, d0 >> 3) + (d0 & 7));
  }
  auto kfrag_at = [&](uint32_t kaddr, int kb, int s) {
    return *(const INFLLM_LDS bf16x8*)(uintptr_t)((kaddr ^ (32u * s)) + kb * 64u * D);
  };
  auto vfrag_at = [&](uint32_t vaddr, int db, int j) {
    const uint32_t a0 = (vaddr ^ (64u * db)) + j * 32u * D;
    const uint32_t a1 = ((vaddr ^ (64u * db) ^ VX) + 16u * D) + j * 32u * D;
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((INFLLM_LDS i16x4*)(uintptr_t)a0);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((INFLLM_LDS i16x4*)(uintptr_t)a1);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // per-tile fragment base addresses (the buffer address is made opaque so that
  // the derived addresses are formed per tile instead of held in registers)
  auto kaddr_of = [&](int kbuf) { return opaque_s(lds_k0 + kbuf * kTileBytes) + koff0; };
  auto vaddr_of = [&](int vbuf) { return opaque_s(lds_v0 + vbuf * kTileBytes) + voff0; };

  // Q rows of this wave as the B operand (8 bf16 per lane per k-step), read back from
  // their LDS rows like K fragments.  Under the remap the rows are turned in place
  // first, by R(l_L) for a memory part and to their own positions for a local one:
  // a lane takes one granule of one query and turns it for all of the query's heads,
  // so that each angle's sine and cosine are formed once (per row and lane they took
  // 4.5 us of a local part's prologue).
  bf16x8 qreg[KSTEPS];
  auto read_q = [&]() {
    if (remap) {
      const int gr = lane % CH, r_end = min(row0 + 32, R);
      const int q_last = div_by(r_end - 1, a.d_group);
      for (int q = div_by(row0, a.d_group) + lane / CH; q <= q_last; q += RPI) {
        float cs[4], sn[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          cs[j] = mcos[j];
          sn[j] = msin[j];
          if (!mem_part) rope_cos_sin(rev[j], geo.past_len + q, cs[j], sn[j]);
        }
        for (int r = max(q * G, row0); r < min((q + 1) * G, r_end); ++r) {
          INFLLM_LDS u32x4* at = (INFLLM_LDS u32x4*)(uintptr_t)(lds_q + (r - row0) * (2 * D) + 16 * (gr ^ swz<D>(r - row0)));
          u32x4 raw = *at;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float x0 = __uint_as_float(raw[j] << 16), x1 = __uint_as_float(raw[j] & 0xFFFF0000u);
            raw[j] = (uint32_t)f32_to_bf16(x0 * cs[j] - x1 * sn[j]) | ((uint32_t)f32_to_bf16(x0 * sn[j] + x1 * cs[j]) << 16);
          }
          *at = raw;
        }
      }
      tk::wave_lds_fence();
    }
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s)
      qreg[s] = *(const INFLLM_LDS bf16x8*)(uintptr_t)((lds_q + koff0) ^ (32u * s));
  };

  f32x16 oacc[DBLK];
#pragma unroll
  for (int db = 0; db < DBLK; ++db)
#pragma unroll
    for (int j = 0; j < 16; ++j) oacc[db][j] = 0.f;
  float m_run = -__builtin_inff();
  float l_run = 0.f;
  const float c2 = a.sm_scale * 1.4426950408889634f;

  // ---- the pieces of one tile's work ----------------------------------------
  // S^T = K Q^T for the tile in K buffer `kb`: two accumulator chains (keys
  // [0,32) and [32,64)), K fragments read one k-step ahead.
  auto qk = [&](int kbuf, f32x16 (&sacc)[2]) {
    const uint32_t ka = kaddr_of(kbuf);
    auto kfrag = [&](int kb, int s) { return kfrag_at(ka, kb, s); };
    bf16x8 a0[2], a1[2];
    a0[0] = kfrag(0, 0);
    a1[0] = kfrag(1, 0);
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) {
      if (s + 1 < KSTEPS) {
        a0[(s + 1) & 1] = kfrag(0, s + 1);
        a1[(s + 1) & 1] = kfrag(1, s + 1);
      }
      if (s == 0) {
        const f32x16 zero = {};
        sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[0], qreg[0], zero, 0, 0, 0);
        sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[0], qreg[0], zero, 0, 0, 0);
      } else {
        sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[s & 1], qreg[s], sacc[0], 0, 0, 0);
        sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[s & 1], qreg[s], sacc[1], 0, 0, 0);
      }
    }
  };
  // Mask of tile t: key kl is visible to query qi iff its virtual index is at
  // most vlim and, with skipped unit entries present, its kvalid flag (K buffer
  // kbuf) is set.
  auto apply_mask = [&](int t, int kbuf, f32x16 (&sacc)[2]) {
    const int lim = vlim - t * KB - 4 * gsel;
    uint32_t kv[4][2];
    if (has_invalid) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int j4 = 0; j4 < 4; ++j4)
          kv[j4][kb] = *(const uint32_t*)&sm.kvalid[kbuf][32 * kb + 8 * j4 + 4 * gsel];
    }
    // one uniform branch for the tile, none per element
    if (has_invalid) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int c = 32 * kb + 8 * (j >> 2) + (j & 3);
          const bool vis = c <= lim && ((kv[j >> 2][kb] >> (8 * (j & 3))) & 0xFFu) != 0;
          sacc[kb][j] = vis ? sacc[kb][j] : -__builtin_inff();
        }
    } else {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int c = 32 * kb + 8 * (j >> 2) + (j & 3);
          sacc[kb][j] = c <= lim ? sacc[kb][j] : -__builtin_inff();
        }
    }
  };
  // Row max of the tile in the exp2 domain (both lane halves combined).
  auto tile_max = [&](const f32x16 (&sacc)[2]) {
    float mx = -__builtin_inff();
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int j = 0; j < 16; ++j) mx = fmaxf(mx, sacc[kb][j]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * c2;  // c2 > 0
  };
  // Lazy running max.  P is formed against the running max m_run without first
  // taking the tile's own maximum; a row whose sum of P over a tile exceeds kLazy
  // (2^16: P stays far inside the float and bf16 range) has met keys well above
  // m_run, and only then is the tile's maximum taken and the row rescaled (a rare
  // path; the decision is wave-uniform, and both lane halves of a row share
  // m_run).  While a row has seen no visible key (m_run = -inf) any nonzero P
  // takes that path, so the first visible tile sets m_run.
  constexpr float kLazy = 65536.f;
  float lazy_bound = 0.f;  // 0 while m_run = -inf
  float neg_m = 0.f;       // -m_run, 0 while m_run = -inf
  auto first_max = [&](float mx) {  // nothing accumulated yet
    m_run = mx;
    neg_m = (mx == -__builtin_inff()) ? 0.f : -mx;
    lazy_bound = (mx == -__builtin_inff()) ? 0.f : kLazy;
  };
  auto force_max = [&](float mx) {
    const float m_new = fmaxf(m_run, mx);
    const float alpha = (m_new == -__builtin_inff()) ? 1.f : fast_exp2(m_run - m_new);
    l_run *= alpha;
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
      for (int j = 0; j < 16; ++j) oacc[db][j] *= alpha;
    m_run = m_new;
    neg_m = (m_new == -__builtin_inff()) ? 0.f : -m_new;
    lazy_bound = (m_new == -__builtin_inff()) ? 0.f : kLazy;
  };
  // Tile t's contribution to the unit masses (MASS): for a tile of the looked-up
  // units (whole tiles: l_I and l_bs are multiples of the tile), the row's sum of
  // P over the tile's 64 keys (this lane's half plus the other lane half's) and
  // the running max it was formed against.  Later rescales of l_run leave the
  // stored pair valid: it carries its own max.
  auto mass_tile = [&](int t, float half_sum) {
    const int ut = t - geo.n_init / KB;  // tile index within the units
    const int n_ut = geo.n_sel * (geo.block_size / KB);
    if (ut < 0 || ut >= n_ut) return;
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(half_sum), __float_as_uint(half_sum), false,
                                                      false);
    const float tsum = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    if (row_ok && gsel == 0)
      a.mass_part[((int64_t)bg * a.mass_tiles + ut) * R + row] = make_float2(tsum, m_run);
  };
  // Two P values as a bf16 pair (one v_cvt_pk_bf16_f32), added unrounded to the
  // two running row sums (the normaliser keeps float32 precision; rounding only
  // the PV operand moves O by at most 2^-9 relative).
  auto p_pair = [&](float z0, float z1, float nm, float (&acc)[2], bool first) -> uint32_t {
    const float e0 = fast_exp2(__builtin_fmaf(z0, c2, nm));
    const float e1 = fast_exp2(__builtin_fmaf(z1, c2, nm));
    acc[0] = first ? e0 : acc[0] + e0;
    acc[1] = first ? e1 : acc[1] + e1;
    bf16x2 pr;
    pr[0] = (__bf16)e0;
    pr[1] = (__bf16)e1;
    // (opaque: the conversion stays in the matrix phase it is written in)
    return opaque_v(__builtin_bit_cast(uint32_t, pr));
  };
  // One 16-key half of P = exp2(S*c2 - m_run) as the bf16 operand pair, and its row sum.
  auto half_p = [&](const f32x16& sh, u32x4 (&ph)[2]) {
    float ps[2];
#pragma unroll
    for (int w = 0; w < 8; ++w) ph[w >> 2][w & 3] = p_pair(sh[2 * w], sh[2 * w + 1], neg_m, ps, w == 0);
    return ps[0] + ps[1];
  };
  auto as_bf16x8 = [](const u32x4& w) { return __builtin_bit_cast(bf16x8, w); };
  // O^T += V^T P^T over the four 16-key steps (V buffer vbuf); DBLK independent
  // accumulator chains, each V^T fragment two transposed 8-byte reads.
  auto pv = [&](int vbuf, const bf16x8 (&pb)[2][2]) {
    const uint32_t vaddr = vaddr_of(vbuf);
    auto vfrag = [&](int db, int j) { return vfrag_at(vaddr, db, j); };
    bf16x8 va[DBLK];
#pragma unroll
    for (int db = 0; db < DBLK; ++db) va[db] = vfrag(db, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int db = 0; db < DBLK; ++db) {
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[db], pb[j >> 1][j & 1], oacc[db], 0, 0, 0);
        if (j + 1 < 4) va[db] = vfrag(db, j + 1);
      }
    }
  };

  // ---- software pipeline over the part's tiles ---------------------------------
  // Tile x lives in K buffer and V buffer (x - t_begin) % 4.  A step of tile t runs
  // QK(t+1) and PV(t): the matrix cores work on QK(t+1) while the vector ALUs form
  // the keys [32, 64) half of P(t), and on PV(t) while they take the mask of tile
  // t+1 and form the keys [0, 32) half of P(t+1) with the running max; both halves
  // of a tile are checked against the lazy bound once, before PV(t).  Everything
  // else a step needs (load offsets, conversions, the first V^T fragments) is
  // formed inside those two phases, so that the matrix cores idle only where the
  // waves meet: one barrier per PAIR of tiles t, t+1.  At its top every load of the
  // previous pair has landed (K(t+1), K(t+2), V(t), V(t+1)); the pair's first phase
  // issues K(t+3), K(t+4), V(t+2), V(t+3) into the buffers whose readers the
  // barrier retired, nearly two tiles of work ahead of their use.  A tile past the
  // part's end is simply loaded too, into a buffer nobody reads.
  // What bounds it: power.  With three buffers, a barrier per tile, per-tile run
  // starts and two lazy checks an iteration took 3,600 cycles (2,048 of matrix work
  // for the two waves of a SIMD); it takes 3,200 now, at a clock that falls as the
  // loop gets denser (1.9 GHz in a 128K step; the loop alone runs 2,770 cycles at
  // 1.62 GHz, 1.7 us per tile, and 2.18 GHz on zeros).  Step at 1M (2,048 queries,
  // 162 tiles) 352 -> 333 us, at 128K 91.6 -> 90.3 us; 24 queries of four
  // sequences, five of eight waves idle, 65.6 -> 61.3 us.
  // Tiles whose keys every row of the workgroup sees need no mask unless skipped
  // unit entries exist.
  const int t_plain = has_invalid ? t_begin : max(t_begin, min(t_end, vis_end / KB));
  f32x16 sA[2], sB[2];
  // p0: the keys [0, 32) half of P(t), formed in the previous step's second phase
  // (or the prologue), and l_pend its row sum, added to l_run once the tile has
  // passed its lazy-max check; replaced there by that half of P(t+1).
  u32x4 p0[2];
  float l_pend = 0.f;
  // load offsets of tiles t+2, t+3, t+4 of the pair at hand, and the table entries
  // of K(t+3), K(t+4) (kept for their validity flags)
  TileOff off2, off3, off4;
  uint32_t e3[NI], e4[NI];
  // the offsets of the pair after the one whose second tile is t, in one go
  auto next_offsets = [&](int t) {
    off2 = off4;
    row_read(t + 4, e3);
    row_read(t + 5, e4);
    row_off(e3, off3);
    row_off(e4, off4);
  };
  // One tile's step: FIRST of the pair (issues the pair's loads) or second (forms
  // the next pair's load offsets); NEXT_MASK: tile t+1 is masked.
  auto tile_step = [&](int t, f32x16 (&cur)[2], f32x16 (&nxt)[2], auto first_of_pair, auto next_mask) {
    constexpr bool FIRST = decltype(first_of_pair)::value;
    constexpr bool MASK = decltype(next_mask)::value;
    const int bc = (t - t_begin) % NBUF, bn = (bc + 1) % NBUF;
    // Phase 1.  Chunk s issues the K fragment reads of k-step s+1, the two MFMAs of
    // k-step s and EPC elements of the second half of P(t); scheduling fences keep
    // that interleave.
    u32x4 w1[2];
    float ps1[2];  // two partial row sums (shorter dependency chains)
    bf16x8 va[DBLK];
    const uint32_t vaddr = vaddr_of(bc);
    auto vfrag = [&](int db, int j) { return vfrag_at(vaddr, db, j); };
    {
      const uint32_t ka = kaddr_of(bn);
      auto kfrag = [&](int kb, int s) { return kfrag_at(ka, kb, s); };
      bf16x8 a0[2], a1[2];
      a0[0] = kfrag(0, 0);
      a1[0] = kfrag(1, 0);
      constexpr int EPC = 16 / KSTEPS;  // elements of P(t)'s keys [32, 64) half per chunk
      static_assert(EPC % 2 == 0, "P elements are formed in bf16 pairs");
      static_assert(4 * NI <= KSTEPS, "one load per chunk");
#pragma unroll
      for (int s = 0; s < KSTEPS; ++s) {
        if (s + 1 < KSTEPS) {
          a0[(s + 1) & 1] = kfrag(0, s + 1);
          a1[(s + 1) & 1] = kfrag(1, s + 1);
        } else {
#pragma unroll
          for (int db = 0; db < DBLK; ++db) va[db] = vfrag(db, 0);
        }
        if (s == 0) {
          const f32x16 zero = {};
          nxt[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[0], qreg[0], zero, 0, 0, 0);
          nxt[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[0], qreg[0], zero, 0, 0, 0);
        } else {
          nxt[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[s & 1], qreg[s], nxt[0], 0, 0, 0);
          nxt[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[s & 1], qreg[s], nxt[1], 0, 0, 0);
        }
        if constexpr (FIRST) {
          // the s-th of this wave's 4*NI loads: K(t+3), V(t+2), K(t+4), V(t+3)
          const int i = s / NI, j = s % NI;
          if (i == 0) load_k((bc + 3) % NBUF, off3, j);
          else if (i == 1) load_v((bc + 2) % NBUF, off2, j);
          else if (i == 2) load_k(bc, off4, j);
          else if (i == 3) load_v((bc + 3) % NBUF, off3, j);
        }
#pragma unroll
        for (int i = 0; i < EPC; i += 2) {
          const int w = (EPC * s + i) >> 1;  // bf16 pair index within the half
          w1[w >> 2][w & 3] = p_pair(cur[1][2 * w], cur[1][2 * w + 1], neg_m, ps1, w == 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    float l_tile = l_pend + (ps1[0] + ps1[1]);
    // lazy-max check before the tile reaches the matrix cores: on the rare row that
    // exceeds the bound, rescale to the tile's maximum and redo both halves
    if (__ballot(l_tile > lazy_bound)) {
      force_max(tile_max(cur));
      l_tile = half_p(cur[0], p0);
      l_tile += half_p(cur[1], w1);
    }
    l_run += l_tile;
    if constexpr (MASS) mass_tile(t, l_tile);

    // Phase 2: PV(t) on the matrix cores; on the vector ALUs the mask of tile t+1
    // (one 8-element group of its 32 accumulator elements per step) and, four
    // elements per step, the keys [0, 32) half of P(t+1) against the running max.
    u32x4 q0[2];
    float ps0[2];
    {
      const int lim = vlim - (t + 1) * KB - 4 * gsel;  // mask bound of tile t+1
      uint32_t kv[4][2];
      if (MASK && has_invalid) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int j4 = 0; j4 < 4; ++j4)
            kv[j4][kb] = *(const uint32_t*)&sm.kvalid[bn][32 * kb + 8 * j4 + 4 * gsel];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if constexpr (!FIRST) {
          // the next pair's load offsets: V(t+3) .. of this pair's last K tile, then
          // the table entries of the two K tiles after it
          if (j == 0) {
            off2 = off4;
            row_read(t + 4, e3);
            row_read(t + 5, e4);
          } else if (j == 2) {
            row_off(e3, off3);
          } else if (j == 3) {
            row_off(e4, off4);
          }
        }
#pragma unroll
        for (int db = 0; db < DBLK; ++db) {
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[db], as_bf16x8(j < 2 ? p0[j & 1] : w1[j & 1]),
                                                            oacc[db], 0, 0, 0);
          if (j + 1 < 4) va[db] = vfrag(db, j + 1);
        }
        if constexpr (MASK) {
          // 8 of the 32 scores of tile t+1: elements [8j, 8j+8); one uniform branch
          // per step, none per element
          if (has_invalid) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const int e = 8 * j + i, kb = e >> 4, jj = e & 15;
              const int c = 32 * kb + 8 * (jj >> 2) + (jj & 3);
              const bool vis = c <= lim && ((kv[jj >> 2][kb] >> (8 * (jj & 3))) & 0xFFu) != 0;
              nxt[kb][jj] = vis ? nxt[kb][jj] : -__builtin_inff();
            }
          } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const int e = 8 * j + i, kb = e >> 4, jj = e & 15;
              const int c = 32 * kb + 8 * (jj >> 2) + (jj & 3);
              nxt[kb][jj] = c <= lim ? nxt[kb][jj] : -__builtin_inff();
            }
          }
        }
        // P(t+1), keys [0, 32): elements [4j, 4j+4) (masked by step j/2 <= j)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int w = 2 * j + i;
          q0[w >> 2][w & 3] = p_pair(nxt[0][2 * w], nxt[0][2 * w + 1], neg_m, ps0, w == 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    p0[0] = q0[0];
    p0[1] = q0[1];
    l_pend = ps0[0] + ps0[1];
  };
  // The top of a pair: its tiles' loads have landed, and the buffers of the
  // previous pair are free.
  auto pair_top = [&](int t) {
    __builtin_amdgcn_s_setprio(0);
    publish_barrier<0>();
    if (has_invalid) {
      note_valid((t - t_begin + 3) % NBUF, e3);
      note_valid((t - t_begin) % NBUF, e4);
    }
    if (t + 6 >= w0 + window) {
      // the second step reads the table for tiles t+5, t+6: move the window there
      // (its readers are past the barrier)
      fill_rows(t + 5);
      publish_barrier<0>();
    }
    // The matrix phases run at raised wave priority: a wave in its MFMA phases
    // wins the issue slots of its SIMD over a wave doing bookkeeping.
    __builtin_amdgcn_s_setprio(1);
  };
  auto copy_state = [](f32x16 (&dst)[2], const f32x16 (&src)[2]) {
    dst[0] = src[0];
    dst[1] = src[1];
  };

  if (t_begin < t_end) {
    // K(t0) needs no table: its rows' positions directly, so that the load is on its
    // way before the table is filled (where no unit is read: see above).
    TileOff off0, off1;
    {
      uint32_t e0[NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const uint32_t r = (uint32_t)(lrow0 + RPI * j);
        e0[j] = group_row(t_begin * KB + (int)(r & ~gr_mask));
      }
      row_off(e0, off0);
      note_valid(0, e0);
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) load_k(0, off0, j);
    fill_rows(t_begin);
    lds_barrier();
    {
      uint32_t e1[NI], e2[NI];
      row_read(t_begin + 1, e1);
      row_read(t_begin + 2, e2);
      row_read(t_begin + 3, e3);
      row_read(t_begin + 4, e4);
      row_off(e1, off1);
      row_off(e2, off2);
      row_off(e3, off3);
      row_off(e4, off4);
      note_valid(1, e1);
      note_valid(2, e2);
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) load_k(1, off1, j);
#pragma unroll
    for (int j = 0; j < NI; ++j) load_k(2, off2, j);
    // the query rows and K(t0) have landed ("memory": the reads of the rows stay behind it)
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * NI) : "memory");
    if (active) read_q();
    lds_barrier();  // K(t0) published, the query rows read
#pragma unroll
    for (int j = 0; j < NI; ++j) load_v(0, off0, j);
#pragma unroll
    for (int j = 0; j < NI; ++j) load_v(1, off1, j);
    if (!active) {
      int t = t_begin;
      for (; t + 2 < t_end; t += 2) {
        pair_top(t);
#pragma unroll
        for (int j = 0; j < NI; ++j) load_k((t - t_begin + 3) % NBUF, off3, j);
#pragma unroll
        for (int j = 0; j < NI; ++j) load_v((t - t_begin + 2) % NBUF, off2, j);
#pragma unroll
        for (int j = 0; j < NI; ++j) load_k((t - t_begin) % NBUF, off4, j);
#pragma unroll
        for (int j = 0; j < NI; ++j) load_v((t - t_begin + 3) % NBUF, off3, j);
        next_offsets(t + 1);
      }
      pair_top(t);  // (its loads are past the part's end)
    } else {
    qk(0, sA);
    if (t_begin >= t_plain) apply_mask(t_begin, 0, sA);
    if (!mem_part && parts_mem > 0 && t_begin * KB < mem_len) {
      // the first local tile also holds the last memory keys: hide them here
      const int lo = mem_len - t_begin * KB - 4 * gsel;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (32 * kb + 8 * (j >> 2) + (j & 3) < lo) sA[kb][j] = -__builtin_inff();
    }
    first_max(tile_max(sA));  // the first tile sets the running max
    l_pend = half_p(sA[0], p0);

    int t = t_begin;
    // pairs whose next tiles are plain, then the rest masked
    for (; t + 2 < t_plain; t += 2) {
      pair_top(t);
      tile_step(t, sA, sB, std::true_type{}, std::false_type{});
      tile_step(t + 1, sB, sA, std::false_type{}, std::false_type{});
    }
    for (; t + 2 < t_end; t += 2) {
      pair_top(t);
      tile_step(t, sA, sB, std::true_type{}, std::true_type{});
      tile_step(t + 1, sB, sA, std::false_type{}, std::true_type{});
    }
    pair_top(t);
    if (t + 1 < t_end) {
      tile_step(t, sA, sB, std::true_type{}, std::true_type{});
      copy_state(sA, sB);
      ++t;
    }
    // drain: P and PV of the last tile
    u32x4 w1[2];
    float l_tile = l_pend + half_p(sA[1], w1);
    if (__ballot(l_tile > lazy_bound)) {
      force_max(tile_max(sA));
      l_tile = half_p(sA[0], p0);
      l_tile += half_p(sA[1], w1);
    }
    l_run += l_tile;
    if constexpr (MASS) mass_tile(t, l_tile);
    const bf16x8 pb[2][2] = {{as_bf16x8(p0[0]), as_bf16x8(p0[1])}, {as_bf16x8(w1[0]), as_bf16x8(w1[1])}};
    pv((t - t_begin) % NBUF, pb);
    }
    publish_barrier<0>();  // no load is left in flight
    __builtin_amdgcn_s_setprio(0);
  }

  // Epilogue: combine the two lane halves' partial sums; write O (bf16, one part)
  // or the scaled fp16 partial row and lse.  The accumulator layout gives each
  // lane 8-byte pieces of its row; they are staged through LDS (the tile buffers
  // are free once every wave has passed the barrier below) so that each store
  // moves 16 contiguous bytes and a wave's store covers four whole rows.
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const float lse_v = (m_run == -__builtin_inff() || l_tot <= 0.f)
                          ? -__builtin_inff()
                          : (m_run + __log2f(l_tot)) * 0.6931471805599453f;
  const bool one_part = a.parts == 1;
  float sc = inv;
  int ex = 0;
  if (!one_part) {
    // fp16 partial row scaled by 2^-e (both lane halves of the row agree on e)
    float amax = 0.f;
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
      for (int j = 0; j < 16; ++j) amax = fmaxf(amax, fabsf(oacc[db][j]));
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(amax), __float_as_uint(amax), false, false);
    amax = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * inv;
    ex = partial_row_exponent(amax);
    sc = inv * exp2_int(-ex);
  }
  constexpr int kRowBytes = D * 2;
  constexpr int kStageRow = kRowBytes + 16;  // padded: the 32 rows of a wave spread over the LDS banks
  static_assert(NWAVE * 32 * kStageRow <= (int)sizeof(sm.k) + (int)sizeof(sm.v), "staging fits the tile buffers");
  __syncthreads();  // every wave is done with the tile buffers
  {
    INFLLM_LDS char* stage = (INFLLM_LDS char*)(INFLLM_LDS bf16_t*)sm.k[0] + wave * 32 * kStageRow;
#pragma unroll
    for (int db = 0; db < DBLK; ++db) {
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) {
        const int d = 32 * db + 8 * jq + 4 * gsel;
        const float o0 = oacc[db][4 * jq] * sc, o1 = oacc[db][4 * jq + 1] * sc;
        const float o2 = oacc[db][4 * jq + 2] * sc, o3 = oacc[db][4 * jq + 3] * sc;
        u32x2 w;
        if (one_part) {
          w[0] = (uint32_t)f32_to_bf16(o0) | ((uint32_t)f32_to_bf16(o1) << 16);
          w[1] = (uint32_t)f32_to_bf16(o2) | ((uint32_t)f32_to_bf16(o3) << 16);
        } else {
          w[0] = pack_f16x2(o0, o1);
          w[1] = pack_f16x2(o2, o3);
        }
        *(INFLLM_LDS u32x2*)(stage + n * kStageRow + d * 2) = w;
      }
    }
  }
  if (row_ok && gsel == 0) {
    const int64_t grow = ((int64_t)(b * a.n_q_heads + qh)) * geo.n_q + qi;
    if (one_part) {
      if (a.lse != nullptr) a.lse[grow] = lse_v;
    } else {
      const int64_t rows_total = (int64_t)a.batch * a.n_q_heads * geo.n_q;
      a.part_lse[(int64_t)part * rows_total + grow] = lse_v;
      a.part_exp[(int64_t)part * rows_total + grow] = ex;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  {
    constexpr int CPR = kRowBytes / 16;  // 16-byte chunks per row
    const INFLLM_LDS char* stage = (const INFLLM_LDS char*)(const INFLLM_LDS bf16_t*)sm.k[0] + wave * 32 * kStageRow;
    static_assert(CPR == CH, "a lane stores the rows it loaded");
    // first row of the kv head's group: [G][n_q] rows of a partial, or of the output
    const int64_t rows_total = (int64_t)a.batch * a.n_q_heads * geo.n_q;
    const int64_t head0 = b * a.n_q_heads + g * G;
    char* base = one_part ? (char*)a.out + head0 * a.out_head_stride * 2
                          : (char*)a.part_o + ((int64_t)part * rows_total + head0 * geo.n_q) * kRowBytes;
    const int64_t hstride = one_part ? a.out_head_stride * 2 : (int64_t)geo.n_q * kRowBytes;
    int i = li0, h = lh0;
#pragma unroll
    for (int k = 0; k < 32 * CPR / 64; ++k) {
      const int r = RPI * k + lane / CH, ch = lane % CH;
      const u32x4 w = *(const INFLLM_LDS u32x4*)(stage + r * kStageRow + ch * 16);
      if (active && row0 + r < R) *(u32x4*)(base + h * hstride + (int64_t)i * kRowBytes + ch * 16) = w;
      next_row(i, h);
    }
  }
}

}  // namespace

hipError_t launch_attend_mfma(const AttendArgs& args, hipStream_t s) {
  AttendArgs a = args;
  const int G = a.n_q_heads / a.n_kv_heads;
  const int R = G * a.geom.n_q;
  const int n_row_tiles = (R + 32 * a.row_waves - 1) / (32 * a.row_waves);
  a.d_row_tiles = fast_div(n_row_tiles);
  a.d_parts = fast_div(a.parts);
  a.d_kv = fast_div(a.n_kv_heads);
  a.d_group = fast_div(G);
  a.d_block = fast_div(a.geom.block_size);
  const int blocks = n_row_tiles * a.parts * a.batch * a.n_kv_heads;
  const dim3 grid(blocks), block(64 * NWAVE);
  const bool sel = a.idx_out != nullptr, mass = sel && a.mass_part != nullptr;
  if (sel && (a.sel_units < 0 || a.sel_units > kFusedSelectMax)) return hipErrorInvalidValue;
  const bool long_rows = sel && a.sel_units > kFusedSelectShort;
#define INFLLM_ATTEND_MFMA(DD)                                                                         \
  do {                                                                                                 \
    if (mass && long_rows) hipLaunchKernelGGL((attend_mfma_kernel<DD, 16, true>), grid, block, 0, s, a); \
    else if (mass) hipLaunchKernelGGL((attend_mfma_kernel<DD, 2, true>), grid, block, 0, s, a);          \
    else if (long_rows) hipLaunchKernelGGL((attend_mfma_kernel<DD, 16, false>), grid, block, 0, s, a);   \
    else if (sel) hipLaunchKernelGGL((attend_mfma_kernel<DD, 2, false>), grid, block, 0, s, a);          \
    else hipLaunchKernelGGL((attend_mfma_kernel<DD, 0, false>), grid, block, 0, s, a);                   \
  } while (0)
  if (a.head_dim == 128) INFLLM_ATTEND_MFMA(128);
  else INFLLM_ATTEND_MFMA(64);
#undef INFLLM_ATTEND_MFMA
  return hipGetLastError();
}

}  // namespace infllm

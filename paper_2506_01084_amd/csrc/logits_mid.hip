// extended_logits, base-vocabulary part for up to 192 hidden rows in all (gfx950, bf16, d a multiple of 64): a
// decode step of 65..192 sequences, one of 5..64 where the tiles fill the CUs (greedy or a draw), a few rows per sequence at a
// small batch, a short chunk; dense layers on up to 128 rows.  With one or two sequences of more than 64 rows the launch takes the
// tiles of W_hyper along, and the backward pass of the loss makes dZ here.  (zip2zip paper, section 2.3, steps 7-9.)
//
// With so few rows the part is bound by the bytes of W_base, like the one-row-per-sequence step.  That kernel's
// base units hold 64 hidden rows in registers (one pass over W_base per 64 rows); the 256 x 256 tile kernel shares
// both operands between its waves, which meet at every slab (3.4-3.5 TB/s of weights at these row counts).  Here:
//
//   workgroup = 8 waves = one tile of 256 weight rows x all hidden rows; wave w owns weight rows 32 w .. 32 w + 31:
//   2, 4 or 6 blocks of v_mfma_f32_32x32x16_bf16 (the kernel is built for up to 64, 128 and 192 rows).
//   K advances in slabs of 64.  A wave moves its own weights straight from global memory into a ring of its
//   own in LDS, four requests of 8 whole lines per slab, two or three slabs ahead, and reads its operands from there; nobody else
//   touches the ring, so it needs no barrier.  (Loaded in operand layout, 32 rows and half a line each way, a
//   request takes 64 pieces of 16 bytes: 1 GB of weights for 64 rows 190 us; through the ring 180; and since
//   every request takes whole lines, the weights can go past the caches, which the halves of a line cannot: 162, 6.5 TB/s.)
//   The hidden rows of a slab (up to 192 x 128 bytes, shared by the 8 waves, served by L2) go straight from global memory
//   into LDS stages, two slabs ahead (one in the 192-row build, which has room for two stages beside three ring slots), in the
//   tile kernel's swizzled layout (conflict-free operand reads); one barrier per slab.
//   The tiles start their walk over K at different slabs (+5-7 %: see below).
//   Where tiles of 256 would leave half of the CUs without one, a workgroup is four waves and 128 weight rows, and has the LDS
//   for both operands up to five slabs ahead (z2z_logits_mid_columns).
//
// V = 128256, d = 4096, whole calls in us, operand-layout loads -> ring: 8 x 5 rows 207 -> 187, 24 x 5 258 -> 211, steps of
// 16 / 64 / 100 / 128 sequences 213 -> 185, 272 -> 244, 340 -> 300, 365 -> 323,
// 160 / 192 438 -> 390, 480 -> 423.
// The fold of the finished tile into (max, sum-exp,
// argmax) triples is the tile kernel's; the 8 waves' triples of a hidden row are merged through LDS and leave one
// part per (row, weight tile).
#include "logits_mid.h"

#include <string.h>

namespace {

using namespace z2z_logits;

constexpr int M_WAVES = 8;                // of a workgroup; four where tiles of 256 weight rows are too few for the CUs
constexpr int M_WT = 32 * M_WAVES;        // weight rows of a workgroup's tile
constexpr int M_HT = 192;                 // hidden rows of a call at most (the builds below: 2, 4 or 6 blocks of 32)
constexpr int M_MAX_ROWS = M_HT;
static_assert(M_HT <= 64 * M_WAVES / 2, "a thread per row");
constexpr int M_SLAB = 128;               // bytes per row per K slab (64 bf16)
// LDS per build (blocks of 32 hidden rows, waves): stages of a slab's hidden rows, and slots of the waves' rings.  Four waves
// have the CU to themselves and ask for both up to five slabs ahead.
constexpr int mid_stages(int njv, int waves) { return waves == 4 ? (njv == 2 ? 6 : njv == 4 ? 5 : 4) : njv == 6 ? 2 : 3; }
constexpr int mid_ring(int njv, int waves) { return waves == 4 ? mid_stages(njv, 4) : njv == 2 ? 4 : 3; }
constexpr int mid_lds(int njv, int waves) {
  return mid_stages(njv, waves) * 32 * njv * M_SLAB + waves * 32 * M_SLAB * mid_ring(njv, waves);
}
constexpr int M_LDS_MAX = 160 * 1024;
static_assert(mid_lds(2, 8) <= M_LDS_MAX && mid_lds(4, 8) <= M_LDS_MAX && mid_lds(6, 8) <= M_LDS_MAX, "");
static_assert(mid_lds(2, 4) <= M_LDS_MAX && mid_lds(4, 4) <= M_LDS_MAX && mid_lds(6, 4) <= M_LDS_MAX, "");
static_assert(M_WAVES * M_HT * (int)(sizeof(Triple) + sizeof(Draw)) <= mid_lds(6, 8), "the waves' triples are merged in the idle stages and rings");

// 16 bytes per lane, global -> LDS without passing through registers (as in the tile kernel): address = 64-bit
// scalar base + 32-bit per-lane offset; the LDS address is the wave-uniform byte offset in M0 plus 16 * lane.
// Inline assembly, so the compiler does not count these loads: every wait for them is written out below.
__device__ __forceinline__ void load16_to_lds(const unsigned char* base, uint32_t lane_offset, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(lane_offset), "s"(base), "s"(lds_dst)
               : "memory");
}

// The same for bytes that nothing reads again before the caches have turned over: past them.
__device__ __forceinline__ void load16_to_lds_once(const unsigned char* base, uint32_t lane_offset, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
               :
               : "v"(lane_offset), "s"(base), "s"(lds_dst)
               : "memory");
}

// Wait until at most N of this wave's loads are in flight.  Inline assembly with a memory clobber: the compiler
// moves no load across it, so the number of requests that follow a given one is the number written below.
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

__device__ __forceinline__ uint32_t lds_offset_of(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// NJV: blocks of 32 hidden rows the instance is built for (rows of the tile <= 32 NJV); SMODE: 0 = fold the logits, 1 = fold logit / T and the Gumbel-max
// draw (a.sample = 1: part_v, part_l, and the drawn column in part_i), 2 = store logit / T and fold it
// (a.sample = 2) -- the tile kernel's epilogues for its modes 0, 6 and 7; 3 = a dense layer with K split over
// gridDim.y workgroups per tile: the fp32 partial tile goes to a.partial[ks][row][col] (the tile kernel's mode 5);
// 4, 5, 6 = 0, 1, 2 with the sums in levels, for a step of up to 64 sequences; 7 = the gradient of the loss with respect to the logits (the
// tile kernel's mode 3).
// What a workgroup's tile is cut from: weight tile vt of W (n_valid rows), all `rows` hidden rows at H, which are rows row0 ... of the call; its
// columns start at col0, its part is `part`.
struct MidTile {
  const void *W, *H;
  int vt, n_valid, rows, row0, col0, part;
  void* out;                               // SMODE 7
  int ldo;
};

// The gradient of the loss with respect to the logits of one finished tile (LogitsArgs, probability mode): four columns of a row at a time.
template <int NJV>
__device__ __forceinline__ void store_prob_tile(const f32x16 (&acc)[1][NJV], const LogitsArgs& a, const MidTile& t, int col_base) {
  const int lane31 = threadIdx.x & 31;
#pragma unroll
  for (int j = 0; j < NJV; ++j) {
    const int r = j * 32 + lane31;
    if (r >= t.rows) continue;
    const int row = t.row0 + r;
    const float lse = a.lse[row], g = a.row_grad[row];
    const int tgt = a.targets[row] - t.col0;
    uint16_t* out = reinterpret_cast<uint16_t*>(t.out) + (size_t)row * t.ldo;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = col_base + q * 8;
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p = __expf(read_acc(acc[0][j][q * 4 + e]) - lse) - (col + e == tgt ? 1.f : 0.f);
        x[e] = col + e < t.n_valid ? g * p : 0.f;
      }
      if (col < t.ldo)                     // (a multiple of 64)
        *reinterpret_cast<uint2*>(out + col) = uint2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
    }
  }
}

template <int NJV, int SMODE, int WAVES>
__device__ __forceinline__ void mid_tile(const LogitsArgs& a, const MidTile& t, unsigned char* lds) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  constexpr int STAGES = mid_stages(NJV, WAVES), RING = mid_ring(NJV, WAVES), TILE = 32 * WAVES;
  constexpr int STAGE = 32 * NJV * M_SLAB, STAGE_BYTES = STAGES * STAGE;
  constexpr int W_SLAB = 32 * M_SLAB;                      // a wave's weights of one slab
  const int vt = t.vt;                                     // weight tile (and one row tile: a call has at most M_HT rows)
  // SMODE 3 (a dense layer's partial sums): the rows that exist may be known on the device only, and blockIdx.y is
  // the part of K this workgroup takes (slabs [ks * slabs_per_part, ...))
  const int r_end = (SMODE == 3 && a.rows_dev) ? min(t.rows, *a.rows_dev) : t.rows;
  if (r_end <= 0) return;                                  // (the whole workgroup)
  const int nr = min(32 * NJV, r_end);                     // valid hidden rows
  const int n_valid = t.n_valid;
  const int v0 = vt * TILE;
  const size_t row_bytes = (size_t)a.d * 2;
  const int ks = SMODE == 3 ? (int)blockIdx.y : 0;
  const int slab0 = SMODE == 3 ? ks * a.slabs_per_part : 0;
  const int n_slabs = SMODE == 3 ? min(a.slabs_per_part, (int)(row_bytes / M_SLAB) - slab0) : (int)(row_bytes / M_SLAB);

  // The tiles walk K in the same order but start at different slabs (tile t at slab t mod n_slabs, wrapping round):
  // at any moment the workgroups in flight ask for different 128-byte columns of their weight rows, not all for
  // the same one, which would keep landing on the same few memory channels (rows are a power of two apart).
  const int rot = vt % n_slabs;
  auto slab_at = [&](int s) {                              // step -> slab
    const int x = s + rot;
    return slab0 + (x >= n_slabs ? x - n_slabs : x);
  };
  // weights through the wave's own ring: its 32 rows in four requests of 8 whole lines, laid out as the hidden rows are
  const unsigned char* Wt = reinterpret_cast<const unsigned char*>(t.W) + (size_t)v0 * row_bytes;
  uint32_t wsrc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = wave * 32 + i * 8 + (lane >> 3);
    wsrc[i] = (uint32_t)(min(row, n_valid - 1 - v0) * (int)row_bytes + (((lane & 7) ^ ((row >> 1) & 7)) << 4));
  }
  const uint32_t ring0 = lds_offset_of(lds) + (uint32_t)(STAGE_BYTES + wave * (RING * W_SLAB));
  auto issue_w = [&](int slab, int slot) {
    const unsigned char* p = Wt + (size_t)slab_at(slab) * M_SLAB;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t to = ring0 + (uint32_t)(slot * W_SLAB + i * 1024);
      if (a.once)
        load16_to_lds_once(p, wsrc[i], to);
      else
        load16_to_lds(p, wsrc[i], to);
    }
  };
  // hidden rows: the 4 NJV groups of 8 rows of a slab are dealt to the waves, group g = i * WAVES + wave for the
  // wave's i-th request; lane l moves, for row g * 8 + (l >> 3), the chunk that lands at position l & 7 of the row's
  // 128 LDS bytes: chunk (l & 7) ^ ((row >> 1) & 7).  Rows past the last valid one read the last valid one.
  constexpr int HL = (4 * NJV) / WAVES;                    // requests per wave and slab
  static_assert(HL * WAVES == 4 * NJV, "whole groups per wave");
  const unsigned char* Ht = reinterpret_cast<const unsigned char*>(t.H);
  const uint32_t lds_base = lds_offset_of(lds);
  uint32_t hsrc[HL];
#pragma unroll
  for (int i = 0; i < HL; ++i) {
    const int row = (i * WAVES + wave) * 8 + (lane >> 3);
    hsrc[i] = (uint32_t)(min(row, nr - 1) * (int)row_bytes + (((lane & 7) ^ ((row >> 1) & 7)) << 4));
  }
  auto issue_h = [&](int slab, int stage) {
    const unsigned char* p = Ht + (size_t)slab_at(slab) * M_SLAB;
#pragma unroll
    for (int i = 0; i < HL; ++i)
      load16_to_lds(p, hsrc[i], lds_base + (uint32_t)(stage * STAGE + (i * WAVES + wave) * 1024));
  };
  // operand reads: block j, row lane & 31, logical chunk 2 q + half
  const int sw = (lane >> 1) & 7;
  const int offB = (lane & 31) * M_SLAB;

  f32x16 acc[1][NJV];
#pragma unroll
  for (int j = 0; j < NJV; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][j][v] = 0.f;

  // A decode step of up to 64 sequences: the logits are added up in three levels: two slabs (8 MFMAs) in the accumulators,
  // sixteen slabs, all.  One accumulator over all of K rounds every step at the
  // size of the whole sum: d = 4096, relative error of the maxima 2.7e-7 to 3.3e-7; in two levels 5.7e-8 to 8.0e-8, in
  // three 4.4e-8 to 5.2e-8; the decode kernel's base units, which such a step ran on before and which add up 128 elements at a
  // time, 4.5e-8 to 4.9e-8.  (Calls with a few rows per sequence keep the one accumulator.  Hyper tiles, 66 to 192 rows of one or two sequences, d = 3072 to
  // 4096: 2.7e-7 to 3.6e-7 of the maxima; the tile kernel, which had them before, 2.5e-7 to 3.6e-7, the means over 18 shapes alike.)
  constexpr bool LEVELS = SMODE >= 4 && SMODE <= 6;
  f32x16 total[NJV], top[NJV];
  if (LEVELS) {
#pragma unroll
    for (int j = 0; j < NJV; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) total[j][v] = top[j][v] = 0.f;
  }
  auto third_level = [&]() {
#pragma unroll
    for (int j = 0; j < NJV; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        top[j][v] += total[j][v];
        total[j][v] = 0.f;
      }
  };
  auto next_level = [&]() {
#pragma unroll
    for (int j = 0; j < NJV; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        total[j][v] += acc[0][j][v];
        acc[0][j][v] = 0.f;
      }
  };

  auto compute = [&](const uint4 (&w)[4], int stage) {
    const unsigned char* Bs = lds + stage * STAGE + offB;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int pos = ((2 * q + half) ^ sw) << 4;
#pragma unroll
      for (int j = 0; j < NJV; ++j) {
        const uint4 b = *reinterpret_cast<const uint4*>(Bs + j * 32 * M_SLAB + pos);
        acc[0][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[q]),
                                                            __builtin_bit_cast(bf16x8, b), acc[0][j], 0, 0, 0);
      }
    }
  };

  // One step = one slab: on entry to step s the hidden rows of slab s are in stage s % STAGES for all, and its weights in the
  // wave's ring slot s % RING.  Requested during the step: the hidden rows of slab s + STAGES - 1 (HL requests), then the
  // weights of slab s + RING - 1 (4), both into what step s - 1 has read.  At its end slab s + 1 must have landed: KEEP
  // requests come behind the later of its two.  The last steps request nothing that does not exist, and wait for all.
  constexpr int BEHIND_H = 4 + (STAGES - 2) * (HL + 4), BEHIND_W = (RING - 2) * (HL + 4);
  constexpr int KEEP = BEHIND_H < BEHIND_W ? BEHIND_H : BEHIND_W;
  static_assert(KEEP < 64, "");
  int stage = 0, slot = 0;
  auto step_compute = [&]() {
    const unsigned char* As = lds + STAGE_BYTES + wave * (RING * W_SLAB) + slot * W_SLAB + offB;
    uint4 w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = *reinterpret_cast<const uint4*>(As + (((2 * q + half) ^ sw) << 4));
    compute(w, stage);
  };
  auto next_step = [&]() {
    __syncthreads();
    stage = stage == STAGES - 1 ? 0 : stage + 1;
    slot = slot == RING - 1 ? 0 : slot + 1;
  };
#pragma unroll
  for (int u = 0; u < (RING > STAGES ? RING : STAGES) - 1; ++u) {
    if (u < STAGES - 1 && u < n_slabs) issue_h(u, u);
    if (u < RING - 1 && u < n_slabs) issue_w(u, u);
  }
  if (n_slabs >= RING - 1)
    wait_loads<(STAGES - 2) * HL + 4 * (RING - 2)>();
  else
    wait_loads<0>();
  __syncthreads();
  int s = 0;
  for (; s + RING - 1 < n_slabs; ++s) {
    issue_h(s + STAGES - 1, stage == 0 ? STAGES - 1 : stage - 1);
    issue_w(s + RING - 1, slot == 0 ? RING - 1 : slot - 1);
    step_compute();
    if (LEVELS && (s & 1)) next_level();
    if (LEVELS && (s & 15) == 15) third_level();
    wait_loads<KEEP>();
    next_step();
  }
  for (; s < n_slabs; ++s) {
    if (s + STAGES - 1 < n_slabs) issue_h(s + STAGES - 1, stage == 0 ? STAGES - 1 : stage - 1);
    step_compute();
    if (LEVELS && (s & 1)) next_level();
    if (LEVELS && (s & 15) == 15) third_level();
    wait_loads<0>();
    next_step();
  }
  // (the last step ended with a wait for all requests and a barrier: the stages and rings are free)
  if (LEVELS) {
    next_level();
    third_level();
#pragma unroll
    for (int j = 0; j < NJV; ++j) acc[0][j] = top[j];
  }

  // ---- fold the tile, then one triple (and draw) per hidden row --------------------------------------------
  Triple run[NJV];
  Draw draw[NJV];
#pragma unroll
  for (int j = 0; j < NJV; ++j) {
    run[j] = empty_triple();
    draw[j] = empty_draw();
  }
  const int col_base = v0 + wave * 32 + half * 4;
  if (SMODE == 3) {
    // a dense layer's K part: the fp32 tile as it is; linear_sum_kernel adds the parts and runs the layer's epilogue
    store_partial_tile<1, NJV>(acc, a.partial + (size_t)ks * a.rows * a.ldo, a.ldo, 0, r_end, col_base, n_valid);
    return;
  }
  if (SMODE == 7) {
    store_prob_tile<NJV>(acc, a, t, col_base);
    return;
  }
  if (SMODE == 1 || SMODE == 5)
    fold_tile_sample<1, NJV>(acc, run, draw, a, 0, col_base, n_valid);
  else if (SMODE == 2 || SMODE == 6)
    fold_tile_store<1, NJV>(acc, run, a, 0, r_end, col_base, n_valid);
  else
    fold_tile<1, NJV>(acc, run, col_base, t.col0, n_valid, v0 + TILE > n_valid);
#pragma unroll
  for (int j = 0; j < NJV; ++j) {                          // lanes l and l + 32 hold the same hidden row
    Triple o;
    o.m = __shfl_xor(run[j].m, 32);
    o.s = __shfl_xor(run[j].s, 32);
    o.i = __shfl_xor(run[j].i, 32);
    merge_triple(run[j], o);
    if (SMODE == 1 || SMODE == 5) {
      Draw od;
      od.v = __shfl_xor(draw[j].v, 32);
      od.l = __shfl_xor(draw[j].l, 32);
      od.i = __shfl_xor(draw[j].i, 32);
      merge_draw(draw[j], od);
    }
  }
  Triple* xch = reinterpret_cast<Triple*>(lds);            // [wave][hidden row of the tile]
  Draw* xdr = reinterpret_cast<Draw*>(xch + WAVES * M_HT);
  if (lane < 32) {
#pragma unroll
    for (int j = 0; j < NJV; ++j) {
      xch[wave * M_HT + j * 32 + lane] = run[j];
      if (SMODE == 1 || SMODE == 5) xdr[wave * M_HT + j * 32 + lane] = draw[j];
    }
  }
  __syncthreads();
  if (tid < nr) {
    Triple tr = xch[tid];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) merge_triple(tr, xch[w * M_HT + tid]);
    const size_t p = (size_t)(t.row0 + tid) * a.n_parts + t.part;
    a.part_m[p] = tr.m;
    a.part_s[p] = tr.s;
    if (SMODE == 1 || SMODE == 5) {
      Draw dw = xdr[tid];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) merge_draw(dw, xdr[w * M_HT + tid]);
      a.part_v[p] = dw.v;
      a.part_l[p] = dw.l;
      a.part_i[p] = dw.i;
    } else {
      a.part_i[p] = tr.i;
    }
  }
}

template <int NJV, int SMODE, int WAVES = M_WAVES>
__global__ void __launch_bounds__(64 * WAVES) logits_mid_kernel(LogitsArgs a) {
  extern __shared__ __align__(1024) unsigned char lds[];
  MidTile t = {a.W, a.H, (int)blockIdx.x, a.w_rows, a.rows, 0, a.col0, a.part0 + (int)blockIdx.x, a.out, a.ldo};
  if constexpr (SMODE == 0 || SMODE == 7) {
    // Workgroups behind the base part's tiles take the hyper part's (a.hyper): tile u of sequence b against that sequence's rows alone, the first
    // tile of every sequence first.  In a launch of its own on the tile kernel this part was one round of a few workgroups, 58-80
    // us: V = 32064, 1 x 72 rows 99 -> 43 us; V = 128256, 1 x 80 242 -> 179, 2 x 79 275 -> 230; V = 151936, 1 x 103 277 -> 220.
    if (a.hyper.n_work > 0 && (int)blockIdx.x >= a.n_vtiles) {
      const int id = (int)blockIdx.x - a.n_vtiles, u = id / a.hyper.n_seq, b = id - u * a.hyper.n_seq;
      t.W = reinterpret_cast<const unsigned char*>(a.hyper.W) + (size_t)b * a.hyper.cap * a.d * 2;
      t.H = reinterpret_cast<const unsigned char*>(a.H) + (size_t)b * a.rows_per_seq * a.d * 2;
      t.vt = u;
      t.n_valid = min(max(a.hyper.size[b], 0), a.hyper.cap);
      t.rows = a.rows_per_seq;
      t.row0 = b * a.rows_per_seq;
      t.col0 = a.hyper.col0;
      t.part = a.hyper.part0 + u;
      t.out = a.hyper.out;
      t.ldo = a.hyper.ldo;
      if (u * 32 * WAVES >= t.n_valid) {                   // entries that do not exist: empty triples
        if (SMODE == 0 && (int)threadIdx.x < t.rows) {     // (a thread per row)
          const size_t p = (size_t)(t.row0 + (int)threadIdx.x) * a.n_parts + t.part;
          a.part_m[p] = kNegInf;
          a.part_s[p] = 0.f;
          a.part_i[p] = kNoColumn;
        }
        return;
      }
    }
  }
  if constexpr (SMODE == 3 && NJV == 4) {
    // (the rows that exist may be half of those laid out: known here only)
    if ((a.rows_dev ? min(a.rows, *a.rows_dev) : a.rows) <= 64)
      mid_tile<2, SMODE, WAVES>(a, t, lds);
    else
      mid_tile<4, SMODE, WAVES>(a, t, lds);
  } else {
    mid_tile<NJV, SMODE, WAVES>(a, t, lds);
  }
}

}  // namespace

bool z2z_logits_mid_ok(const z2z_ctx* c, int rows) {
  return c->mid_ready && c->cfg.dtype == Z2Z_BF16 && c->cfg.d % 64 == 0 && rows >= 1 && rows <= M_MAX_ROWS;
}

// Columns of a part: 256, or 128 (workgroups of four waves) where that gives every tile a CU of its own and 256 would leave
// half of the CUs without one.  V = 32064, d = 3072 (126 tiles of 256), whole calls in us, 256 -> 128: 2 x 5 rows 88 -> 71, 8 x 8 82
// -> 63, 3 x 36 91 -> 74, 180 131 -> 117; steps of 17 sequences, 4096 entries each, 118 -> 105, 90 162 -> 146, a draw of 150 264 -> 247.
int z2z_logits_mid_columns(const z2z_ctx* c, int w_rows) {
  return (w_rows + M_WT - 1) / M_WT * 2 <= c->num_cu ? M_WT / 2 : M_WT;
}

template <int WAVES>
static void launch_mid(const LogitsArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)(a.n_vtiles + a.hyper.n_work)), block(64 * WAVES);
  const int blocks = a.rows <= 64 ? 2 : (a.rows <= 128 ? 4 : 6);
  if (a.row_grad) {
    if (blocks == 2)
      hipLaunchKernelGGL((logits_mid_kernel<2, 7, WAVES>), grid, block, mid_lds(2, WAVES), s, a);
    else if (blocks == 4)
      hipLaunchKernelGGL((logits_mid_kernel<4, 7, WAVES>), grid, block, mid_lds(4, WAVES), s, a);
    else
      hipLaunchKernelGGL((logits_mid_kernel<6, 7, WAVES>), grid, block, mid_lds(6, WAVES), s, a);
    return;
  }
  if (a.sample == 1) {
    if (blocks == 2)
      hipLaunchKernelGGL((logits_mid_kernel<2, 5, WAVES>), grid, block, mid_lds(2, WAVES), s, a);
    else if (blocks == 4)
      hipLaunchKernelGGL((logits_mid_kernel<4, 1, WAVES>), grid, block, mid_lds(4, WAVES), s, a);
    else
      hipLaunchKernelGGL((logits_mid_kernel<6, 1, WAVES>), grid, block, mid_lds(6, WAVES), s, a);
  } else if (a.sample == 2) {
    if (blocks == 2)
      hipLaunchKernelGGL((logits_mid_kernel<2, 6, WAVES>), grid, block, mid_lds(2, WAVES), s, a);
    else if (blocks == 4)
      hipLaunchKernelGGL((logits_mid_kernel<4, 2, WAVES>), grid, block, mid_lds(4, WAVES), s, a);
    else
      hipLaunchKernelGGL((logits_mid_kernel<6, 2, WAVES>), grid, block, mid_lds(6, WAVES), s, a);
  } else {
    if (blocks == 2 && a.rows_per_seq == 1)
      hipLaunchKernelGGL((logits_mid_kernel<2, 4, WAVES>), grid, block, mid_lds(2, WAVES), s, a);
    else if (blocks == 2)
      hipLaunchKernelGGL((logits_mid_kernel<2, 0, WAVES>), grid, block, mid_lds(2, WAVES), s, a);
    else if (blocks == 4)
      hipLaunchKernelGGL((logits_mid_kernel<4, 0, WAVES>), grid, block, mid_lds(4, WAVES), s, a);
    else
      hipLaunchKernelGGL((logits_mid_kernel<6, 0, WAVES>), grid, block, mid_lds(6, WAVES), s, a);
  }
}

// The base part of a call: one part per tile of z2z_logits_mid_columns weight rows.  a: H, rows, d, the part arrays, n_parts, part0
// filled by the caller; with a.sample = 1 or 2 also the generator words, inv_temperature and part_v / part_l or
// logits / ld, as for the tile kernel's sampling modes; a.once where the caller knows of more weights that the call reads.
int z2z_launch_logits_mid(z2z_ctx* c, LogitsArgs a, const void* W, int w_rows, int col0, hipStream_t s) {
  if (!z2z_logits_mid_ok(c, a.rows) || w_rows < 1) return Z2Z_EUNSUPPORTED;
  a.W = W;
  a.w_rows = w_rows;
  a.col0 = col0;
  const int columns = z2z_logits_mid_columns(c, w_rows);
  a.n_vtiles = (w_rows + columns - 1) / columns;
  a.once = a.once || (size_t)w_rows * a.d * sizeof(uint16_t) > kKeepBytes;
  c->n_launch[Z2Z_KERNEL_MID]++;
  if (a.hyper.n_work > 0 && (a.sample != 0 || (a.rows_per_seq <= 64 && !a.row_grad))) return Z2Z_EUNSUPPORTED;
  // (two workgroups of the 64-row build per weight tile for 65..128 rows, sharing the tile's weights through an
  // XCD's L2, measured slower than one of the 128-row build: 383 against 293 us at config 2's shape)
  // builds: 2, 4 or 6 blocks of 32 hidden rows; the sampling calls come with one row per sequence.  (8 blocks, up to 256
  // rows, measured level with the tile kernel when weights still went through registers: 650 against 645 us for a decode step of
  // 256 sequences.)
  if (columns == M_WT)
    launch_mid<M_WAVES>(a, s);
  else
    launch_mid<M_WAVES / 2>(a, s);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

// Parts of K per weight tile: the split (parts of at least four slabs, at most 16 parts) with the fewest slab steps
// on the busiest CU -- rounds of 256 workgroups x (slabs per part + 3 for filling and draining the pipeline); a
// split that puts a few workgroups into a second round costs a whole round.
int z2z_linear_mid_ksplit(int N, int K) {
  const int n_vt = (N + M_WT - 1) / M_WT, n_slabs = K / 64;
  int best = 1;
  long long best_cost = -1;
  for (int ks = 1; ks <= 16 && (ks == 1 || n_slabs / ks >= 4); ++ks) {
    const int per = (n_slabs + ks - 1) / ks;
    const int parts = (n_slabs + per - 1) / per;           // no empty parts
    const long long cost = (long long)((n_vt * parts + 255) / 256) * (per + 3);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = parts;
    }
  }
  return best;
}

// Dense layer out = act(A W^T + bias) + residual on R <= 128 rows (or fewer, *rows_dev): the weight-streaming kernel
// leaves ksplit fp32 partial tiles per weight tile in `partial` ([ksplit][R][N]); the caller sums them
// (linear_sum_kernel in dense.hip).  Returns the ksplit chosen through *ksplit_out.
int z2z_launch_linear_mid(z2z_ctx* c, const void* A, const void* W, int R, const int32_t* rows_dev, int N, int K,
                          bool once, float* partial, size_t partial_floats, int* ksplit_out, hipStream_t s) {
  if (!z2z_logits_mid_ok(c, R) || R > 128 || K % 64 != 0 || N < 1) return Z2Z_EUNSUPPORTED;
  const int n_vt = (N + M_WT - 1) / M_WT, n_slabs = K / 64;
  const int ksplit = z2z_linear_mid_ksplit(N, K);
  const int per = (n_slabs + ksplit - 1) / ksplit;
  if ((size_t)ksplit * R * N > partial_floats) return Z2Z_ELIMIT;
  LogitsArgs a;
  memset(&a, 0, sizeof(a));
  a.H = A;
  a.W = W;
  a.rows = R;
  a.d = K;
  a.w_rows = N;
  a.n_vtiles = n_vt;
  a.ldo = N;
  a.rows_dev = rows_dev;
  a.ksplit = ksplit;
  a.slabs_per_part = per;
  a.partial = partial;
  a.once = once ? 1 : 0;
  *ksplit_out = ksplit;
  c->n_launch[Z2Z_KERNEL_MID]++;
  const dim3 grid((unsigned)n_vt, (unsigned)ksplit), block(64 * M_WAVES);
  if (R <= 64)
    hipLaunchKernelGGL((logits_mid_kernel<2, 3>), grid, block, mid_lds(2, M_WAVES), s, a);
  else
    hipLaunchKernelGGL((logits_mid_kernel<4, 3>), grid, block, mid_lds(2, M_WAVES) > mid_lds(4, M_WAVES) ? mid_lds(2, M_WAVES) : mid_lds(4, M_WAVES), s, a);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

int z2z_logits_mid_tiles(int w_rows) { return (w_rows + M_WT - 1) / M_WT; }

int z2z_logits_mid_prepare(z2z_ctx* c) {
  if (c->lds_limit < M_LDS_MAX) return Z2Z_EUNSUPPORTED;
  const void* kernels[] = {reinterpret_cast<const void*>(logits_mid_kernel<2, 3>),
                           reinterpret_cast<const void*>(logits_mid_kernel<4, 3>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 7, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<4, 7, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<6, 7, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 7, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<4, 7, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<6, 7, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 0, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 4, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 5, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 6, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<4, 0, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<4, 1, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<4, 2, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<6, 0, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<6, 1, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<6, 2, M_WAVES>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 0, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 4, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 5, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<2, 6, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<4, 0, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<4, 1, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<4, 2, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<6, 0, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<6, 1, M_WAVES / 2>),
                           reinterpret_cast<const void*>(logits_mid_kernel<6, 2, M_WAVES / 2>)};
  for (const void* k : kernels)
    Z2Z_HIP_TRY(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, M_LDS_MAX));
  return Z2Z_OK;
}

// extended_logits, general tile kernel (any d that is a multiple of the 16-byte chunk, bf16 or fp32).
//
// Both operands are stored with the contraction index k contiguous, so a lane fetches 16 bytes of a row
// for each MFMA operand.  The vocabulary rows are the MFMA "A" operand and the hidden rows the "B"
// operand: in the 32x32 result block a lane then holds 16 vocabulary entries of ONE hidden row, so the
// running (max, sum-exp, argmax) of a row is kept in that lane's registers and crosses lanes only once
// per strip.  A workgroup owns one tile of hidden rows and sweeps a strip of vocabulary tiles.
// This is the fp32 path, and the fallback for shapes the fast bf16 kernel does not take.
//
// fp32 is bound by the matrix cores (v_mfma_f32_32x32x2_f32: 256 flop per CU and clock, 157 TFLOP/s).  A workgroup's loads,
// barriers and folds are covered by the others on its CU, so its tile is as small as keeps three of them there (48 KiB of LDS,
// at most 168 registers): 64 columns x 128 rows, whose LDS reads still take a fifth of the matrix instructions' time.  Smaller
// tiles also fill the last round of a CU better.  With 128 x 128, two per CU, two waves per SIMD kept the matrix cores 62 % busy.
// bf16 takes 128 x 128 but for the smallest calls (z2z_logits_general_columns).
// The instance that stores the logits is a kernel of its own (its store addresses and column tests cost the plain one
// registers), and operand rows are 32-bit offsets from one base address per tile.
// Both parts share a launch, the hyper part's few tiles first; an XCD walks consecutive row tiles of consecutive
// strips, so its L2 reads a weight strip once for all of them.
// Whole calls, fp32, 32000 columns and two codebooks, d = 256, 128 x 128 -> 64 x 128: 512 rows 106 -> 100 us, 1024 rows
// 170 -> 156 (17.6 GFLOP), 2048 rows 306 -> 291, 4096 rows 578 -> 563 (119 TFLOP/s).
#include "logits_common.h"

namespace {

using namespace z2z_logits;

// ------------------------------------------------------------------------------------------------
// Tile kernel, TV = 64 or 128 (vocabulary) x 128 (hidden rows) per workgroup, 4 waves of TV / 2 x 64, K slabs of
// 128 bytes per row.  LDS holds two buffers of (TV + 128) rows x 128 B; the 16-byte chunk c of row
// r sits at chunk (c ^ ((r >> 1) & 7)) so that the 16 rows a quarter-wave reads hit all 64 banks.
// T = bf16 bits (uint16_t) or float.
// ------------------------------------------------------------------------------------------------
constexpr int TR = 128;
constexpr int SLAB_BYTES = 128;
constexpr int B_BYTES = TR * SLAB_BYTES;      // the hidden rows of one slab in LDS (16 KiB)
constexpr int ROW_BLOCK = 8;                  // row tiles that an XCD walks together per strip

// per build (TV = 64 or 128 columns):
constexpr int weight_bytes(int tv) { return tv * SLAB_BYTES; }     // a tile's weight rows of one slab in LDS
constexpr int blocks_v(int tv) { return tv / 64; }                 // MFMA blocks of a wave along the vocabulary
constexpr int stage_rows(int tv) { return tv / 32; }               // weight rows that a thread stages
constexpr int per_cu(int tv) { return tv == 64 ? 3 : 2; }          // workgroups that a CU's LDS and registers hold

struct GeneralArgs {
  LogitsArgs base, hyper;
  int32_t hyper_grid;   // workgroups of the hyper part (the first ones), a multiple of 8
};

// The wave's NI x 2 blocks of 32 x 32 advance by one 16-byte chunk of K per lane.
template <typename T, int NI>
__device__ __forceinline__ void mfma_block(const f32x4 (&fa)[NI], const f32x4 (&fb)[2], f32x16 (&acc)[NI][2]) {
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[i]), __builtin_bit_cast(bf16x8, fb[j]),
                                                            acc[i][j], 0, 0, 0);
  } else {
    // a 16-byte chunk holds 4 consecutive k; lanes 0-31 and 32-63 hold different chunks, and the
    // pairing of k between the two operands is the same, so any order of the 4 steps is a valid sum
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e],
                                                           acc[i][j], 0, 0, 0);
  }
}

// Waves of the workgroup meet.  (Not __syncthreads, which would wait for the next slab's loads as well.)
__device__ __forceinline__ void meet() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Fold the wave's 32 NI x 64 logits into the running triples (and store them).  TAIL: the tile has columns that do not exist.
template <bool STORE, bool TAIL, int NI>
__device__ __forceinline__ void fold_general(const f32x16 (&acc)[NI][2], Triple (&run)[2], const LogitsArgs& a, int row0,
                                             int r_end, int col_base, int n_valid) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int hrow = row0 + j * 32;
    float* out = STORE ? a.logits + (size_t)min(hrow, r_end - 1) * a.ld + a.col0 : nullptr;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      float x[16];
      float gmax = kNegInf;
      int targ = 0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int col = col_base + i * 32 + (v >> 2) * 8 + (v & 3);
        x[v] = acc[i][j][v];
        if (TAIL && col >= n_valid) x[v] = kNegInf;
        if (x[v] > gmax) {
          gmax = x[v];
          targ = v;
        }
        if (STORE && col < n_valid && hrow < r_end) out[col] = x[v];
      }
      if (gmax > run[j].m) {
        run[j].s = (run[j].m == kNegInf) ? 0.f : run[j].s * __expf(run[j].m - gmax);
        run[j].m = gmax;
        run[j].i = a.col0 + col_base + i * 32 + (targ >> 2) * 8 + (targ & 3);
      }
      if (col_base + i * 32 < n_valid) {
        // (where nothing has been above -inf yet, columns that do not exist add 0 and a hidden row's NaN stay NaN)
        const float m = run[j].m == kNegInf ? 0.f : run[j].m;
        float add = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) add += __expf(x[v] - m);
        run[j].s += add;
      }
    }
  }
}

template <typename T, int TV, bool STORE>
__global__ void __launch_bounds__(256, per_cu(TV)) logits_general_kernel(GeneralArgs g) {
  constexpr int A_BYTES = weight_bytes(TV), NI = blocks_v(TV), NA = stage_rows(TV);
  __shared__ __align__(16) unsigned char lds[2 * (A_BYTES + B_BYTES)];   // [buf][A|B]
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wv = wave & 1;    // which half of the tile's vocabulary rows
  const int wr = wave >> 1;   // which 64 hidden rows of the tile

  // ---- which part, rows, W, strip -----------------------------------------------------------------
  const bool hyper = (int)blockIdx.x < g.hyper_grid;
  const LogitsArgs& a = hyper ? g.hyper : g.base;
  // workgroup ids go round-robin over the XCDs: XCD x takes the x-th eighth of the part's tiles, whose order is
  // row tile in its block, strip, row block, sequence
  const int id = hyper ? (int)blockIdx.x : (int)blockIdx.x - g.hyper_grid;
  const int work = (id & 7) * ((a.n_work + 7) >> 3) + (id >> 3);
  if ((id >> 3) >= (a.n_work + 7) >> 3 || work >= a.n_work) return;
  const int per_seq = a.row_tiles * a.n_strips;
  const int b = work / per_seq;                     // (the base part has one "sequence")
  const int in_seq = work - b * per_seq;
  const int blk = in_seq / (ROW_BLOCK * a.n_strips);
  const int in_blk = in_seq - blk * ROW_BLOCK * a.n_strips;
  const int blk_tiles = min(ROW_BLOCK, a.row_tiles - blk * ROW_BLOCK);
  const int st = in_blk / blk_tiles;
  const int rt = blk * ROW_BLOCK + (in_blk - st * blk_tiles);
  const unsigned char* Wp = reinterpret_cast<const unsigned char*>(a.W);
  const uint32_t row_bytes = (uint32_t)a.d * (uint32_t)sizeof(T);
  int r0, r_end, n_valid;
  if (hyper) {
    r0 = b * a.rows_per_seq + rt * TR;
    r_end = (b + 1) * a.rows_per_seq;
    n_valid = min(max(a.size[b], 0), a.w_rows);
    Wp += (size_t)b * a.w_rows * row_bytes;
  } else {
    r0 = rt * TR;
    r_end = a.rows;
    n_valid = a.w_rows;
  }
  const unsigned char* Hp = reinterpret_cast<const unsigned char*>(a.H) + (size_t)r0 * row_bytes;
  const int vt0 = st * a.strip;
  const int vt1 = min(vt0 + a.strip, a.n_vtiles);

  Triple run[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) run[j] = empty_triple();

  // global -> LDS staging: thread t moves chunk t & 7 of rows (t >> 3) + 32 i of each operand tile
  const int n_slabs = (int)((row_bytes + SLAB_BYTES - 1) / SLAB_BYTES);
  const uint32_t my_k = (uint32_t)(tid & 7) * 16;
  uint32_t off_b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) off_b[i] = (uint32_t)min((tid >> 3) + 32 * i, r_end - 1 - r0) * row_bytes + my_k;
  // (the swizzle of row + 32 i is the row's own)
  const int lds_at = (tid >> 3) * SLAB_BYTES + (((tid & 7) ^ ((tid >> 4) & 7)) << 4);
  // operand reads: row = TV / 2 wv (weights) or 64 wr (hidden rows) + 32 i + (lane & 31), chunk 2 q + (lane >> 5)
  const int rd_a = (wv * (TV / 2) + (lane & 31)) * SLAB_BYTES;
  const int rd_b = A_BYTES + (wr * 64 + (lane & 31)) * SLAB_BYTES;
  const int swz = (lane >> 1) & 7;

  for (int vt = vt0; vt < vt1; ++vt) {
    const int v0 = vt * TV;
    if (v0 >= n_valid) break;
    const unsigned char* Wt = Wp + (size_t)v0 * row_bytes;
    uint32_t off_a[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) off_a[i] = (uint32_t)min((tid >> 3) + 32 * i, n_valid - 1 - v0) * row_bytes + my_k;

    f32x16 acc[NI][2];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    f32x4 stage_a[NA], stage_b[4];
    auto fetch = [&](int slab) {
      const uint32_t kb = (uint32_t)slab * SLAB_BYTES;
      const bool in_k = kb + my_k < row_bytes;       // (past the end of a row: zeros add nothing)
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i < NA) stage_a[i] = in_k ? *reinterpret_cast<const f32x4*>(Wt + (off_a[i] + kb)) : z;
        stage_b[i] = in_k ? *reinterpret_cast<const f32x4*>(Hp + (off_b[i] + kb)) : z;
      }
    };
    auto stash = [&](int buf) {
      unsigned char* A = lds + buf * (A_BYTES + B_BYTES) + lds_at;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i < NA) *reinterpret_cast<f32x4*>(A + i * 32 * SLAB_BYTES) = stage_a[i];
        *reinterpret_cast<f32x4*>(A + A_BYTES + i * 32 * SLAB_BYTES) = stage_b[i];
      }
    };

    // Fragments are read a quarter slab ahead; a slab's successor is written to LDS under its second quarter and its own last
    // fragments are read ahead of the barrier, so that what stands between two slabs is the barrier alone.
    f32x4 fa[2][NI], fb[2][2];
    auto read = [&](f32x4 (&ra)[NI], f32x4 (&rb)[2], int buf, int q) {
      const unsigned char* L = lds + buf * (A_BYTES + B_BYTES) + (((2 * q + (lane >> 5)) ^ swz) << 4);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        ra[i] = *reinterpret_cast<const f32x4*>(L + rd_a + i * 32 * SLAB_BYTES);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        rb[i] = *reinterpret_cast<const f32x4*>(L + rd_b + i * 32 * SLAB_BYTES);
      }
    };
    fetch(0);
    __syncthreads();          // the previous tile's readers are done with buffer 0
    stash(0);
    if (n_slabs > 1) fetch(1);
    meet();
    read(fa[0], fb[0], 0, 0);
    for (int slab = 0; slab < n_slabs; ++slab) {
      const int buf = slab & 1;
      const bool more = slab + 1 < n_slabs;
      read(fa[1], fb[1], buf, 1);
      mfma_block<T, NI>(fa[0], fb[0], acc);
      read(fa[0], fb[0], buf, 2);
      if (more) {
        stash(buf ^ 1);       // (its last readers had their fragments ahead of the barrier before)
        if (slab + 2 < n_slabs) fetch(slab + 2);
      }
      mfma_block<T, NI>(fa[1], fb[1], acc);
      read(fa[1], fb[1], buf, 3);
      mfma_block<T, NI>(fa[0], fb[0], acc);
      if (more) {
        meet();
        read(fa[0], fb[0], buf ^ 1, 0);
      }
      mfma_block<T, NI>(fa[1], fb[1], acc);
    }

    // ---- epilogue of this tile: fold its logits into the running triples ----------------------
    const int col_base = v0 + wv * (TV / 2) + (lane >> 5) * 4;
    const int row0 = r0 + wr * 64 + (lane & 31);
    if (v0 + TV <= n_valid)
      fold_general<STORE, false>(acc, run, a, row0, r_end, col_base, n_valid);
    else
      fold_general<STORE, true>(acc, run, a, row0, r_end, col_base, n_valid);
  }

  // ---- end of strip: lanes l and l+32 hold the same hidden row; then the two vocabulary halves ---
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    Triple o;
    o.m = __shfl_xor(run[j].m, 32);
    o.s = __shfl_xor(run[j].s, 32);
    o.i = __shfl_xor(run[j].i, 32);
    merge_triple(run[j], o);
  }
  __syncthreads();            // all waves are done reading the operand tiles
  Triple* xch = reinterpret_cast<Triple*>(lds);   // [2 row halves][64 rows]
  if (wv == 1 && lane < 32) {
    xch[wr * 64 + lane] = run[0];
    xch[wr * 64 + 32 + lane] = run[1];
  }
  __syncthreads();
  if (wv == 0 && lane < 32) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      merge_triple(run[j], xch[wr * 64 + j * 32 + lane]);
      const int hrow = r0 + wr * 64 + j * 32 + lane;
      if (hrow < r_end) {
        const size_t p = (size_t)hrow * a.n_parts + a.part0 + st;
        a.part_m[p] = run[j].m;
        a.part_s[p] = run[j].s;
        a.part_i[p] = run[j].i;
      }
    }
  }
}

}  // namespace

// Columns of a tile, by the workgroups that tiles of 64 columns would make (128 rows each, base and hyper).  fp32: 64.  bf16 is bound
// by LDS reads and epilogues more than by its matrix instructions: 128, whose fragments serve twice the products, unless tiles of
// 64 fill no more than one round of the CUs' three.  Whole calls in us, bf16, 64 / 128 columns: with the logits stored 256 rows x
// 128256, d = 4096 526 / 451; 700 x 151936, d = 3584 1480 / 1290; 128 x 50257, d = 768 52.0 / 46.8 (786 tiles); 64 x 32000, d = 1024
// 34.6 / 37.3 (500); picks alone, d = 1000, 2048 x 32000 236 / 196, 300 rows 56.0 / 51.3, 64 rows 27.7 / 29.8; d = 520, 100 x 5000 14.0 / 16.4.
int z2z_logits_general_columns(bool bf16, long long tiles_of_64) { return bf16 && tiles_of_64 > 3 * 256 ? 128 : 64; }

// One launch for both parts, tiles of `columns` columns; hyper == nullptr: no hyper vocabulary.
int z2z_launch_logits_general(bool bf16, int columns, const LogitsArgs& base, const LogitsArgs* hyper, hipStream_t s) {
  GeneralArgs g;
  g.base = base;
  g.hyper = hyper ? *hyper : base;
  g.hyper_grid = hyper ? (hyper->n_work + 7) / 8 * 8 : 0;
  const dim3 grid((unsigned)g.hyper_grid + (unsigned)((base.n_work + 7) / 8 * 8)), block(256);
  const bool store = base.logits != nullptr;
  if (bf16 && columns == 128 && store)
    hipLaunchKernelGGL((logits_general_kernel<uint16_t, 128, true>), grid, block, 0, s, g);
  else if (bf16 && columns == 128)
    hipLaunchKernelGGL((logits_general_kernel<uint16_t, 128, false>), grid, block, 0, s, g);
  else if (bf16 && store)
    hipLaunchKernelGGL((logits_general_kernel<uint16_t, 64, true>), grid, block, 0, s, g);
  else if (bf16)
    hipLaunchKernelGGL((logits_general_kernel<uint16_t, 64, false>), grid, block, 0, s, g);
  else if (store)
    hipLaunchKernelGGL((logits_general_kernel<float, 64, true>), grid, block, 0, s, g);
  else
    hipLaunchKernelGGL((logits_general_kernel<float, 64, false>), grid, block, 0, s, g);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

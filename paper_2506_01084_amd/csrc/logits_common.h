// Shared pieces of the extended_logits kernels (HIP, gfx950).
//
// Joint softmax over the base and hyper vocabularies (zip2zip paper, section 2.3, steps 7-9) reduced on
// the fly: every kernel folds the logits it produces into per-row triples (max, sum of exp(x - max),
// column of the max) and leaves one triple per (part, row); a small kernel merges the parts.
#pragma once

#include "z2z_internal.h"

#include <math.h>

namespace z2z_logits {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr float kNegInf = -INFINITY;
constexpr int kNoColumn = 0x7FFFFFFF;

struct Triple {
  float m;   // running maximum
  float s;   // sum of exp(x - m)
  int i;     // column of the maximum
};

__device__ __forceinline__ Triple empty_triple() {
  Triple t;
  t.m = kNegInf;
  t.s = 0.f;
  t.i = kNoColumn;
  return t;
}

// Merge b into a; equal maxima keep the lower column.
__device__ __forceinline__ void merge_triple(Triple& a, const Triple& b) {
  const bool b_wins = (b.m > a.m) || (b.m == a.m && b.i < a.i);
  const float hi = b_wins ? b.m : a.m;
  const float lo = b_wins ? a.m : b.m;
  const float s_hi = b_wins ? b.s : a.s;
  const float s_lo = b_wins ? a.s : b.s;
  const float scale = (lo == kNegInf) ? 0.f : __expf(lo - hi);
  a.s = s_hi + s_lo * scale;
  a.m = hi;
  a.i = b_wins ? b.i : a.i;
}

// The running best of a Gumbel-max draw.
struct Draw {
  float v;   // largest perturbed value so far
  float l;   // logit / T at that column
  int i;     // that column
};

__device__ __forceinline__ Draw empty_draw() {
  Draw d;
  d.v = kNegInf;
  d.l = 0.f;
  d.i = kNoColumn;
  return d;
}

__device__ __forceinline__ void merge_draw(Draw& a, const Draw& b) {
  if (b.v > a.v || (b.v == a.v && b.i < a.i)) a = b;
}

// One accumulator element, AGPR -> VGPR.  Spelled as an instruction so that the accumulators stay in
// the accumulation registers and are fetched block by block: left to itself the compiler copies the whole
// accumulator tile into VGPRs at the end of the K loop, and what that displaces is spilled inside the loop.
__device__ __forceinline__ float read_acc(float in_agpr) {
  float x;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(in_agpr));
  return x;
}

// Largest of three in one instruction.  (Spelled as an instruction: on values that come out of read_acc the
// compiler knows nothing about, fmaxf costs a quieting instruction per operand.)
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Fold one finished accumulator tile into the running triples.  acc[i][j] is a 32x32 MFMA result block:
// register v of this lane is the logit of hidden row (j, lane & 31) and vocabulary column
// col_base + i * 32 + (v >> 2) * 8 + (v & 3), where col_base already holds the tile origin, the wave's
// offset and (lane >> 5) * 4.  Columns at and beyond n_valid do not exist (read as -inf; TAIL = false is the
// instance for tiles that lie wholly below n_valid, which is all but the last tile of a matrix: it carries no
// column tests at all).  The fold goes block by block (16 values live at a time, the accumulators are only
// read), in increasing column order per lane, so strict comparisons keep the lowest column among equal
// maxima.  The running sum is kept against the running maximum in base-2 units: exp(x - m) is one
// multiply-add and one hardware exponential per logit.
template <int NI, int NJ, bool TAIL>
__device__ __forceinline__ void fold_tile_impl(const f32x16 (&acc)[NI][NJ], Triple (&run)[NJ], int col_base, int col0,
                                               int n_valid) {
  constexpr float kLog2e = 1.4426950408889634f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      float x[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        x[v] = read_acc(acc[i][j][v]);
        if (TAIL && col_base + i * 32 + (v >> 2) * 8 + (v & 3) >= n_valid) x[v] = kNegInf;
      }
      float gmax = max3(x[0], x[1], x[2]);
#pragma unroll
      for (int v = 3; v < 15; v += 2) gmax = max3(gmax, x[v], x[v + 1]);
      gmax = max3(gmax, x[15], x[15]);
      if (gmax > run[j].m) {
        int targ = 15;
#pragma unroll
        for (int v = 14; v >= 0; --v) targ = (x[v] == gmax) ? v : targ;
        run[j].s = (run[j].m == kNegInf) ? 0.f : run[j].s * __expf(run[j].m - gmax);
        run[j].m = gmax;
        run[j].i = col0 + col_base + i * 32 + (targ >> 2) * 8 + (targ & 3);
      }
      if (!TAIL || col_base + i * 32 < n_valid) {
        // (where nothing has been above -inf yet, columns that do not exist add 0 and a hidden row's NaN stay NaN; without a tail
        // every logit is finite or NaN, and so is the sum)
        const float m2 = TAIL && run[j].m == kNegInf ? 0.f : -run[j].m * kLog2e;
        float add0 = 0.f, add1 = 0.f;
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
          add0 += __builtin_amdgcn_exp2f(fmaf(x[v], kLog2e, m2));
          add1 += __builtin_amdgcn_exp2f(fmaf(x[v + 1], kLog2e, m2));
        }
        run[j].s += add0 + add1;
      }
    }
  }
}

template <int NI, int NJ>
__device__ __forceinline__ void fold_tile(const f32x16 (&acc)[NI][NJ], Triple (&run)[NJ], int col_base, int col0,
                                          int n_valid, bool tail) {
  if (tail)
    fold_tile_impl<NI, NJ, true>(acc, run, col_base, col0, n_valid);
  else
    fold_tile_impl<NI, NJ, false>(acc, run, col_base, col0, n_valid);
}

__device__ __forceinline__ uint32_t bf16_bits_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

// Two values, rounded to nearest even in one instruction; a NaN stays one, whatever its bits (the sum above carries 0xFFFFFFFF over to 0).
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// GELU(x) = x * Phi(x) with the exact (erf) Phi.  erf by the rational approximation 7.1.26 of Abramowitz and
// Stegun, erf(z) = 1 - (a1 t + ... + a5 t^5) exp(-z^2), t = 1 / (1 + p z), z >= 0: absolute error below
// 1.5e-7, far inside the bf16 rounding of the result, at a third of the instructions of the library erff (the
// epilogue of a dense layer evaluates it 65536 times per tile with the matrix cores waiting).
__device__ __forceinline__ float gelu_erf(float x) {
  const float z = fabsf(x) * 0.70710678f;
  const float t = __frcp_rn(fmaf(0.3275911f, z, 1.0f));
  const float poly = t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f),
                              0.254829592f);
  const float erf_abs = 1.0f - poly * __expf(-z * z);
  const float phi = 0.5f * (1.0f + copysignf(erf_abs, x));
  return x * phi;
}

// A dense layer's epilogue on 4 columns of a row, whose first is element `at` of the output and the residual: out = act(x + bias) + residual.
__device__ __forceinline__ void finish_linear(float4 x, const float4& bias, int act, const void* residual, void* out, bool stream_f32, size_t at) {
  x.x += bias.x;
  x.y += bias.y;
  x.z += bias.z;
  x.w += bias.w;
  if (act == 1) {
    x.x = gelu_erf(x.x);
    x.y = gelu_erf(x.y);
    x.z = gelu_erf(x.z);
    x.w = gelu_erf(x.w);
  }
  if (stream_f32) {                                  // fp32 residual and output: no rounding
    if (residual) {
      const float4 rv = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(residual) + at);
      x.x += rv.x;
      x.y += rv.y;
      x.z += rv.z;
      x.w += rv.w;
    }
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + at) = x;
    return;
  }
  if (residual) {
    const uint2 rv = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(residual) + at);
    x.x += __uint_as_float(rv.x << 16);
    x.y += __uint_as_float(rv.x & 0xFFFF0000u);
    x.z += __uint_as_float(rv.y << 16);
    x.w += __uint_as_float(rv.y & 0xFFFF0000u);
  }
  *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out) + at) = uint2{pack_bf16(x.x, x.y), pack_bf16(x.z, x.w)};
}

// ---- the counter-based generator of the sampling kernels: Philox4x32-10 (Salmon et al., SC'11) -------
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t hi0 = __umulhi(0xD2511F53u, c.x), lo0 = 0xD2511F53u * c.x;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c.z), lo1 = 0xCD9E8D57u * c.z;
    c = uint4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
  }
  return c;
}

// The Gumbel value -ln(-ln u) of one generator word, u = ((w >> 9) + 0.5) * 2^-23.  u and 1 - u are both
// exact in float.  e = -ln u has to be accurate relative to itself where it is small (u next to 1: the
// largest perturbations, the ones that win): there it is the series of -ln(1 - x); elsewhere the hardware
// logarithm's absolute error of ~1e-7 is relative 1e-5 at worst.  The outer logarithm only needs absolute
// accuracy.
__device__ __forceinline__ float gumbel_from_word(uint32_t w) {
  const float x = ((float)(0x7FFFFFu - (w >> 9)) + 0.5f) * 0x1p-23f;        // 1 - u
  const float e = x < 0.015625f ? x * (1.f + x * (0.5f + x * (0.33333334f + 0.25f * x))) : -__logf(1.f - x);
  return -__logf(e);
}

// Arguments of one tile-kernel launch (base part or hyper part).
struct LogitsArgs {
  const void* H;          // [rows, d]
  const void* W;          // base: [V, d]; hyper: [B, cap, d]
  const int32_t* size;    // hyper: [B] C_b; base: nullptr
  int32_t rows, rows_per_seq, d;
  int32_t w_rows;         // rows of one W matrix: V (base) or cap (hyper)
  int32_t col0;           // column of this part's first entry in a logits row: 0 or V
  int32_t n_vtiles;       // vocabulary tiles of one W matrix
  int32_t strip;          // vocabulary tiles per workgroup
  int32_t n_strips;       // strips of one W matrix
  int32_t part0;          // index of this launch's first partial
  int32_t n_parts;        // partials per hidden row (row stride of the part arrays)
  int32_t row_tiles;      // base: tiles over all rows; hyper: tiles per sequence
  int32_t n_work;         // workgroups with work: row tiles (x sequences) x strips
  // order of the tile kernel's base part and dense layers over (row tiles, strips), see locate_base: the side walked in
  // blocks (map_p_rows: row tiles), the block, and how many ways either side is dealt out to the 8 XCDs (xp * xq = 8)
  int32_t map_p_rows, map_lp, map_xp, map_xq;
  float* part_m;          // [rows, n_parts]
  float* part_s;
  int32_t* part_i;
  float* logits;          // nullptr or [rows, ld]
  int32_t ld;
  // linear mode of the bf16 MFMA kernel (a dense layer instead of a softmax fold):
  // out[r, n] = act(H[r, :] . W[n, :] + bias[n]) + residual[r, n], bf16, row stride ldo
  void* out;
  const float* bias;      // [w_rows] or nullptr
  const void* residual;   // [rows, ldo] bf16 or nullptr
  int32_t act;            // 0 none, 1 GELU (erf)
  int32_t ldo;
  int32_t stream_f32;     // 1: residual and out are fp32 (a residual stream kept unrounded between layers)
  // probability mode (the backward pass of the loss): out[r, c] = g[r] * (exp(logit - lse[r]) - [col0 + c == target[r]])
  // for the existing columns c < n_valid, 0 for the other columns below ldo; bf16, row stride ldo
  const float* lse;       // [rows]
  const float* row_grad;  // [rows] g: the upstream gradient, 0 for rows without a usable target
  const int32_t* targets; // [rows]
  const int32_t* rows_dev;  // nullptr, or the number of rows that exist (<= rows), known on the device only
  // linear mode with K split over ksplit workgroups per tile (few rows: too few tiles to fill the machine):
  // part ks covers K slabs [ks * slabs_per_part, ...) and leaves its fp32 tile in partial[ks][row][col]
  int32_t ksplit, slabs_per_part;
  float* partial;           // [ksplit][rows][ldo]
  // dense layer whose last round of tiles may be cut along K, as the device sees fit: 256 tile buffers of 256 x 256; nullptr: never
  float* split;
  // sampling fold (base part of a sampled decode step with many rows): the triples are taken over
  // logit * inv_temperature, and next to them the largest perturbed value (part_v), the scaled logit there
  // (part_l) and its column (part_i, instead of the maximum's); generator key and counter words as in the
  // decode kernel: word col & 3 of Philox4x32-10 at counter (col >> 2, row, ctr2, ctr3)
  int32_t sample;         // 1: fold the draw (part_v, part_l); 2: store logit * inv_temperature in `logits` and fold
  float inv_temperature;
  uint32_t key0, key1, ctr2, ctr3;
  float* part_v;
  float* part_l;
  // dense layer whose contraction length is only known on the device (a product over the rows of a pass):
  // K beyond *k_dev, up to the next multiple of 64, holds zeros and the slabs after that are not read
  const int32_t* k_dev;
  int32_t ldh, ldw;         // row pitch of H and W in elements (dense layers; 0: d)
  int32_t k_rows;           // rows of the K-major operands (dense layers whose contraction runs over them; at most *k_dev)
  int32_t batch;            // products with K-major operands in one launch (0, 1: one); the operands' steps in elements
  size_t batch_h, batch_w;
  int32_t once;             // weight-streaming kernel: the weights are read past the caches
  // the hyper part in the base part's launch (n_work > 0; fields as above, `out` and `ldo` in probability mode)
  struct {
    const void* W;
    const int32_t* size;
    void* out;
    int32_t ldo, cap, col0, strip, n_strips, part0, row_tiles, n_work, n_seq;
  } hyper;
};

// Weights of up to this many bytes are read through the memory-side cache (256 MB), where the next step finds them; more
// go past the caches (logits_decode.hip has the figures).
constexpr size_t kKeepBytes = (size_t)128 << 20;

// fold_tile for a filtered sampled pick: x = logit * inv_temperature enters the running triple and is stored,
// fp32, at logits[row, col0 + column] (the selection kernels read the rows back); 16-byte stores where the four
// columns of a group all exist.
template <int NI, int NJ>
__device__ __forceinline__ void fold_tile_store(const f32x16 (&acc)[NI][NJ], Triple (&run)[NJ], const LogitsArgs& a,
                                                int row_base, int r_end, int col_base, int n_valid) {
  const int lane31 = threadIdx.x & 31;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (row_base + j * 32 >= r_end) break;           // (uniform)
    const int row = row_base + j * 32 + lane31;
    float* out = a.logits + (size_t)min(row, r_end - 1) * a.ld + a.col0;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      float x[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int col = col_base + i * 32 + (v >> 2) * 8 + (v & 3);
        x[v] = col < n_valid ? read_acc(acc[i][j][v]) * a.inv_temperature : kNegInf;
      }
      float gmax = x[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) gmax = fmaxf(gmax, x[v]);
      if (gmax > run[j].m) {
        int targ = 15;
#pragma unroll
        for (int v = 14; v >= 0; --v) targ = (x[v] == gmax) ? v : targ;
        run[j].s = (run[j].m == kNegInf) ? 0.f : run[j].s * __expf(run[j].m - gmax);
        run[j].m = gmax;
        run[j].i = a.col0 + col_base + i * 32 + (targ >> 2) * 8 + (targ & 3);
      }
      if (run[j].m != kNegInf) {
        const float m = run[j].m;
        float add = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) add += __expf(x[v] - m);
        run[j].s += add;
      }
      if (row < r_end) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = col_base + i * 32 + q * 8;
          // (a row of the logits starts 4-byte aligned only: ld = V + cap is any number)
          if (col + 3 < n_valid && ((((size_t)row * a.ld + a.col0 + col) & 3) == 0)) {
            *reinterpret_cast<float4*>(out + col) = float4{x[q * 4], x[q * 4 + 1], x[q * 4 + 2], x[q * 4 + 3]};
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (col + k < n_valid) out[col + k] = x[q * 4 + k];
          }
        }
      }
    }
  }
}

// fold_tile for a sampled pick: the same register layout; x = logit * inv_temperature enters the running triple,
// and x + Gumbel(u[row, col]) the running draw.  A lane's columns come in aligned fours (one generator call
// each) and in increasing order, so a strict comparison keeps the lowest column among equal values.  The four
// groups of a 32 x 32 block are a real loop (the generator is long: unrolled 256 times per tile it would not fit
// the register file next to the accumulators).
template <int NI, int NJ>
__device__ __forceinline__ void fold_tile_sample(const f32x16 (&acc)[NI][NJ], Triple (&run)[NJ], Draw (&draw)[NJ],
                                                 const LogitsArgs& a, int row_base, int col_base, int n_valid) {
  const int lane31 = threadIdx.x & 31;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (row_base + j * 32 >= a.rows) break;          // (uniform; 24 sequences over 128256 columns: 236 -> 224 us, before the scratch memory went)
    const uint32_t row = (uint32_t)(row_base + j * 32 + lane31);
    Triple t = run[j];
    Draw dr = draw[j];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      float x[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) x[v] = read_acc(acc[i][j][v]);
#pragma unroll 1
      for (int q = 0; q < 4; ++q) {
        const int c0 = a.col0 + col_base + i * 32 + q * 8;
        const uint4 w = philox4x32_10(uint4{(uint32_t)(c0 >> 2), row, a.ctr2, a.ctr3}, a.key0, a.key1);
        const uint32_t word[4] = {w.x, w.y, w.z, w.w};
        float z[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          // (columns past the last valid one: -inf never enters the triple or wins the draw)
          z[k] = c0 - a.col0 + k < n_valid ? x[k] * a.inv_temperature : kNegInf;
          const float pv = z[k] + gumbel_from_word(word[k]);
          if (pv > dr.v) {
            dr.v = pv;
            dr.l = z[k];
            dr.i = c0 + k;
          }
        }
        const float m4 = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
        if (m4 > t.m) {
          t.s = (t.m == kNegInf) ? 0.f : t.s * __expf(t.m - m4);
          t.m = m4;
          t.i = c0 + (z[0] == m4 ? 0 : (z[1] == m4 ? 1 : (z[2] == m4 ? 2 : 3)));
        }
        const float m = t.m == kNegInf ? 0.f : t.m;  // (columns that do not exist add 0, a hidden row's NaN stay NaN)
        t.s += (__expf(z[0] - m) + __expf(z[1] - m)) + (__expf(z[2] - m) + __expf(z[3] - m));
        // (the next four move up: picked by q, the values go through scratch memory -- draws of 24 sequences over 128256
        // columns 224 -> 208 us, 64: 284 -> 267)
#pragma unroll
        for (int v = 0; v < 12; ++v) x[v] = x[v + 4];
      }
    }
    run[j] = t;
    draw[j] = dr;
  }
}

// Store one finished accumulator tile as it is (fp32), for a dense layer whose K range is split over several
// workgroups: 16-byte stores.
template <int NI, int NJ>
__device__ __forceinline__ void store_partial_tile(const f32x16 (&acc)[NI][NJ], float* part, int ld, int row_base,
                                                   int r_end, int col_base, int n_valid) {
  const int lane31 = threadIdx.x & 31;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int row = row_base + j * 32 + lane31;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = col_base + i * 32 + q * 8;
        float4 x;
        x.x = read_acc(acc[i][j][q * 4 + 0]);
        x.y = read_acc(acc[i][j][q * 4 + 1]);
        x.z = read_acc(acc[i][j][q * 4 + 2]);
        x.w = read_acc(acc[i][j][q * 4 + 3]);
        if (row < r_end && col < n_valid) *reinterpret_cast<float4*>(part + (size_t)row * ld + col) = x;
      }
    }
  }
}

}  // namespace z2z_logits

// kernel launchers, one per translation unit
int z2z_logits_general_columns(bool bf16, long long tiles_of_64);
int z2z_launch_logits_general(bool bf16, int columns, const z2z_logits::LogitsArgs& base, const z2z_logits::LogitsArgs* hyper, hipStream_t s);
// mode: 0 base part, 1 hyper part (both fold the joint softmax), 2 dense layer (stores the tile),
// 3 storing the gradient with respect to the logits, 5 dense layer with K split
// (fp32 partial tiles)
int z2z_launch_logits_fast(int mode, const z2z_logits::LogitsArgs& a, unsigned grid, hipStream_t s);
// mode 2 with W K-major, and H too (rows_too)
int z2z_launch_linear_kmajor(const z2z_logits::LogitsArgs& a, bool rows_too, unsigned grid, hipStream_t s);
// whether the device may cut the last round of a dense layer's tiles along K (LogitsArgs::split; z2z_logits_fast_order first): as far as
// the host knows the rows and the contraction
bool z2z_logits_fast_cuts(const z2z_logits::LogitsArgs& a);
// behind a dense layer launched with LogitsArgs::split, on 256 workgroups: the sums of the tiles that the device has cut along K
int z2z_launch_tile_sum(const z2z_logits::LogitsArgs& a, hipStream_t s);
// order and grid of a base part or dense layer (modes 0, 2, 3, 6 - 9): a.row_tiles, n_vtiles and n_strips are set; `forced`:
// Z2Z_OPT_LOGITS_MAP, 0 for the automatic order
unsigned z2z_logits_fast_order(z2z_logits::LogitsArgs& a, int forced);
// out[R, N] = act(A[R, K] . W[N, K]^T + bias) + residual, all matrices bf16 (bias float), on the bf16 MFMA kernel
// (R rows are laid out; with rows_dev only the first *rows_dev of them exist: the others are neither read nor
// written).  stream_f32: residual and out are fp32 instead (a residual stream that is not rounded between layers).
struct z2z_linear_pitch {
  int a, w, out;           // row pitches of A, W and the output (a residual has the output's)
};
int z2z_launch_linear(z2z_ctx* c, const void* A, const void* W, const float* bias, const void* residual, int act,
                      void* out, int R, const int32_t* rows_dev, int N, int K, hipStream_t s,
                      bool stream_f32 = false, const z2z_linear_pitch* pitch = nullptr,
                      bool once = false);
// The two products of a dense layer's backward pass, bf16, operands as the forward pass has them (nothing is transposed or padded;
// widths and pitches are multiples of 8, see logits_fast.hip).  All are row-major with pitches ld..:
//   z2z_launch_linear_input    out[R, N] = A[R, K] . W[k_rows, N] + residual;  A's columns from k_rows to K (K: a multiple of 64) are finite
//   z2z_launch_linear_weight   out[R, N] = A[k_rows, R]^T . W[k_rows, N] + residual;  with k_dev only the first *k_dev rows exist
// A batch of them: outputs of R rows below each other, W (and the second's A) batch_w (batch_a) elements apart.
struct z2z_linear_batch {
  int n;
  size_t a, w;
};
int z2z_launch_linear_input(z2z_ctx* c, const void* A, int lda, const void* W, int ldw, int k_rows, const void* residual, void* out, int ldo,
                            int R, const int32_t* rows_dev, int N, int K, hipStream_t s, z2z_linear_batch batch = {1, 0, 0});
int z2z_launch_linear_weight(z2z_ctx* c, const void* A, int lda, const void* W, int ldw, int k_rows, const int32_t* k_dev,
                             const void* residual, void* out, int R, int N, hipStream_t s, z2z_linear_batch batch = {1, 0, 0});
// Row pitch for n columns of an activation that is an operand of dense layers: n, or 64 more where n columns are a
// multiple of 4 KiB -- the tile kernel's workgroups read the same slab of 256 rows at a time, and rows that far apart
// on a power of two put it on a few memory channels (35400 rows x 4096 columns, K = 16384: 1.07 -> 1.18
// PFLOP/s; whole passes at n = 4096 2 % faster, n = 12288 level).  Odd
// multiples of 16 KiB stay: with 64 more columns the product at n = 8192 (29000 rows x 2048) takes 1061 us instead of
// 970.  (128 more gain nothing at 8192 and lose the gain at 16384.)
inline int z2z_activation_pitch(int n) { return n % 2048 || n % 16384 == 8192 ? n : n + 64; }
// Pitches are taken by the tile kernel alone; true if the layer runs on it, with K whole.
bool z2z_linear_takes_pitch(const z2z_ctx* c, int R, int N, int K);
// The same product where the layer's K is split over workgroups (few rows): only the fp32 partial tiles,
// [*ksplit][R][N] at *partial, which the caller adds up in order before the next dense layer is launched; *ksplit = 0:
// the layer is not split at this shape, nothing was launched.
int z2z_launch_linear_parts(z2z_ctx* c, const void* A, const void* W, int R, const int32_t* rows_dev, int N, int K,
                            const float** partial, int* ksplit, hipStream_t s, bool once = false);
int z2z_logits_fast_prepare(z2z_ctx* c);
int z2z_logits_fast_sequences();   // most sequences whose hyper part a launch of the tile kernel takes along
// One launch of the bf16 MFMA tile kernel over the base part (hyper = false), over the hyper part of n_seq sequences, or over both
// (z2z_add_hyper_part first)
int z2z_launch_logits_part(z2z_ctx* c, bool hyper, z2z_logits::LogitsArgs a, const void* W, int w_rows, int col0,
                           int part0, int strip, int rows, int rows_per_seq, bool timed, hipStream_t s, bool prob = false);
// Fills in a.hyper: sequences [seq0, seq0 + n_seq) with their W_hyper, columns from V on, parts from part0 on.
void z2z_add_hyper_part(const z2z_ctx* c, z2z_logits::LogitsArgs& a, const void* W_hyper, int part0, int strip, int rows_per_seq, int seq0, int n_seq);
// temperature sampling (one-row-per-sequence kernel only): softmax(logit / temperature), generator key and
// counter words from seed and step
struct z2z_sample_params {
  float temperature;
  uint64_t seed, step;
};
// hyper_only_base_parts >= 0: only the per-sequence hyper units run, and they leave their partials behind that
// many parts per row, which another launch (the tile kernel over the base vocabulary) fills
// parts: where the partial triples go (nullptr: the context's buffers)
int z2z_launch_logits_decode(z2z_ctx* c, const void* H, const void* W_base, const void* W_hyper, int* n_parts,
                             bool timed, const z2z_sample_params* sample, float* logits, hipStream_t s,
                             int hyper_only_base_parts = -1, const z2z_parts* parts = nullptr, int rows_per_seq = 1,
                             int seq_unit = 512);
// (hyper_only_base_parts >= 0, one row per sequence: seq_unit weight rows per hyper unit, z2z_logits_decode_hyper_unit)
// (units halve until there are `enough`)
int z2z_logits_decode_hyper_unit(const z2z_ctx* c, int enough = 512);
// rows_per_seq in 2..64 (with hyper_only_base_parts >= 0): the hyper part alone, one workgroup per sequence and
// seq_unit (64, 128 or 256) rows of its W_hyper; parts per row then: base parts + ceil(cap / seq_unit)
int z2z_logits_decode_seq_unit(const z2z_ctx* c);
// `logits` hold logit / temperature as the decode kernel stored them, `row_stat` the rows' maxima, then their
// log-sum-exps, of those values; `work` is scratch of z2z_sample_truncated_work_floats(rows) floats.
// z2z_sample_truncated_merges_parts: true when the selection's first kernel merges the parts into `row_stat` itself
// (the caller then launches no merge); otherwise `row_stat` must hold them when the call is made.
bool z2z_sample_truncated_merges_parts(const z2z_ctx* c, int n_parts, int32_t top_k, int base_columns, int hyper_columns);
int z2z_sample_list_parts();   // most parts per row that the short-list pass takes
int z2z_launch_sample_truncated(z2z_ctx* c, const float* logits, float* row_stat, int32_t rows, int n_parts,
                                float* work, const z2z_sample_params* sp, int32_t top_k, float top_p,
                                int32_t* token, float* logprob, hipStream_t s, int base_columns, int hyper_columns);
size_t z2z_sample_truncated_work_floats(int32_t rows);
// the same layer on the bandwidth-bound kernel of the decode step (few rows: every weight byte is read once per
// 64 rows); K a multiple of 128, N even
int z2z_launch_linear_skinny(z2z_ctx* c, const void* A, const void* W, const float* bias, const void* residual,
                             int act, void* out, int R, const int32_t* rows_dev, int N, int K, hipStream_t s,
                             bool stream_f32 = false);
int z2z_logits_decode_parts(const z2z_ctx* c);
void z2z_logits_decode_units(int* base_columns, int* hyper_columns);
bool z2z_logits_decode_ok(const z2z_ctx* c);
int z2z_logits_decode_prepare(z2z_ctx* c);

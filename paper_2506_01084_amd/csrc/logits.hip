// extended_logits: launch planning (which tile kernel, strips, workgroup mapping), the merge of the
// per-strip partial triples, and the scratch buffer that holds them.
//
// The base part (columns < V, shared W_base) and the hyper part (columns V.., one W_hyper per sequence,
// only the first C_b rows exist: section 2.3 of the zip2zip paper, "Consistent Vocabulary Updates") are
// two launches; both leave (max, sum-exp, argmax) triples per (strip, row), merged in column order.
#include "logits_common.h"
#include "logits_mid.h"

#include <string.h>

#include <algorithm>
#include <mutex>

namespace {

using namespace z2z_logits;

// ROW_THREADS (64 or 256) threads per hidden row: they take the row's partial triples round-robin
// (contiguous in memory), merge across lanes, then across the waves of the row; merge_triple keeps the
// lowest column among equal maxima, so the order of the merges does not matter.  A block is 256 threads:
// four rows with a wave each (few parts per row: prefill), or one row (a thousand parts: decode steps).
template <int ROW_THREADS>
__global__ void __launch_bounds__(256) logits_combine_kernel(const float* part_m, const float* part_s,
                                                             const int32_t* part_i, int n_parts, int rows,
                                                             int32_t* argmax, float* mx, float* lse) {
  constexpr int ROWS_PER_BLOCK = 256 / ROW_THREADS;
  const int lane = threadIdx.x & 63;
  const int t = threadIdx.x % ROW_THREADS;
  const int r = blockIdx.x * ROWS_PER_BLOCK + threadIdx.x / ROW_THREADS;
  Triple tr = empty_triple();
  if (r < rows) {
    const size_t base = (size_t)r * n_parts;
    for (int p = t; p < n_parts; p += ROW_THREADS) {
      Triple o;
      o.m = part_m[base + p];
      o.s = part_s[base + p];
      o.i = part_i[base + p];
      merge_triple(tr, o);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    Triple o;
    o.m = __shfl_xor(tr.m, off);
    o.s = __shfl_xor(tr.s, off);
    o.i = __shfl_xor(tr.i, off);
    merge_triple(tr, o);
  }
  if (ROW_THREADS > 64) {
    __shared__ Triple xch[4];
    if (lane == 0) xch[threadIdx.x >> 6] = tr;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
      for (int w = 1; w < 4; ++w) merge_triple(tr, xch[w]);
    }
  }
  if (t == 0 && r < rows) {
    if (argmax) argmax[r] = tr.i;
    if (mx) mx[r] = tr.m;
    if (lse) lse[r] = tr.m + logf(tr.s);
  }
}

int launch_combine(const z2z_parts& p, int n_parts, int rows, int32_t* argmax, float* mx, float* lse, hipStream_t s) {
  if (n_parts > 256)
    hipLaunchKernelGGL(logits_combine_kernel<256>, dim3(rows), dim3(256), 0, s, p.m, p.s, p.i, n_parts, rows, argmax,
                       mx, lse);
  else
    hipLaunchKernelGGL(logits_combine_kernel<64>, dim3((rows + 3) / 4), dim3(256), 0, s, p.m, p.s, p.i, n_parts, rows,
                       argmax, mx, lse);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

// Full-logits output only: unused hyper slots read -inf.
__global__ void __launch_bounds__(256) logits_mask_kernel(float* logits, int rows, int rows_per_seq, int V, int cap,
                                                          const int32_t* size) {
  const int r = blockIdx.x;
  if (r >= rows) return;
  const int b = r / rows_per_seq;
  const int C = min(max(size[b], 0), cap);
  float* row = logits + (size_t)r * (V + cap) + V;
  for (int c = C + threadIdx.x; c < cap; c += blockDim.x) row[c] = kNegInf;
}

// Sampling: merge the parts of a hidden row into the drawn column (largest perturbed value, lowest column
// among equals) and its log-probability, scaled logit there minus the log-sum-exp of the scaled logits.
// One block of 256 threads per row.
__global__ void __launch_bounds__(256) sample_combine_kernel(const float* part_m, const float* part_s,
                                                             const float* part_v, const float* part_l,
                                                             const int32_t* part_i, int n_parts, int rows,
                                                             int32_t* token, float* logprob) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x;
  Triple tr = empty_triple();        // .i unused here
  float bv = kNegInf, bl = 0.f;
  int bi = kNoColumn;
  const size_t base = (size_t)r * n_parts;
  for (int p = threadIdx.x; p < n_parts; p += 256) {
    Triple o;
    o.m = part_m[base + p];
    o.s = part_s[base + p];
    o.i = kNoColumn;
    merge_triple(tr, o);
    const float v = part_v[base + p];
    const int i = part_i[base + p];
    if (v > bv || (v == bv && i < bi)) {
      bv = v;
      bl = part_l[base + p];
      bi = i;
    }
  }
  __shared__ Triple xt[4];
  __shared__ float xv[4], xl[4];
  __shared__ int xi[4];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    Triple o;
    o.m = __shfl_xor(tr.m, off);
    o.s = __shfl_xor(tr.s, off);
    o.i = kNoColumn;
    merge_triple(tr, o);
    const float v = __shfl_xor(bv, off), l = __shfl_xor(bl, off);
    const int i = __shfl_xor(bi, off);
    if (v > bv || (v == bv && i < bi)) {
      bv = v;
      bl = l;
      bi = i;
    }
  }
  if (lane == 0) {
    const int w = threadIdx.x >> 6;
    xt[w] = tr;
    xv[w] = bv;
    xl[w] = bl;
    xi[w] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      merge_triple(tr, xt[w]);
      if (xv[w] > bv || (xv[w] == bv && xi[w] < bi)) {
        bv = xv[w];
        bl = xl[w];
        bi = xi[w];
      }
    }
    token[r] = bi;
    if (logprob) logprob[r] = bl - (tr.m + logf(tr.s));
  }
}

// nll[r] = lse[r] - H[r] . W[target[r]] (section 2.4 of the zip2zip paper: the next-token objective taken
// over the compressed sequence; the target is a base token or a hypertoken of the row's sequence).  One
// wave per hidden row, 16-byte chunks, fp32 accumulation of the products of the stored values (what the
// tile kernels compute for that column).  target < 0: no target, 0; a column that does not exist: +inf.
template <bool BF16>
__global__ void __launch_bounds__(256) target_nll_kernel(const uint4* H, const uint4* W_base, const uint4* W_hyper,
                                                         const int32_t* size, const int32_t* targets,
                                                         const float* lse, float* nll, int rows, int rows_per_seq,
                                                         int V, int cap, int d) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const int b = r / rows_per_seq;
  const int t = targets[r];
  const int C = min(max(size[b], 0), cap);
  if (t < 0 || t >= V + C) {
    if (lane == 0) nll[r] = t < 0 ? 0.f : INFINITY;
    return;
  }
  constexpr int EPC = BF16 ? 8 : 4;
  const int n_chunks = d / EPC;
  const uint4* w = t < V ? W_base + (size_t)t * n_chunks : W_hyper + ((size_t)b * cap + (t - V)) * n_chunks;
  const uint4* h = H + (size_t)r * n_chunks;
  float acc = 0.f;
  for (int c = lane; c < n_chunks; c += 64) {
    const uint4 x = h[c], y = w[c];
    const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (BF16) {
        acc = fmaf(__uint_as_float(xs[e] << 16), __uint_as_float(ys[e] << 16), acc);
        acc = fmaf(__uint_as_float(xs[e] & 0xFFFF0000u), __uint_as_float(ys[e] & 0xFFFF0000u), acc);
      } else {
        acc = fmaf(__uint_as_float(xs[e]), __uint_as_float(ys[e]), acc);
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) nll[r] = lse[r] - acc;
}

int ensure_sample_scratch(z2z_ctx* c, size_t need, hipStream_t s) {
  if (need <= c->part_vl_capacity) return Z2Z_OK;
  Z2Z_TRY_GROW(s);
  if (c->part_v) (void)hipFree(c->part_v);
  if (c->part_l) (void)hipFree(c->part_l);
  c->part_v = nullptr;
  c->part_l = nullptr;
  c->part_vl_capacity = 0;
  if (!z2z_device_malloc(&c->part_v, need * sizeof(float))) return Z2Z_ENOMEM;
  if (!z2z_device_malloc(&c->part_l, need * sizeof(float))) return Z2Z_ENOMEM;
  c->part_vl_capacity = need;
  return Z2Z_OK;
}

int ensure_scratch(z2z_ctx* c, size_t need, hipStream_t s) {
  if (need <= c->part_capacity) return Z2Z_OK;
  Z2Z_TRY_GROW(s);
  if (c->part_m) (void)hipFree(c->part_m);
  if (c->part_s) (void)hipFree(c->part_s);
  if (c->part_i) (void)hipFree(c->part_i);
  c->part_m = nullptr;
  c->part_s = nullptr;
  c->part_i = nullptr;
  c->part_capacity = 0;
  if (!z2z_device_malloc(&c->part_m, need * sizeof(float))) return Z2Z_ENOMEM;
  if (!z2z_device_malloc(&c->part_s, need * sizeof(float))) return Z2Z_ENOMEM;
  if (!z2z_device_malloc(&c->part_i, need * sizeof(int32_t))) return Z2Z_ENOMEM;
  c->part_capacity = need;
  return Z2Z_OK;
}

z2z_parts ctx_parts(const z2z_ctx* c) { return z2z_parts{c->part_m, c->part_s, c->part_i, c->part_capacity}; }

}  // namespace

// ---- the allocation-free entry point's scratch ------------------------------------------------------------
// One array per device (every GPU that loads the library holds its own copy, at its own address, until the
// process ends): three runs of Z2Z_STATIC_PARTS four-byte elements, the (max, sum-exp, argmax) partials.  In
// host code the array's name is a stand-in, not a device address: its address on a device is asked for once
// per device (with that device current) and only that pointer is ever handed to a kernel.
static __device__ __align__(256) unsigned char scratch[3 * (size_t)Z2Z_STATIC_PARTS * 4];

constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];   // nullptr: not looked up yet on that device
static std::mutex g_scratch_mutex;

int z2z_static_scratch_prepare(z2z_ctx* c) {
  if (c->device < 0 || c->device >= kMaxDevices) return Z2Z_EUNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[c->device]) return Z2Z_OK;
  int cur = -1;
  Z2Z_HIP_TRY(hipGetDevice(&cur));
  if (cur != c->device) return Z2Z_EHIP;   // the symbol's address is that of the current device's copy
  void* ptr = nullptr;
  Z2Z_HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
  if (!ptr) return Z2Z_EHIP;
  g_scratch_ptr[c->device] = ptr;
  return Z2Z_OK;
}

namespace {

// The static array of the context's device as three part arrays; false if its address is not known.
bool static_parts(const z2z_ctx* c, z2z_parts* out) {
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (c->device >= 0 && c->device < kMaxDevices) ptr = g_scratch_ptr[c->device];
  }
  if (!ptr) return false;
  float* f = reinterpret_cast<float*>(ptr);
  out->m = f;
  out->s = f + Z2Z_STATIC_PARTS;
  out->i = reinterpret_cast<int32_t*>(f + 2 * (size_t)Z2Z_STATIC_PARTS);
  out->capacity = Z2Z_STATIC_PARTS;
  return true;
}

}  // namespace

// The shape-dependent fields of one part's arguments (tiles of `tile` rows, strips); B: sequences of a hyper part.
static void fill_part(LogitsArgs& a, const int32_t* size, int tile, int tile_v, int B, const void* W, int w_rows, int col0, int part0,
                      int strip, int rows, int rows_per_seq) {
  a.W = W;
  a.size = size;
  a.w_rows = w_rows;
  a.col0 = col0;
  a.n_vtiles = (w_rows + tile_v - 1) / tile_v;
  a.strip = strip;
  a.n_strips = (a.n_vtiles + strip - 1) / strip;
  a.part0 = part0;
  a.row_tiles = size ? (rows_per_seq + tile - 1) / tile : (rows + tile - 1) / tile;
  a.n_work = (size ? B : 1) * a.row_tiles * a.n_strips;
}

void z2z_add_hyper_part(const z2z_ctx* c, LogitsArgs& a, const void* W_hyper, int part0, int strip, int rows_per_seq, int seq0, int n_seq) {
  LogitsArgs h;
  fill_part(h, c->st.size + seq0, 256, 256, n_seq, W_hyper, c->cfg.cap, c->cfg.V, part0, strip, 0, rows_per_seq);
  a.hyper.W = h.W;
  a.hyper.size = h.size;
  a.hyper.cap = h.w_rows;
  a.hyper.col0 = h.col0;
  a.hyper.strip = h.strip;
  a.hyper.n_strips = h.n_strips;
  a.hyper.part0 = h.part0;
  a.hyper.row_tiles = h.row_tiles;
  a.hyper.n_work = h.n_work;
  a.hyper.n_seq = n_seq;
}

int z2z_launch_logits_part(z2z_ctx* c, bool hyper, LogitsArgs a, const void* W, int w_rows, int col0,
                           int part0, int strip, int rows, int rows_per_seq, bool timed, hipStream_t s, bool prob) {
  fill_part(a, hyper ? c->st.size : nullptr, 256, 256, c->cfg.B, W, w_rows, col0, part0, strip, rows, rows_per_seq);
  unsigned grid = (unsigned)a.n_work;
  if (!hyper) grid = z2z_logits_fast_order(a, c->opt_logits_map);
  c->n_launch[hyper ? Z2Z_KERNEL_TILE_HYPER : Z2Z_KERNEL_TILE_BASE]++;
  if (a.hyper.n_work > 0) c->n_launch[Z2Z_KERNEL_TILE_HYPER]++;
  if (timed) Z2Z_HIP_TRY(hipEventRecord(c->ev_start[c->n_timed], s));
  // (measurement probes of the base part: see logits_fast_kernel, modes 8 and 9)
  const int plain_base = c->opt_logits_kernel == 2 ? 8 : (c->opt_logits_kernel == 3 ? 9 : 0);
  const int rc = z2z_launch_logits_fast(prob ? 3 : (a.sample && !hyper ? (a.sample == 2 ? 7 : 6) : (hyper ? 1 : plain_base)), a, grid, s);
  if (timed) {
    Z2Z_HIP_TRY(hipEventRecord(c->ev_stop[c->n_timed], s));
    c->n_timed++;
  }
  return rc;
}

// A workgroup sweeps a strip of 4 weight tiles with its rows' tile resident; with few row tiles that leaves CUs
// idle, so the strips shorten until there are `want` workgroups (or one tile per workgroup): two per CU for the
// bf16 tile kernel, four for the general kernel, of which two (tiles of 128 columns) or three (64) run on a CU at a time (fp32, 64, d = 256,
// 32000 columns, strips of 1 / 2 / 4 tiles: 1024 rows 159 / 156 / 179 us, 2048 rows 299 / 291 / 314).
static int pick_strip_for(const z2z_ctx* c, long long row_tiles, int n_vt, int want = 512) {
  if (c->opt_logits_strip > 0) return c->opt_logits_strip;
  int st = 4;
  while (st > 1 && row_tiles * ((n_vt + st - 1) / st) < want) st >>= 1;
  return st;
}


// A decode step of 5..64 sequences whose base vocabulary goes to the weight-streaming kernel, with the hyper units in a
// launch of their own, instead of the decode kernel's base and hyper units in one.  Either kernel has one tile of 256 weight
// rows per CU, so a last round of tiles that leaves CUs idle costs as much as a full one -- but in the decode kernel the
// hyper units run there.  d = 4096 (V = 151936: 3584), cap = 1024, codebooks full, us, one launch -> split, calls in a row:
//   tiles (of the rounds')            8 sequences   24           40           64
//   256 (V = 65536)         greedy    191 -> 103    201 -> 124   204 -> 142   203 -> 169
//                           draw      211 -> 112    220 -> 130   224 -> 153   223 -> 180
//                           filtered  206 -> 117    218 -> 135   225 -> 164   227 -> 185
//   313 (of 512, 80000)     greedy    193 -> 154    207 -> 174   209 -> 193   224 -> 222
//                           draw      214 -> 164    226 -> 186   228 -> 211   231 -> 240
//                           filtered  208 -> 167    224 -> 186   231 -> 217   239 -> 238
//   384 (of 512, 98304)     greedy    198 -> 159    216 -> 178   238 -> 197   238 -> 224
//                           draw      218 -> 169    232 -> 187   245 -> 214   241 -> 244
//                           filtered  215 -> 169    234 -> 192   256 -> 228   257 -> 250
//   448 (of 512, 114688)    greedy    214 -> 162    242 -> 182   290 -> 202   303 -> 230
//                           draw      233 -> 174    254 -> 192   320 -> 220   327 -> 251
//                           filtered  231 -> 175    261 -> 202   316 -> 239   332 -> 262
//   501 (of 512, 128256)    greedy    282 -> 180    289 -> 198   298 -> 217   307 -> 247
//                           draw      316 -> 189    321 -> 209   326 -> 238   332 -> 270
//                           filtered  312 -> 193    317 -> 219   330 -> 253   343 -> 275
//   594 (of 768, 151936)    greedy    262 -> 208    270 -> 227   283 -> 246   305 -> 271
//                           draw      294 -> 222    302 -> 243   310 -> 274   331 -> 303
//                           filtered  284 -> 224    298 -> 252   312 -> 283   337 -> 303
// Behind other work that has turned the caches over the one launch is 40-60 us slower and the split 2-5.
// Hence: up to 16 sequences, or more than two rounds, or a last round at least 7/8 full over all rounds, or hyper units that
// would open another round in one launch.
// 112 to 255 tiles leave so many CUs to the hyper units that the last of these decides.  Tiles + hyper units, one launch -> split, three
// sets of weights in turn; in brackets behind 600 MB of other writes:
//   d = 3072, greedy      112 tiles: 5 x 1024 73 -> 58 (96 -> 58), 24 x 2048 91 -> 92 (131 -> 94), 50 x 2048 (of 312) 177 -> 149 (234 -> 151)
//                         126: 24 x 1024 79 -> 72 (113 -> 73), 40 x 1024 86 -> 86 (130 -> 87), 17 x 4096 (of 262) 149 -> 118 (198 -> 119)
//                         160: 17 x 4096 151 -> 131 (205 -> 131)   197: 40 x 1024 149 -> 103 (205 -> 103)   254: 8 x 4096 143 -> 103 (196 -> 103)
//             draw        112: 5 x 1024 85 -> 65, 24 x 2048 95 -> 96    126: 40 x 1024 93 -> 95, 17 x 4096 168 -> 126    254: 8 x 4096 163 -> 111
//             filtered    126: 17 x 4096 153 -> 129    197: 40 x 1024 164 -> 120    254: 8 x 4096 159 -> 112, 64 x 4096 344 -> 323
//   d = 1024, greedy      112: 40 x 1024 46 -> 42 (58 -> 42)   126: 17 x 4096 58 -> 55 (77 -> 55)   197: 40 x 1024 64 -> 48 (83 -> 50)
//             draw        112: 40 x 1024 71 -> 52    126: 17 x 4096 78 -> 65    254: 40 x 1024 86 -> 67
//   d = 4096, greedy      126: 8 x 4096 106 -> 99 (148 -> 100)   160: 64 x 1024 197 -> 149 (242 -> 150)   254: 40 x 1024 204 -> 146 (263 -> 144)
// (d = 512, 768, 1536, 2048 alike; 24 x 2048 over 112 tiles at d = 2048 62 -> 67 in a row, 85 -> 67 behind other writes.)  The split needs
// halved tiles (up to 128) as long as all fits one round, and up to 208 tiles and units; above a round it needs 64 units, which
// count whole however few entries they have, so that they are what opens it.  Filtered steps stay in one launch
// where all fits one round, and for short rows (d <= 1024) until the units fill half of another.  That line was drawn when their split had hyper
// units of 512 rows (5 x 1024 over 112 tiles 104 -> 124; d = 1024, 197 tiles: 40 x 1024 86 -> 92; 254: 8 x 4096 81 -> 92) and lies too high for
// units of 64 to 256 (78 -> 64, 79 -> 60, 74 -> 58; d = 512, 126: 17 x 4096 75 -> 48, 50 x 2048 over 112 79 -> 60).
static bool split_few(const z2z_ctx* c, int rows, bool filtered) {
  const long long tiles = z2z_logits_mid_tiles(c->cfg.V), slots = (tiles + 255) / 256 * 256;
  int base_columns, hyper_columns;
  z2z_logits_decode_units(&base_columns, &hyper_columns);
  const long long units = (long long)rows * ((c->cfg.cap + hyper_columns - 1) / hyper_columns);
  const bool full = tiles + units > slots && (filtered && c->cfg.d <= 1024 ? units > 128 : units >= 64);
  const bool halves = !filtered && z2z_logits_mid_columns(c, c->cfg.V) < 256 && 16 * (tiles + units) <= 13 * slots;
  const bool pays = tiles >= 256 ? rows <= 16 || tiles > 512 || 8 * tiles >= 7 * slots || tiles + units > slots
                                 : tiles >= 112 && (full || halves);
  return rows > 4 && rows <= 64 && c->opt_decode_kernel == 0 && c->opt_logits_kernel == 0 && pays && z2z_logits_mid_ok(c, rows);
}

// Whether such a step reads its base vocabulary past the caches: by all of its weights, like the decode kernel that it leaves.
static bool split_few_once(const z2z_ctx* c, int rows) {
  return rows <= 64 && z2z_logits_mid_tiles(c->cfg.V) < 256 &&
         ((size_t)c->cfg.V + (size_t)c->cfg.B * c->cfg.cap) * c->cfg.d * sizeof(uint16_t) > kKeepBytes;
}

// Parts per row that any kind of step may leave (hyper units of 64 rows): every step sizes the scratch for all of them,
// so that a greedy one can be captured behind an eager draw at the same shape and the other way round.
static size_t step_parts(const z2z_ctx* c) {
  const int columns = z2z_logits_mid_columns(c, c->cfg.V);
  return (size_t)(c->cfg.V + columns - 1) / columns + (size_t)(c->cfg.cap + 63) / 64;
}

int z2z_launch_extended_logits(z2z_ctx* c, const void* H, int32_t rows, int32_t rows_per_seq, const void* W_base,
                               const void* W_hyper, int32_t* argmax, float* mx, float* lse, float* logits,
                               hipStream_t s, bool use_static) {
  const int V = c->cfg.V, cap = c->cfg.cap;
  const bool timed = c->opt_timing && c->n_timed < Z2Z_MAX_TIMED && c->ev_created;
  z2z_parts parts;
  if (use_static && !static_parts(c, &parts)) return Z2Z_EHIP;
  // the partial triples of this call: the device's static array must hold them as it is, the context's
  // buffers grow to hold them
  auto reserve = [&](size_t need) -> int {
    if (use_static) return need <= parts.capacity ? Z2Z_OK : Z2Z_ELIMIT;
    const int rc = ensure_scratch(c, need, s);
    parts = ctx_parts(c);
    return rc;
  };

  // the fast kernels never store logits: the full-logits output (small shapes) takes the general kernel
  const bool fast_ok = c->cfg.dtype == Z2Z_BF16 && c->cfg.d % 64 == 0 && c->fast_ready && logits == nullptr;
  // decode step: one hidden row per sequence -> the bandwidth-bound kernel (it can store the logits too).
  // Its base units serve 64 rows per pass over W_base, each pass at about the cost of the first; from the second
  // pass on the tile kernel takes the base vocabulary (all rows at once) and only the hyper units run here
  const bool decode_step = rows_per_seq == 1 && c->decode_ready && c->opt_decode_kernel != 1;
  const bool decode_split = decode_step && fast_ok && (rows > 64 || split_few(c, rows, false)) && c->opt_logits_kernel != 1;
  // a few rows per sequence (2..64: a verification step over drafted codes, a short chunk): every sequence's
  // W_hyper meets only its own rows, so the hyper part is bandwidth-bound like the decode step's; it goes to
  // that kernel's matrix-core units (one pass over each W_hyper), the base vocabulary to the tile kernel
  const bool seq_split = !decode_step && fast_ok && rows_per_seq >= 2 && rows_per_seq <= 64 && cap > 0 &&
                         c->decode_ready && c->opt_decode_kernel != 1 && c->opt_logits_kernel != 1;
  if (decode_step && !decode_split) {
    int n_parts = z2z_logits_decode_parts(c);
    int rc = reserve((use_static ? (size_t)n_parts : step_parts(c)) * rows);
    if (rc != Z2Z_OK) return rc;
    rc = z2z_launch_logits_decode(c, H, W_base, W_hyper, &n_parts, timed, nullptr, logits, s, -1, &parts);
    if (rc != Z2Z_OK) return rc;
    if (logits && cap > 0) {
      hipLaunchKernelGGL(logits_mask_kernel, dim3(rows), dim3(256), 0, s, logits, rows, rows_per_seq, V, cap,
                         c->st.size);
      Z2Z_HIP_TRY(hipGetLastError());
    }
    return launch_combine(parts, n_parts, rows, argmax, mx, lse, s);
  }

  // (the general kernel is many times slower per bf16 tile: even a tile with a few valid rows goes to the tile kernel)
  const bool fast = fast_ok && c->opt_logits_kernel != 1;

  // number of parts (strips of both launches), then the scratch for them
  const int tile = fast ? 256 : 128;
  const long long tiles_b = (rows + tile - 1) / tile, tiles_h = (long long)c->cfg.B * ((rows_per_seq + tile - 1) / tile);
  const int tile_v = fast ? 256 : z2z_logits_general_columns(c->cfg.dtype == Z2Z_BF16, tiles_b * ((V + 63) / 64) + tiles_h * ((cap + 63) / 64));
  const int base_vt = (V + tile_v - 1) / tile_v, hyp_vt = (cap + tile_v - 1) / tile_v;
  // few hidden rows in all (several per sequence, or 65..192 sequences): the base part is bound by the bytes of
  // W_base and goes to the kernel that streams the weights past all rows at once, one part per 256 weight rows (or 128)
  // (measured against the decode kernel's base units in a launch of their own at up to 64 rows: 260 against 305 us
  // for the call at config 2's shape; two or three passes of those units for more rows cost more still)
  const bool mid_base = fast && c->opt_logits_kernel == 0 && z2z_logits_mid_ok(c, rows);
  int strip_b = 1, strip_h = 1;
  if (fast) {
    if (!mid_base) strip_b = pick_strip_for(c, tiles_b, base_vt);
    strip_h = pick_strip_for(c, tiles_h, hyp_vt);
  } else {
    // (strips asked for, and those where the static array could not hold the parts of shorter ones, count in 128 columns;
    // the other entry point cuts the same way)
    const bool asked = c->opt_logits_strip > 0;
    const int unit = 128 / tile_v;
    const int units_b = (base_vt + unit - 1) / unit, units_h = (hyp_vt + unit - 1) / unit;
    strip_b = asked ? unit * c->opt_logits_strip : pick_strip_for(c, tiles_b, base_vt, 1024);
    strip_h = asked ? unit * c->opt_logits_strip : pick_strip_for(c, tiles_h, hyp_vt, 1024);
    if (!asked && (size_t)((base_vt + strip_b - 1) / strip_b + (hyp_vt + strip_h - 1) / strip_h) * rows > Z2Z_STATIC_PARTS) {
      strip_b = unit * pick_strip_for(c, tiles_b, units_b, 1024);
      strip_h = unit * pick_strip_for(c, tiles_h, units_h, 1024);
    }
  }
  const int mid_columns = z2z_logits_mid_columns(c, V);
  // the streaming kernel takes the hyper part of longer runs of rows along (up to 64 rows a sequence it has units of its own)
  const bool mid_both = mid_base && cap > 0 && rows_per_seq > 64 &&
                        (size_t)((V + mid_columns - 1) / mid_columns + (cap + mid_columns - 1) / mid_columns) * rows <= Z2Z_STATIC_PARTS;
  const int base_strips = mid_base ? (V + mid_columns - 1) / mid_columns : (base_vt + strip_b - 1) / strip_b;
  int hyp_strips = mid_both ? (cap + mid_columns - 1) / mid_columns : cap > 0 ? (hyp_vt + strip_h - 1) / strip_h : 0;
  int seq_unit = 0;
  if (decode_split || seq_split) {
    seq_unit = seq_split ? z2z_logits_decode_seq_unit(c) : z2z_logits_decode_hyper_unit(c);
    // (the static array may be too small for the parts of the smaller units; the other entry point cuts the same way)
    if ((size_t)(base_strips + (cap + seq_unit - 1) / seq_unit) * rows > Z2Z_STATIC_PARTS) seq_unit = seq_split ? 256 : 512;
    hyp_strips = (cap + seq_unit - 1) / seq_unit;
  }
  if (decode_split && !use_static) {
    const int rc = reserve(step_parts(c) * rows);
    if (rc != Z2Z_OK) return rc;
  }
  const int n_parts = base_strips + hyp_strips;
  int rc = reserve((size_t)n_parts * rows);
  if (rc != Z2Z_OK) return rc;

  LogitsArgs a;
  memset(&a, 0, sizeof(a));
  a.H = H;
  a.rows = rows;
  a.rows_per_seq = rows_per_seq;
  a.d = c->cfg.d;
  a.part_m = parts.m;
  a.part_s = parts.s;
  a.part_i = parts.i;
  a.logits = logits;
  a.ld = V + cap;
  a.n_parts = n_parts;

  if (!fast) {
    // both parts in one launch of the general kernel
    LogitsArgs h = a;
    fill_part(a, nullptr, tile, tile_v, 1, W_base, V, 0, 0, strip_b, rows, rows_per_seq);
    if (cap > 0) fill_part(h, c->st.size, tile, tile_v, c->cfg.B, W_hyper, cap, V, base_strips, strip_h, rows, rows_per_seq);
    c->n_launch[Z2Z_KERNEL_GENERAL]++;
    if (timed) Z2Z_HIP_TRY(hipEventRecord(c->ev_start[c->n_timed], s));
    rc = z2z_launch_logits_general(c->cfg.dtype == Z2Z_BF16, tile_v, a, cap > 0 ? &h : nullptr, s);
    if (rc != Z2Z_OK) return rc;
    if (timed) {
      Z2Z_HIP_TRY(hipEventRecord(c->ev_stop[c->n_timed], s));
      c->n_timed++;
    }
    if (logits && cap > 0) {
      hipLaunchKernelGGL(logits_mask_kernel, dim3(rows), dim3(256), 0, s, logits, rows, rows_per_seq, V, cap,
                         c->st.size);
      Z2Z_HIP_TRY(hipGetLastError());
    }
    return launch_combine(parts, n_parts, rows, argmax, mx, lse, s);
  }

  // Both parts in one launch of the tile kernel (the measurement probes run the base part alone), up to 32768 tiles, where the hyper part is a hundredth
  // of the call and its launch full anyway.  Two launches -> one, us: V = 32064, d = 3072 (126 tiles a row of them) 32 x 512 rows 2283 -> 2235, 128 x 128
  // 2275 -> 2211, 500 x 66 5035 -> 4956, 8 x 1024, 8 x 4096 and 16 x 4096 (32256 tiles) within 0.8 % either way; V = 128256, d = 4096 (501) 8 x 512
  // 2993 -> 2912, 8 x 1100 6964 -> 6872, 8 x 1800 level, 4 x 4100 (32565) 12463 -> 12403, 8 x 4096 (64128) 23420 -> 23560; V = 8192, d = 1024, 64 x 4000 (32000)
  // 3998 -> 3810.  (The same code twice: 0.6 % at that length.)
  const bool one_launch = !mid_base && cap > 0 && !decode_split && !seq_split && c->opt_logits_kernel != 2 && c->opt_logits_kernel != 3 &&
                          c->cfg.B <= z2z_logits_fast_sequences() && tiles_b * base_vt <= 32768;
  if (one_launch) z2z_add_hyper_part(c, a, W_hyper, base_strips, strip_h, rows_per_seq, 0, c->cfg.B);
  if (mid_both) {
    z2z_add_hyper_part(c, a, W_hyper, base_strips, 1, rows_per_seq, 0, c->cfg.B);
    a.hyper.n_work = c->cfg.B * hyp_strips;
  }
  if (mid_base) {
    if (timed) Z2Z_HIP_TRY(hipEventRecord(c->ev_start[c->n_timed], s));
    a.once = decode_split && split_few_once(c, rows);
    rc = z2z_launch_logits_mid(c, a, W_base, V, 0, s);
    if (timed && !decode_split) {
      Z2Z_HIP_TRY(hipEventRecord(c->ev_stop[c->n_timed], s));
      c->n_timed++;
    }
  } else {
    rc = z2z_launch_logits_part(c, false, a, W_base, V, 0, 0, strip_b, rows, rows_per_seq, timed, s);
  }
  if (rc != Z2Z_OK) return rc;
  if (cap > 0 && (decode_split || seq_split)) {
    int np = 0;
    rc = z2z_launch_logits_decode(c, H, W_base, W_hyper, &np, false, nullptr, nullptr, s, base_strips, &parts,
                                  seq_split ? rows_per_seq : 1, seq_unit);
    if (rc != Z2Z_OK) return rc;
  } else if (cap > 0 && !one_launch && !mid_both) {
    rc = z2z_launch_logits_part(c, true, a, W_hyper, cap, V, base_strips, strip_h, rows, rows_per_seq, false, s);
    if (rc != Z2Z_OK) return rc;
  }
  if (timed && mid_base && decode_split) {        // a step's two launches are timed together
    Z2Z_HIP_TRY(hipEventRecord(c->ev_stop[c->n_timed], s));
    c->n_timed++;
  }
  return launch_combine(parts, n_parts, rows, argmax, mx, lse, s);
}

int z2z_launch_extended_sample(z2z_ctx* c, const void* H, int32_t rows, int32_t rows_per_seq, const void* W_base,
                               const void* W_hyper, float temperature, int32_t top_k, float top_p, uint64_t seed,
                               uint64_t step, int32_t* token, float* logprob, hipStream_t s) {
  // built for the generation step: one hidden row per sequence, the bandwidth-bound kernel
  if (rows_per_seq != 1 || !c->decode_ready) return Z2Z_EUNSUPPORTED;
  int n_parts = z2z_logits_decode_parts(c);
  int rc = ensure_scratch(c, step_parts(c) * rows, s);
  if (rc != Z2Z_OK) return rc;
  z2z_sample_params sp;
  sp.temperature = temperature;
  sp.seed = seed;
  sp.step = step;
  const bool timed = c->opt_timing && c->n_timed < Z2Z_MAX_TIMED && c->ev_created;
  // 65..192 rows, and fewer by the rule of a greedy step: the base vocabulary goes to the weight-streaming kernel (with the
  // tile kernel's sampling epilogues)
  const bool mid_base = (rows > 64 || split_few(c, rows, top_k > 0 || top_p < 1.0f)) && c->opt_logits_kernel == 0 && z2z_logits_mid_ok(c, rows);
  const bool timed_pair = timed && mid_base && rows <= 64;       // a split step's two launches are timed together
  if (top_k <= 0 && top_p >= 1.0f && (rows > 128 || mid_base) && c->cfg.d % 64 == 0 && c->fast_ready &&
      c->opt_logits_kernel != 1) {
    // no filter, more than two passes of the decode kernel's base units (the generator in the tile kernel's
    // epilogue costs more than the second pass), or the streaming kernel: as for the argmax, the tile kernel takes the base vocabulary
    // (with the draw folded into its epilogue) and the hyper units run alone
    const int base_vt = (c->cfg.V + 255) / 256;
    const int strip_b = mid_base ? 1 : pick_strip_for(c, (rows + 255) / 256, base_vt);
    const int mid_columns = z2z_logits_mid_columns(c, c->cfg.V);
    const int base_strips = mid_base ? (c->cfg.V + mid_columns - 1) / mid_columns : (base_vt + strip_b - 1) / strip_b;
    const int unit = z2z_logits_decode_hyper_unit(c);
    n_parts = base_strips + (c->cfg.cap + unit - 1) / unit;
    rc = ensure_scratch(c, (size_t)n_parts * rows, s);
    if (rc != Z2Z_OK) return rc;
    // (a step's scratch serves every kind of step, captured ones too)
    rc = ensure_sample_scratch(c, std::max((size_t)n_parts, step_parts(c)) * rows, s);
    if (rc != Z2Z_OK) return rc;
    LogitsArgs a;
    memset(&a, 0, sizeof(a));
    a.H = H;
    a.rows = rows;
    a.rows_per_seq = 1;
    a.d = c->cfg.d;
    a.part_m = c->part_m;
    a.part_s = c->part_s;
    a.part_i = c->part_i;
    a.part_v = c->part_v;
    a.part_l = c->part_l;
    a.n_parts = n_parts;
    a.sample = 1;
    a.inv_temperature = 1.0f / temperature;
    a.key0 = (uint32_t)seed;
    a.key1 = (uint32_t)(seed >> 32);
    a.ctr2 = (uint32_t)step;
    a.ctr3 = (uint32_t)(step >> 32);
    if (timed_pair) Z2Z_HIP_TRY(hipEventRecord(c->ev_start[c->n_timed], s));
    a.once = mid_base && split_few_once(c, rows);
    if (mid_base)
      rc = z2z_launch_logits_mid(c, a, W_base, c->cfg.V, 0, s);
    else
      rc = z2z_launch_logits_part(c, false, a, W_base, c->cfg.V, 0, 0, strip_b, rows, 1, timed, s);
    if (rc != Z2Z_OK) return rc;
    if (c->cfg.cap > 0) {
      int np = 0;
      rc = z2z_launch_logits_decode(c, H, W_base, W_hyper, &np, false, &sp, nullptr, s, base_strips, nullptr, 1, unit);
      if (rc != Z2Z_OK) return rc;
    }
    if (timed_pair) Z2Z_HIP_TRY(hipEventRecord(c->ev_stop[c->n_timed++], s));
    hipLaunchKernelGGL(sample_combine_kernel, dim3(rows), dim3(256), 0, s, c->part_m, c->part_s, c->part_v,
                       c->part_l, c->part_i, n_parts, rows, token, logprob);
    Z2Z_HIP_TRY(hipGetLastError());
    return Z2Z_OK;
  }
  if (top_k <= 0 && top_p >= 1.0f) {
    // no filter: the draw is folded into the kernel that computes the logits, which are never stored
    rc = ensure_sample_scratch(c, (size_t)n_parts * rows, s);
    if (rc != Z2Z_OK) return rc;
    rc = z2z_launch_logits_decode(c, H, W_base, W_hyper, &n_parts, timed, &sp, nullptr, s);
    if (rc != Z2Z_OK) return rc;
    hipLaunchKernelGGL(sample_combine_kernel, dim3(rows), dim3(256), 0, s, c->part_m, c->part_s, c->part_v,
                       c->part_l, c->part_i, n_parts, rows, token, logprob);
    Z2Z_HIP_TRY(hipGetLastError());
    return Z2Z_OK;
  }
  // filters: the kernel stores the rows' logits / T (rows x (V + cap) floats of library scratch), the merge
  // gives the row maxima and log-sum-exps, and one workgroup per row selects the kept prefix and draws
  if (!c->trunc_ready) return Z2Z_EUNSUPPORTED;
  const size_t need = (size_t)rows * (size_t)(c->cfg.V + c->cfg.cap);
  if (need > c->sample_logits_capacity) {
    Z2Z_TRY_GROW(s);
    if (c->sample_logits) (void)hipFree(c->sample_logits);
    if (c->row_max) (void)hipFree(c->row_max);
    c->sample_logits = nullptr;
    c->row_max = nullptr;
    c->sample_logits_capacity = 0;
    if (!z2z_device_malloc(&c->sample_logits, need * sizeof(float))) return Z2Z_ENOMEM;
    // the row maxima and log-sum-exps, followed by the selection kernels' scratch
    if (!z2z_device_malloc(&c->row_max, (2 * (size_t)rows + z2z_sample_truncated_work_floats(rows)) * sizeof(float)))
      return Z2Z_ENOMEM;
    c->sample_logits_capacity = need;
  }
  int base_columns = 0, hyper_columns = 0;           // of a part: the decode kernel's units unless set
  if ((rows > 64 || mid_base) && c->cfg.d % 64 == 0 && c->fast_ready && c->opt_logits_kernel != 1) {
    // more than one pass of the decode kernel's base units, or a split step: the tile or the streaming kernel stores and folds the base
    // vocabulary's scaled logits, the hyper units run alone (strips of at most 2 tiles: the selection kernels'
    // short-list pass takes parts of up to 512 columns)
    const int base_vt = (c->cfg.V + 255) / 256;
    int strip_b = mid_base ? 1 : pick_strip_for(c, (rows + 255) / 256, base_vt);
    if (strip_b > 2) strip_b = 2;
    const int mid_columns = z2z_logits_mid_columns(c, c->cfg.V);
    const int base_strips = mid_base ? (c->cfg.V + mid_columns - 1) / mid_columns : (base_vt + strip_b - 1) / strip_b;
    // (hyper units of 512 rows are too few for a small batch: smaller ones, while the short-list pass takes as many parts.  21 sequences of up to
    // 4096 entries, V = 32064 121 -> 84 us, 20 x 1024, V = 128256 271 -> 213, 6 x 4096, V = 151936 291 -> 250.  From 200 of 512 rows on those
    // are the better ones here: a unit's logits leave it row by row, 108 x 1024 356 us, 361 in 432 of 256; 56 x 2048 341 and 348, 32 x 4096 338
    // and 349.  Below that at least 512 where those of 256 would be more than a round (129 to 199 of 512; units of 512 / 256 / 128 rows, codebooks full:
    // 33 x 2048, V = 128256 283 / 304 / 286 us, V = 32064 133 / 145 / 130, V = 151936 318 / 333 / 312; 96 x 1024 314 / 323 / 317, 150 / 156 / 150, 346 /
    // 352 / 344; a third full 40 x 2048 271 / 237 / 227, 120 / 94 / 84, 301 / 271 / 260) and where room for more than 2048 entries is seldom full and the units
    // that exist are few of them (21 x 730 of 4096 96 us in 336 units, 84 in 672; full 8 x 4096, V = 128256 260 -> 221))
    const long long wide = (long long)rows * ((c->cfg.cap + 511) / 512);
    hyper_columns = z2z_logits_decode_hyper_unit(c, wide < 200 && (c->cfg.cap > 2048 || wide > 128) ? 512 : 200);
    while (hyper_columns < 512 && base_strips + (c->cfg.cap + hyper_columns - 1) / hyper_columns > z2z_sample_list_parts()) hyper_columns *= 2;
    n_parts = base_strips + (c->cfg.cap + hyper_columns - 1) / hyper_columns;
    base_columns = mid_base ? mid_columns : strip_b * 256;
    LogitsArgs a;
    memset(&a, 0, sizeof(a));
    a.H = H;
    a.rows = rows;
    a.rows_per_seq = 1;
    a.d = c->cfg.d;
    a.part_m = c->part_m;
    a.part_s = c->part_s;
    a.part_i = c->part_i;
    a.n_parts = n_parts;
    a.sample = 2;
    a.inv_temperature = 1.0f / temperature;
    a.logits = c->sample_logits;
    a.ld = c->cfg.V + c->cfg.cap;
    if (timed_pair) Z2Z_HIP_TRY(hipEventRecord(c->ev_start[c->n_timed], s));
    a.once = mid_base && split_few_once(c, rows);
    if (mid_base)
      rc = z2z_launch_logits_mid(c, a, W_base, c->cfg.V, 0, s);
    else
      rc = z2z_launch_logits_part(c, false, a, W_base, c->cfg.V, 0, 0, strip_b, rows, 1, timed, s);
    if (rc != Z2Z_OK) return rc;
    if (c->cfg.cap > 0) {
      int np = 0;
      rc = z2z_launch_logits_decode(c, H, W_base, W_hyper, &np, false, &sp, c->sample_logits, s, base_strips, nullptr, 1, hyper_columns);
      if (rc != Z2Z_OK) return rc;
    }
    if (timed_pair) Z2Z_HIP_TRY(hipEventRecord(c->ev_stop[c->n_timed++], s));
  } else {
    rc = z2z_launch_logits_decode(c, H, W_base, W_hyper, &n_parts, timed, &sp, c->sample_logits, s);
    if (rc != Z2Z_OK) return rc;
  }
  if (!z2z_sample_truncated_merges_parts(c, n_parts, top_k, base_columns, hyper_columns)) {
    rc = launch_combine(ctx_parts(c), n_parts, rows, nullptr, c->row_max, c->row_max + rows, s);
    if (rc != Z2Z_OK) return rc;
  }
  return z2z_launch_sample_truncated(c, c->sample_logits, c->row_max, rows, n_parts, c->row_max + 2 * (size_t)rows, &sp,
                                     top_k, top_p, token, logprob, s, base_columns, hyper_columns);
}

int z2z_launch_extended_nll(z2z_ctx* c, const void* H, int32_t rows, int32_t rows_per_seq, const void* W_base,
                            const void* W_hyper, const int32_t* targets, float* nll, float* lse, hipStream_t s) {
  int rc = z2z_launch_extended_logits(c, H, rows, rows_per_seq, W_base, W_hyper, nullptr, nullptr, lse, nullptr, s);
  if (rc != Z2Z_OK) return rc;
  const dim3 grid((rows + 3) / 4), block(256);
  if (c->cfg.dtype == Z2Z_BF16)
    hipLaunchKernelGGL(target_nll_kernel<true>, grid, block, 0, s, reinterpret_cast<const uint4*>(H),
                       reinterpret_cast<const uint4*>(W_base), reinterpret_cast<const uint4*>(W_hyper), c->st.size,
                       targets, lse, nll, rows, rows_per_seq, c->cfg.V, c->cfg.cap, c->cfg.d);
  else
    hipLaunchKernelGGL(target_nll_kernel<false>, grid, block, 0, s, reinterpret_cast<const uint4*>(H),
                       reinterpret_cast<const uint4*>(W_base), reinterpret_cast<const uint4*>(W_hyper), c->st.size,
                       targets, lse, nll, rows, rows_per_seq, c->cfg.V, c->cfg.cap, c->cfg.d);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

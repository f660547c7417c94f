// Dense layers out = act(A W^T + bias) + residual on the logits kernels (bf16): which kernel serves which row
// count, the workgroup -> tile mapping of the tile kernel, and the sum of K-split partial tiles.  Used by the
// learned hyper-encoder (zip2zip paper, section 2.2) and by the backward pass of the loss (section 2.4).
#include "logits_common.h"
#include "logits_mid.h"

#include <string.h>

#include <algorithm>

using namespace z2z_logits;

namespace {

// Dense layer with K split over workgroups of the tile kernel: out = act(sum_ks partial[ks] + bias) + residual,
// the parts added in a fixed order; one thread per run of 4 columns.
__global__ void __launch_bounds__(256) linear_sum_kernel(const float* partial, int ksplit, int rows, const int32_t* rows_dev,
                                                         int N, const float* bias, int act, const void* residual,
                                                         void* out, int stream_f32) {
  const int n4 = N >> 2;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  const int r_end = rows_dev ? min(rows, *rows_dev) : rows;
  if (i >= (long long)r_end * n4) return;
  const int row = (int)(i / n4), col = (int)(i % n4) * 4;
  const size_t at = (size_t)row * N + col;
  float4 x = *reinterpret_cast<const float4*>(partial + at);
  for (int k = 1; k < ksplit; ++k) {
    const float4 y = *reinterpret_cast<const float4*>(partial + (size_t)k * rows * N + at);
    x.x += y.x;
    x.y += y.y;
    x.z += y.z;
    x.w += y.w;
  }
  const float4 b = bias ? *reinterpret_cast<const float4*>(bias + col) : float4{0.f, 0.f, 0.f, 0.f};
  finish_linear(x, b, act, residual, out, stream_f32, at);
}

// The partial tiles' buffer, at least `need` bytes of it.
int ensure_partial(z2z_ctx* c, size_t need, hipStream_t s) {
  if (need <= c->skinny_partial_bytes) return Z2Z_OK;
  Z2Z_TRY_GROW(s);
  if (c->skinny_partial) (void)hipFree(c->skinny_partial);
  c->skinny_partial = nullptr;
  c->skinny_partial_bytes = 0;
  const size_t want = need > ((size_t)64 << 20) ? need : ((size_t)64 << 20);
  if (!z2z_device_malloc(&c->skinny_partial, want)) return Z2Z_ENOMEM;
  c->skinny_partial_bytes = want;
  return Z2Z_OK;
}

}  // namespace

int z2z_launch_linear_parts(z2z_ctx* c, const void* A, const void* W, int R, const int32_t* rows_dev, int N, int K,
                            const float** partial, int* ksplit_out, hipStream_t s, bool once) {
  *ksplit_out = 0;
  // up to 128 rows (a decode step's new entries through the learned encoder at a small batch): bound by the weight
  // bytes; the weight-streaming kernel with K split over workgroups, its fp32 partial tiles summed with the layer's
  // epilogue.  (The encoder's newest-entry pass at d = 4096, d_ff = 4 d: 347 -> 302 us for 8 sequences, 401 -> 374
  // for 40; with the 192-row build for 129..192 rows laid out the tile kernel's K split below is faster, 432
  // against 459 us for 64 sequences.)
  if (R <= 128 && K % 64 == 0 && N % 4 == 0 && c->opt_logits_kernel == 0 && z2z_logits_mid_ok(c, R)) {
    const int ksplit = z2z_linear_mid_ksplit(N, K);
    int rc = ensure_partial(c, (size_t)ksplit * R * N * sizeof(float), s);
    if (rc != Z2Z_OK) return rc;
    *partial = reinterpret_cast<const float*>(c->skinny_partial);
    return z2z_launch_linear_mid(c, A, W, R, rows_dev, N, K, once, reinterpret_cast<float*>(c->skinny_partial),
                                 c->skinny_partial_bytes / sizeof(float), ksplit_out, s);
  }
  // more rows than the 64 the decode-step kernel serves per pass over the weights, but fewer 256 x 256 output
  // tiles than would give every CU one (a few hundred rows, or up to a few thousand with a narrow layer): the
  // tile kernel with K split over workgroups, so that the weights stream once for all rows and every CU has a
  // part (without it a layer of 144 tiles ran on 144 of the 256 CUs: 1.5 ms against 0.8 ms for 422 rows)
  if (R > 64 && c->fast_ready && K % 64 == 0 && N % 8 == 0 && c->opt_logits_kernel != 1) {
    const int row_tiles = (R + 255) / 256, n_vt = (N + 255) / 256, tiles = row_tiles * n_vt;
    const int n_slabs = K / 64;
    int ksplit = 1;
    while (tiles * ksplit < 192 && n_slabs / (ksplit * 2) >= 8) ksplit *= 2;
    if (ksplit > 1) {
      const int per = (n_slabs + ksplit - 1) / ksplit;
      ksplit = (n_slabs + per - 1) / per;
      int rc = ensure_partial(c, (size_t)ksplit * R * N * sizeof(float), s);
      if (rc != Z2Z_OK) return rc;
      LogitsArgs a;
      memset(&a, 0, sizeof(a));
      a.H = A;
      a.W = W;
      a.rows = R;
      a.rows_per_seq = R;
      a.d = K;
      a.w_rows = N;
      a.n_vtiles = n_vt;
      a.row_tiles = row_tiles;
      a.strip = 1;
      a.n_strips = n_vt;
      a.ldo = N;
      a.rows_dev = rows_dev;
      a.ksplit = ksplit;
      a.slabs_per_part = per;
      a.partial = reinterpret_cast<float*>(c->skinny_partial);
      *partial = a.partial;
      *ksplit_out = ksplit;
      return z2z_launch_logits_fast(5, a, (unsigned)(tiles * ksplit), s);
    }
  }
  return Z2Z_OK;
}

namespace {
constexpr size_t kSplitBytes = (size_t)256 * 256 * 256 * sizeof(float);      // LogitsArgs::split
// Contractions from this many slabs on may be cut: half of them saved is worth the launch of the sum (5 us where nothing was cut;
// where the host knows rows and contraction it sees that itself and launches none).  Learned encoder over codebooks with room for 2048 entries, a whole prompt: 2 x 148 tokens, d = 3584
// 1054 -> 694 us, 2 x 354, d = 3072 1019 -> 742, 8 x 847, d = 4096 8.59 -> 8.21 ms; a training step with it, 1 x 67 tokens, d = 4096 6.50 ->
// 5.24 ms; where the host knows the rows, 4 x 1347 without it, V = 151936 21.3 -> 19.3 ms (84 tiles: four parts were two rounds, three are one).
constexpr int kSplitSlabs = 32;

// Order and grid of a dense layer on the tile kernel; parts: its last round may be cut, if the device finds that worth it (without room for the
// parts, under capture for instance, the tiles stay whole).
unsigned order_dense(z2z_ctx* c, LogitsArgs& a, bool parts, hipStream_t s) {
  const unsigned grid = z2z_logits_fast_order(a, 0);
  if (!parts || !z2z_logits_fast_cuts(a) || ensure_partial(c, kSplitBytes, s) != Z2Z_OK) return grid;
  a.split = reinterpret_cast<float*>(c->skinny_partial);
  return 256;
}
}  // namespace

bool z2z_linear_takes_pitch(const z2z_ctx* c, int R, int N, int K) {
  // (more rows than the few-row kernels take, and not split over K by z2z_launch_linear_parts)
  const long long tiles = (long long)((R + 255) / 256) * ((N + 255) / 256);
  return R > 512 && c->fast_ready && K % 64 == 0 && N % 8 == 0 && (tiles >= 192 || K / 64 < 16);
}

int z2z_launch_linear(z2z_ctx* c, const void* A, const void* W, const float* bias, const void* residual, int act,
                      void* out, int R, const int32_t* rows_dev, int N, int K, hipStream_t s, bool stream_f32, const z2z_linear_pitch* pitch, bool once) {
  if (pitch && !z2z_linear_takes_pitch(c, R, N, K)) return Z2Z_EUNSUPPORTED;
  // (more rows than one tile's: how many there are, and with them whether a cut along K pays, may be known on the device only)
  const bool tile_parts = R > 256 && K / 64 >= kSplitSlabs && c->fast_ready && K % 64 == 0 && N % 8 == 0 && c->opt_logits_kernel != 1;
  const float* partial = nullptr;
  int ksplit = 0;
  int rc = Z2Z_OK;
  if (!tile_parts) rc = z2z_launch_linear_parts(c, A, W, R, rows_dev, N, K, &partial, &ksplit, s, once);
  if (rc != Z2Z_OK) return rc;
  if (ksplit > 0) {
    const long long n_threads = (long long)R * (N / 4);
    hipLaunchKernelGGL(linear_sum_kernel, dim3((unsigned)((n_threads + 255) / 256)), dim3(256), 0, s, partial, ksplit, R,
                       rows_dev, N, bias, act, residual, out, stream_f32 ? 1 : 0);
    Z2Z_HIP_TRY(hipGetLastError());
    return Z2Z_OK;
  }
  // few rows: bound by the weight bytes, which the decode-step kernel streams at HBM rate (it re-reads them
  // once per 64 rows, so it loses to the tile kernel beyond a few hundred rows)
  if (!tile_parts && R <= 512 && c->skinny_ready && K % 128 == 0 && N % 2 == 0 && c->opt_logits_kernel != 2)
    return z2z_launch_linear_skinny(c, A, W, bias, residual, act, out, R, rows_dev, N, K, s, stream_f32);
  if (!c->fast_ready || K % 64 != 0 || N % 8 != 0 || R < 1) return Z2Z_EUNSUPPORTED;
  LogitsArgs a;
  memset(&a, 0, sizeof(a));
  a.H = A;
  a.W = W;
  a.rows = R;
  a.rows_per_seq = R;
  a.d = K;
  a.w_rows = N;
  a.n_vtiles = (N + 255) / 256;
  a.row_tiles = (R + 255) / 256;
  a.strip = 1;
  a.n_strips = a.n_vtiles;
  a.out = out;
  a.bias = bias;
  a.residual = residual;
  a.act = act;
  a.ldo = pitch ? pitch->out : N;
  a.ldh = pitch ? pitch->a : 0;
  a.ldw = pitch ? pitch->w : 0;
  a.stream_f32 = stream_f32 ? 1 : 0;
  a.rows_dev = rows_dev;
  const unsigned grid = order_dense(c, a, tile_parts, s);
  rc = z2z_launch_logits_fast(2, a, grid, s);
  return rc == Z2Z_OK && a.split ? z2z_launch_tile_sum(a, s) : rc;
}

namespace {

int launch_kmajor(z2z_ctx* c, LogitsArgs& a, bool rows_too, const void* A, int lda, const void* W, int ldw, int k_rows, const void* residual,
                  void* out, int ldo, int R, int N, z2z_linear_batch batch, hipStream_t s) {
  if (!c->fast_ready || a.d % 64 != 0 || N % 8 != 0 || lda % 8 != 0 || ldw % 8 != 0 || R < 1 || N < 1 || batch.n < 1) return Z2Z_EUNSUPPORTED;
  a.H = A;
  a.W = W;
  a.ldh = lda;
  a.ldw = ldw;
  a.k_rows = k_rows;
  a.residual = residual;
  a.out = out;
  a.ldo = ldo;
  a.rows = R;
  a.rows_per_seq = R;
  a.w_rows = N;
  a.batch = batch.n;
  a.batch_h = batch.a;
  a.batch_w = batch.w;
  a.n_vtiles = (N + 255) / 256;
  a.row_tiles = batch.n * ((R + 255) / 256);
  a.strip = 1;
  a.n_strips = a.n_vtiles;
  const unsigned grid = order_dense(c, a, a.d / 64 >= kSplitSlabs, s);
  const int rc = z2z_launch_linear_kmajor(a, rows_too, grid, s);
  return rc == Z2Z_OK && a.split ? z2z_launch_tile_sum(a, s) : rc;
}

}  // namespace

int z2z_launch_linear_input(z2z_ctx* c, const void* A, int lda, const void* W, int ldw, int k_rows, const void* residual, void* out, int ldo,
                            int R, const int32_t* rows_dev, int N, int K, hipStream_t s, z2z_linear_batch batch) {
  LogitsArgs a;
  memset(&a, 0, sizeof(a));
  a.d = K;
  a.rows_dev = rows_dev;
  return launch_kmajor(c, a, false, A, lda, W, ldw, k_rows, residual, out, ldo, R, N, batch, s);
}

int z2z_launch_linear_weight(z2z_ctx* c, const void* A, int lda, const void* W, int ldw, int k_rows, const int32_t* k_dev,
                             const void* residual, void* out, int R, int N, hipStream_t s, z2z_linear_batch batch) {
  LogitsArgs a;
  memset(&a, 0, sizeof(a));
  a.d = (k_rows + 63) / 64 * 64;
  a.k_dev = k_dev;
  return launch_kmajor(c, a, true, A, lda, W, ldw, k_rows, residual, out, N, R, N, batch, s);
}

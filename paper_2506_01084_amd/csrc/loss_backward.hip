// Backward pass of the loss over the extended vocabulary (zip2zip paper, section 2.4, the objective over the
// compressed sequence): gradient into the hidden rows and both unembedding matrices, and through the pooling of
// the averaging hyper-encoder.
#include "logits_common.h"
#include "logits_mid.h"

#include <string.h>

#include <algorithm>

using namespace z2z_logits;

namespace {

// g[r]: the upstream gradient of row r (1 without one), 0 for rows without a target or whose target names no
// existing column.
__global__ void __launch_bounds__(256) row_grad_kernel(const int32_t* targets, const float* grad_nll, const int32_t* size,
                                                       int rows, int rows_per_seq, int V, int cap, float* g) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= rows) return;
  const int t = targets[r];
  const int C = min(max(size[r / rows_per_seq], 0), cap);
  g[r] = (t >= 0 && t < V + C) ? (grad_nll ? grad_nll[r] : 1.0f) : 0.f;
}

__global__ void __launch_bounds__(256) fill_zero_kernel(uint4* p, size_t n16) {
  const uint4 z = {0u, 0u, 0u, 0u};
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) p[i] = z;
}

// dE[t_j] += a_j * dW_hyper[b, e] for the tokens of every existing entry, float atomics (tokens recur across entries and
// sequences): a wave per entry and 512 features, lane l those at l + 64 t, so that an instruction adds to 256 bytes in a row; the entry's row
// is read once.  (A wave per entry, the row once per token: 8 x 1024 entries, d = 4096 442 us, 350 entries, d = 3072 83.)
__global__ void __launch_bounds__(256) pool_backward_kernel(const uint16_t* dW, float* dE, const int32_t* size,
                                                            const int32_t* ent_tokens, const int32_t* ent_len, int B,
                                                            int V, int M, int cap, int d, int groups, int mean,
                                                            const float* coef /* [Z2Z_MAX_M + 1][Z2Z_MAX_M] */) {
  const int lane = threadIdx.x & 63;
  const long long wid = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const long long row = wid / groups;
  if (row >= (long long)B * cap) return;
  const int b = (int)(row / cap), e = (int)(row % cap);
  if (e >= min(max(size[b], 0), cap)) return;
  const int f0 = (int)(wid % groups) * 512 + lane;
  float g[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) g[t] = f0 + 64 * t < d ? __uint_as_float((uint32_t)dW[row * d + f0 + 64 * t] << 16) : 0.f;
  const int L = min(max(ent_len[row], 1), M);
  for (int j = 0; j < L; ++j) {
    const int tok = min(max(ent_tokens[row * M + j], 0), V - 1);
    const float a = mean ? 1.0f / (float)L : coef[L * Z2Z_MAX_M + j];
    float* to = dE + (size_t)tok * d + f0;
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (f0 + 64 * t < d) atomicAdd(to + 64 * t, a * g[t]);
  }
}

size_t round_up(size_t x, size_t m) { return (x + m - 1) / m * m; }

}  // namespace

int z2z_launch_hyper_embed_backward(z2z_ctx* c, const void* dW_hyper, float* dE, hipStream_t s) {
  const int B = c->cfg.B, cap = c->cfg.cap;
  if (cap == 0) return Z2Z_OK;
  if (!c->coef_dev) return Z2Z_EHIP;       // (allocated and filled by z2z_create)
  const long long rows = (long long)B * cap;
  const int groups = (c->cfg.d + 511) / 512;
  hipLaunchKernelGGL(pool_backward_kernel, dim3((unsigned)((rows * groups + 3) / 4)), dim3(256), 0, s,
                     reinterpret_cast<const uint16_t*>(dW_hyper), dE, c->st.size, c->st.ent_tokens, c->st.ent_len, B,
                     c->cfg.V, c->cfg.M, cap, c->cfg.d, groups, c->cfg.pool == Z2Z_POOL_MEAN ? 1 : 0,
                     reinterpret_cast<const float*>(c->coef_dev));
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

// Gradient of sum_r grad_nll[r] * nll[r] with respect to H, W_base and W_hyper.  The gradient with respect to
// the logits, dZ = g * (softmax - onehot), is written out once in bf16 (the logits are recomputed by the
// forward kernel with another epilogue, using the forward pass's lse), then
//   dH = dZ_base W_base + dZ_hyper[b] W_hyper[b],   dW_base = dZ_base^T H,   dW_hyper[b] = dZ_hyper[b]^T H[b]
// are four dense products on the same MFMA kernel (the last and the second term, one per sequence, in a launch each), which reads
// every operand as it is.
int z2z_launch_extended_nll_backward(z2z_ctx* c, const void* H, int32_t rows, int32_t rows_per_seq, const void* W_base,
                                     const void* W_hyper, const int32_t* targets, const float* lse,
                                     const float* grad_nll, void* dH, void* dW_base, void* dW_hyper, hipStream_t s) {
  const int B = c->cfg.B, V = c->cfg.V, cap = c->cfg.cap, d = c->cfg.d;
  if (c->cfg.dtype != Z2Z_BF16 || d % 64 != 0 || !c->fast_ready) return Z2Z_EUNSUPPORTED;
  const size_t Vp = round_up(V, 64), capp = round_up(cap, 64);
  // The sequences go in chunks of n_seq, as many as the work-space limit allows (all of them at the sizes of
  // the benchmark configurations): dH and dW_hyper of a chunk are its own, dW_base of a later chunk adds to the
  // bf16 result of the earlier ones (one more rounding per chunk).
  // work space (bf16 unless noted), 256-byte aligned pieces
  size_t off = 0;
  size_t o_g, o_Pb, o_Ph;
  auto take = [&](size_t bytes) { const size_t at = off; off += round_up(bytes, 256); return at; };
  auto layout = [&](int n_seq) {
    const size_t rc = (size_t)n_seq * rows_per_seq;
    off = 0;
    o_g = take(rc * 4);                              // float g[rows of the chunk]
    o_Pb = take(rc * Vp * 2);                        // dZ, base columns      [rows, Vp]
    o_Ph = take(rc * capp * 2);                      // dZ, hyper columns     [rows, capp]
    return off;
  };
  const size_t limit = (size_t)200 << 30;
  int n_seq = B;
  if (c->opt_backward_chunk > 0 && c->opt_backward_chunk < n_seq) n_seq = c->opt_backward_chunk;
  while (n_seq > 1 && layout(n_seq) > limit) n_seq = (n_seq + 1) / 2;
  if (layout(n_seq) > limit) return Z2Z_ENOMEM;      // one sequence alone does not fit
  if (off > c->bwd_ws_bytes) {
    Z2Z_TRY_GROW(s);
    if (c->bwd_ws) (void)hipFree(c->bwd_ws);
    c->bwd_ws = nullptr;
    c->bwd_ws_bytes = 0;
    if (!z2z_device_malloc(&c->bwd_ws, off)) return Z2Z_ENOMEM;
    c->bwd_ws_bytes = off;
  }
  unsigned char* ws = reinterpret_cast<unsigned char*>(c->bwd_ws);
  float* g = reinterpret_cast<float*>(ws + o_g);
  void *Pb = ws + o_Pb, *Ph = ws + o_Ph;
  // (nothing is folded over a strip here, and a workgroup's operand stream runs on from tile to tile anyway.  Tiles one by one, against
  // strips of four: base part of 1448 rows, V = 151936 1332 -> 1238 us, 109, V = 32064 237 -> 66, 32768, V = 128256 24.55 -> 24.39 ms;
  // hyper part of 2 x 724 rows 217 -> 77 us.)
  const int strip = c->opt_logits_strip > 0 ? c->opt_logits_strip : 1;
  const uint16_t* H16 = reinterpret_cast<const uint16_t*>(H);
  const uint16_t* Wh16 = reinterpret_cast<const uint16_t*>(W_hyper);

  int rc;
  for (int b0 = 0; b0 < B; b0 += n_seq) {
    const int nb = b0 + n_seq <= B ? n_seq : B - b0;
    const int r0 = b0 * rows_per_seq, rows_c = nb * rows_per_seq;
    const uint16_t* Hc = H16 + (size_t)r0 * d;
    const uint16_t* Whc = Wh16 + (size_t)b0 * cap * d;
    hipLaunchKernelGGL(row_grad_kernel, dim3((rows_c + 255) / 256), dim3(256), 0, s, targets + r0,
                       grad_nll ? grad_nll + r0 : nullptr, c->st.size + b0, rows_c, rows_per_seq, V, cap, g);
    // ---- dZ: the forward kernel with the probability epilogue -------------------------------------------
    // (up to 192 rows are bound by the weights' bytes, as in the forward pass: the streaming kernel)
    const bool few = c->opt_logits_kernel == 0 && z2z_logits_mid_ok(c, rows_c);
    if (cap > 0) {
      const size_t n16 = (size_t)rows_c * capp * 2 / 16;
      hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)std::min<size_t>((n16 + 255) / 256, 4096)), dim3(256), 0, s,
                         reinterpret_cast<uint4*>(Ph), n16);
    }
    // (in one launch as many sequences as the tile kernel takes the hyper part of)
    const int most = cap > 0 ? z2z_logits_fast_sequences() : nb;
    for (int q0 = 0; q0 < nb; q0 += most) {
      const int nq = q0 + most <= nb ? most : nb - q0;
      const size_t row = (size_t)q0 * rows_per_seq;
      const uint16_t* Whq = Whc + (size_t)q0 * cap * d;
      LogitsArgs a;
      memset(&a, 0, sizeof(a));
      a.H = Hc + row * d;
      a.rows = nq * rows_per_seq;
      a.rows_per_seq = rows_per_seq;
      a.d = d;
      a.lse = lse + r0 + row;
      a.row_grad = g + row;
      a.targets = targets + r0 + row;
      a.out = reinterpret_cast<uint16_t*>(Pb) + row * Vp;
      a.ldo = (int)Vp;
      if (cap > 0) {
        z2z_add_hyper_part(c, a, Whq, 0, few ? 1 : strip, rows_per_seq, b0 + q0, nq);
        a.hyper.out = reinterpret_cast<uint16_t*>(Ph) + row * capp;
        a.hyper.ldo = (int)capp;
      }
      if (few) {
        const int columns = z2z_logits_mid_columns(c, V);
        a.hyper.n_work = cap > 0 ? nq * ((cap + columns - 1) / columns) : 0;
        rc = z2z_launch_logits_mid(c, a, W_base, V, 0, s);
      } else {
        rc = z2z_launch_logits_part(c, false, a, W_base, V, 0, 0, strip, nq * rows_per_seq, rows_per_seq, false, s, true);
      }
      if (rc != Z2Z_OK) return rc;
    }
    // ---- the products ------------------------------------------------------------------------------------------
    uint16_t* dHc = reinterpret_cast<uint16_t*>(dH) + (size_t)r0 * d;
    rc = z2z_launch_linear_input(c, Pb, (int)Vp, W_base, d, V, nullptr, dHc, d, rows_c, nullptr, d, (int)Vp, s);
    if (rc != Z2Z_OK) return rc;
    rc = z2z_launch_linear_weight(c, Pb, (int)Vp, Hc, d, rows_c, nullptr, b0 > 0 ? dW_base : nullptr, dW_base, V, d, s);
    if (rc != Z2Z_OK) return rc;
    if (cap > 0) {                                   // one product per sequence
      uint16_t* dWh = reinterpret_cast<uint16_t*>(dW_hyper) + (size_t)b0 * cap * d;
      rc = z2z_launch_linear_input(c, Ph, (int)capp, Whc, d, cap, dHc, dHc, d, rows_per_seq, nullptr, d, (int)capp, s,
                                   {nb, 0, (size_t)cap * d});
      if (rc != Z2Z_OK) return rc;
      rc = z2z_launch_linear_weight(c, Ph, (int)capp, Hc, d, rows_per_seq, nullptr, nullptr, dWh, cap, d, s,
                                    {nb, (size_t)rows_per_seq * capp, (size_t)rows_per_seq * d});
      if (rc != Z2Z_OK) return rc;
    }
  }
  return Z2Z_OK;
}

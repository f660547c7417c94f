// The pooling of one codebook entry's constituent embeddings (section 2.2 of the zip2zip paper, the "Averaging"
// hyper-encoder: padding contributes nothing, the divisor is the entry's own length), shared by hyper_embed's
// kernel and the fused generation-step update.  A wave owns 16-byte column chunks of the row: 1 KiB of each
// constituent row per instruction, fp32 accumulation in token order, one rounding (nearest-even) to the
// storage type.
#pragma once

#include "z2z_internal.h"

namespace z2z_embed {

struct EmbedArgs {
  const void* E;
  void* W;
  const int32_t* size;        // [B] C_b
  const int32_t* ent_tokens;  // [B, cap, M]
  const int32_t* ent_len;     // [B, cap]
  const int32_t* first;       // [B] or nullptr
  int32_t last_n;             // first == nullptr: 0 = all of [0, cap), n > 0 = the last n entries only
  int32_t B, V, M, cap, d;
  int32_t units_per_seq;      // entry walkers assigned to each sequence
  int32_t split;              // waves that share one entry's row (each takes every split-th group of 64 chunks)
  int32_t pool;
  float coef[Z2Z_MAX_M + 1][Z2Z_MAX_M];
};

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

// x / n for a small whole n, correctly rounded: the product with the rounded reciprocal and one correction by the
// exact remainder (Markstein), a third of a division's instructions.  (inf: the remainder is NaN, the product stands.)
__device__ __forceinline__ float div_small(float x, float n, float rcp_n) {
  const float q = x * rcp_n;
  const float c = fmaf(fmaf(-q, n, x), rcp_n, q);
  return c == c ? c : q;
}

template <bool PAST>
__device__ __forceinline__ void store_chunk(u32x4 v, u32x4* to) {
  if (PAST)
    __builtin_nontemporal_store(v, to);
  else
    *to = v;
}

// One row of L constituents.  U chunks of every constituent row are requested before the first is used: with one
// load in flight per wave the kernel waits for memory, not for its bandwidth.  PAST: the row goes out past the caches
// (nothing reads it again before the cache has turned over, and the popular embedding rows stay in L2 instead).
// 16 x 16384 entries, d = 3584 (1.9 GB written): 578 us; loads ahead 494; stores past the caches 322.
// 8 x 2048, d = 4096: 50, 37, 34.6 us.
template <bool BF16, int L, bool PAST>
__device__ __forceinline__ void embed_row_l(const EmbedArgs& a, const int32_t* toks, size_t out_row, int lane, int part) {
  constexpr int U = L <= 2 ? 4 : (L <= 4 ? 2 : 1);
  // elements per 16-byte chunk: 8 (bf16) or 4 (f32)
  constexpr int EPC = BF16 ? 8 : 4;
  const int n_chunks = a.d / EPC;
  const int step = 64 * a.split;
  u32x4* W = reinterpret_cast<u32x4*>(a.W) + out_row * (size_t)n_chunks;
  const u32x4* row[L];
  float cf[L];
#pragma unroll
  for (int j = 0; j < L; ++j) {
    row[j] = reinterpret_cast<const u32x4*>(a.E) + (size_t)min(max(toks[j], 0), a.V - 1) * n_chunks;
    cf[j] = a.coef[L][j];
  }
  const bool mean = a.pool == Z2Z_POOL_MEAN;                     // mean: plain sum, divided by L at the end
  constexpr float fL = (float)L, rL = 1.0f / (float)L;
  for (int c0 = part * 64 + lane; c0 < n_chunks; c0 += U * step) {
    u32x4 x[U][L];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < L; ++j) x[u][j] = row[j][min(c0 + u * step, n_chunks - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float acc[EPC];
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
#pragma unroll
      for (int j = 0; j < L; ++j) {
        const float w = mean ? 1.0f : cf[j];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (BF16) {
            acc[2 * e] = fmaf(w, __uint_as_float(x[u][j][e] << 16), acc[2 * e]);
            acc[2 * e + 1] = fmaf(w, __uint_as_float(x[u][j][e] & 0xFFFF0000u), acc[2 * e + 1]);
          } else {
            acc[e] = fmaf(w, __uint_as_float(x[u][j][e]), acc[e]);
          }
        }
      }
      if (mean && L > 1) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] = (L & (L - 1)) ? div_small(acc[e], fL, rL) : acc[e] * rL;
      }
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (BF16)
          o[e] = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)acc[2 * e], (__bf16)acc[2 * e + 1]});
        else
          o[e] = __float_as_uint(acc[e]);
      }
      if (c0 + u * step < n_chunks) store_chunk<PAST>(o, W + c0 + u * step);
    }
  }
}

// Entry row `out_row`: the pooled rows of its L tokens (L uniform over the wave).
template <bool BF16, bool PAST>
__device__ __forceinline__ void embed_row(const EmbedArgs& a, const int32_t* toks, int L, size_t out_row, int lane,
                                          int part) {
  static_assert(Z2Z_MAX_M == 8, "one case per length");
  switch (L) {
    case 1: return embed_row_l<BF16, 1, PAST>(a, toks, out_row, lane, part);
    case 2: return embed_row_l<BF16, 2, PAST>(a, toks, out_row, lane, part);
    case 3: return embed_row_l<BF16, 3, PAST>(a, toks, out_row, lane, part);
    case 4: return embed_row_l<BF16, 4, PAST>(a, toks, out_row, lane, part);
    case 5: return embed_row_l<BF16, 5, PAST>(a, toks, out_row, lane, part);
    case 6: return embed_row_l<BF16, 6, PAST>(a, toks, out_row, lane, part);
    case 7: return embed_row_l<BF16, 7, PAST>(a, toks, out_row, lane, part);
    default: return embed_row_l<BF16, 8, PAST>(a, toks, out_row, lane, part);
  }
}

// The arguments every launch fills alike.
inline void fill_embed_args(const z2z_ctx* c, const void* E, void* W_hyper, EmbedArgs* a) {
  a->E = E;
  a->W = W_hyper;
  a->size = c->st.size;
  a->ent_tokens = c->st.ent_tokens;
  a->ent_len = c->st.ent_len;
  a->first = nullptr;
  a->last_n = 0;
  a->B = c->cfg.B;
  a->V = c->cfg.V;
  a->M = c->cfg.M;
  a->cap = c->cfg.cap;
  a->d = c->cfg.d;
  a->units_per_seq = 1;
  a->split = 1;
  a->pool = c->cfg.pool;
  for (int L = 0; L <= Z2Z_MAX_M; ++L)
    for (int j = 0; j < Z2Z_MAX_M; ++j) a->coef[L][j] = c->coef[L][j];
}

}  // namespace z2z_embed

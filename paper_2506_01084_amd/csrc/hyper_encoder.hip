// Learned hyper-encoder for gfx950 (bf16): the network that turns the embeddings of a hypertoken's constituent
// base tokens, padded to M slots, into the hypertoken's vector (zip2zip paper, section 2.2; the attention and
// transformer rows of the hyper-encoder ablation table; the two-layer transformer of the training setup).
// The paper names the architectures only; what is computed here is the standard pre-norm encoder over the M
// slots, padding masked out as keys, mean of the real slots at the end:
//
//   X_i = E[y_i] + P_i;  A = LN1(X);  QKV = A Wqkv^T + b;  O = softmax(Q K^T / sqrt(d_head)) V per head;
//   Y = X + O Wo^T + bo;  Z = Y + GELU(LN2(Y) W1^T + b1) W2^T + b2  (transformer layers);  h = mean_i Z_i.
//
// All entries of a pass are batched, and only their real slots are rows: a one-workgroup scan over the entry
// lengths gives every entry its first row (padding slots and missing entries take no rows at all; a quarter
// of the M slots of a typical codebook is padding), the number of rows stays on the device and the kernels
// read it there.  Every dense layer is then one [rows, K] x [N, K]^T product on the bf16 MFMA kernel with
// bias / GELU / residual in its epilogue.  The kernels in this file are the bandwidth-bound rest: gather +
// LayerNorm (one wave per row, the row held in registers: read once), the L x L attention per entry and head
// (a wave per entry and 512 features: 64 lanes x 16 bytes, a head's dot products reduced across its lanes),
// and the final mean.  The residual stream (X, Y, Z) is fp32 from the gather to the final mean; the operands of
// the matrix products (LayerNorm outputs, q | k | v, attention outputs, the hidden layer) are bf16;
// accumulation and statistics are fp32.
#include "logits_common.h"

namespace {

using z2z_logits::bf16_bits_rne;

constexpr int E_KCH = 8;             // 16-byte chunks per lane of one row: d <= 64 * 8 * E_KCH = 4096
constexpr float E_EPS = 1e-5f;

struct RowMap {                      // which entries a pass covers, and where their rows sit
  const int32_t* size;               // [B] C_b
  const int32_t* ent_tokens;         // [B, cap, M]
  const int32_t* ent_len;            // [B, cap]
  const int32_t* first;              // [B] or nullptr
  int32_t last_n;                    // first == nullptr: 0 = entries from 0, n > 0 = the last n entries
  int32_t B, V, M, cap, d;
  int32_t u0, un;                    // entry units [u0, u0 + un) of every sequence
  // packed rows of this pass: entry unit bu = b * un + u owns rows [row0[bu], row0[bu + 1]), one per real slot;
  // row0[B * un] is the number of rows; row_slot[r] = bu * 8 + slot of row r
  int32_t* row0;
  int32_t* row_slot;
};

__device__ __forceinline__ int entry_of(const RowMap& m, int b, int u, int* C_out) {
  const int C = min(max(m.size[b], 0), m.cap);
  *C_out = C;
  const int base = m.first ? max(m.first[b], 0) : (m.last_n > 0 ? max(C - m.last_n, 0) : 0);
  return base + m.u0 + u;
}

// *p, or zeros.  (A choice between two vectors, `ok ? *p : zero`, is made between their addresses: a flat load, and scratch memory
// for the zeros.)
__device__ __forceinline__ uint4 load_if(bool ok, const uint4* p) {
  uint4 v = {0u, 0u, 0u, 0u};
  if (ok) v = *p;
  return v;
}

__device__ __forceinline__ void unpack8(const uint4& x, float (&f)[8]) {
  f[0] = __uint_as_float(x.x << 16);
  f[1] = __uint_as_float(x.x & 0xFFFF0000u);
  f[2] = __uint_as_float(x.y << 16);
  f[3] = __uint_as_float(x.y & 0xFFFF0000u);
  f[4] = __uint_as_float(x.z << 16);
  f[5] = __uint_as_float(x.z & 0xFFFF0000u);
  f[6] = __uint_as_float(x.w << 16);
  f[7] = __uint_as_float(x.w & 0xFFFF0000u);
}

// 8 consecutive fp32 values of a residual-stream row (two 16-byte accesses)
__device__ __forceinline__ void load8(const float* p, float (&f)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
  f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
  f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
}

__device__ __forceinline__ void store8(float* p, const float (&f)[8]) {
  *reinterpret_cast<float4*>(p) = float4{f[0], f[1], f[2], f[3]};
  *reinterpret_cast<float4*>(p + 4) = float4{f[4], f[5], f[6], f[7]};
}

__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
  uint4 o;
  o.x = bf16_bits_rne(f[0]) | (bf16_bits_rne(f[1]) << 16);
  o.y = bf16_bits_rne(f[2]) | (bf16_bits_rne(f[3]) << 16);
  o.z = bf16_bits_rne(f[4]) | (bf16_bits_rne(f[5]) << 16);
  o.w = bf16_bits_rne(f[6]) | (bf16_bits_rne(f[7]) << 16);
  return o;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

__device__ __forceinline__ int entry_len(const RowMap& m, int b, int u) {
  int C;
  const int e = entry_of(m, b, u, &C);
  return e < C ? min(max(m.ent_len[(size_t)b * m.cap + e], 1), m.M) : 0;
}

// Rows of the pass: exclusive scan of the entry lengths over all entry units, one workgroup of 1024 threads,
// each taking a run of consecutive units.
__global__ void __launch_bounds__(1024) enc_rows_kernel(RowMap m, int n_units) {
  __shared__ int wave_tot[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (n_units + 1023) / 1024;
  const int b0 = tid * per, b1 = min(b0 + per, n_units);
  int mine = 0;
  for (int bu = b0; bu < b1; ++bu) mine += entry_len(m, bu / m.un, bu % m.un);
  int incl = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  int base = incl - mine;
  for (int w = 0; w < wave; ++w) base += wave_tot[w];
  for (int bu = b0; bu < b1; ++bu) {
    const int L = entry_len(m, bu / m.un, bu % m.un);
    m.row0[bu] = base;
    for (int i = 0; i < L; ++i) m.row_slot[base + i] = bu * 8 + i;
    base += L;
  }
  if (tid == 1023) {
    int total = 0;
    for (int w = 0; w < 16; ++w) total += wave_tot[w];
    m.row0[n_units] = total;
  }
}

// One wave per row.  The residual stream X is fp32 (the layers add to it without rounding; only what feeds a
// matrix product is bf16).  GATHER: X[r] = E[token] + P[slot] is formed and stored first.  Then
// A[r] = bf16(LN(X[r]) * gamma + beta), statistics in two steps: mean, then the mean of the squared deviations.
template <bool GATHER>
__global__ void __launch_bounds__(256) enc_norm_kernel(RowMap m, const uint4* E, const uint4* P, float* X, uint4* A,
                                                       const float* gamma, const float* beta, int n_units) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= m.row0[n_units]) return;
  const int n_chunks = m.d / 8;
  float* xr = X + (size_t)r * m.d;
  uint4* ar = A + (size_t)r * n_chunks;
  float x[E_KCH][8];
  if (GATHER) {
    const int rs = m.row_slot[r];
    const int i = rs & 7;
    const int bu = rs >> 3;
    const int b = bu / m.un, u = bu % m.un;
    int C;
    const int e = entry_of(m, b, u, &C);
    const int tok = min(max(m.ent_tokens[((size_t)b * m.cap + e) * m.M + i], 0), m.V - 1);
    const uint4* er = E + (size_t)tok * n_chunks;
#pragma unroll
    for (int k = 0; k < E_KCH; ++k) {
      const int c = lane + 64 * k;
      if (c < n_chunks) {
        float ev[8];
        unpack8(er[c], ev);
        if (P) {
          float pv[8];
          unpack8(P[(size_t)i * n_chunks + c], pv);
#pragma unroll
          for (int t = 0; t < 8; ++t) ev[t] += pv[t];
        }
        store8(xr + c * 8, ev);
#pragma unroll
        for (int t = 0; t < 8; ++t) x[k][t] = ev[t];
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < E_KCH; ++k) {
      const int c = lane + 64 * k;
      if (c < n_chunks) load8(xr + c * 8, x[k]);
    }
  }
  float sum = 0.f;
#pragma unroll
  for (int k = 0; k < E_KCH; ++k)
    if (lane + 64 * k < n_chunks) {
#pragma unroll
      for (int t = 0; t < 8; ++t) sum += x[k][t];
    }
  const float mean = wave_sum(sum) / (float)m.d;
  float sq = 0.f;
#pragma unroll
  for (int k = 0; k < E_KCH; ++k)
    if (lane + 64 * k < n_chunks) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float dv = x[k][t] - mean;
        sq += dv * dv;
      }
    }
  const float rstd = rsqrtf(wave_sum(sq) / (float)m.d + E_EPS);
#pragma unroll
  for (int k = 0; k < E_KCH; ++k) {
    const int c = lane + 64 * k;
    if (c < n_chunks) {
      const float4 g0 = *reinterpret_cast<const float4*>(gamma + c * 8), g1 = *reinterpret_cast<const float4*>(gamma + c * 8 + 4);
      const float4 b0 = *reinterpret_cast<const float4*>(beta + c * 8), b1 = *reinterpret_cast<const float4*>(beta + c * 8 + 4);
      const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
      const float bt[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
      float y[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) y[t] = (x[k][t] - mean) * rstd * g[t] + bt[t];
      ar[c] = pack8(y);
    }
  }
}

// ---- few rows: a workgroup per row or entry -------------------------------------------------------------------
// With a hundred rows in a pass every one of these launches is a chain of trips to memory, so a row gets a wave per
// 256 columns instead of one for all, and what follows a K-split dense layer adds up its partial tiles itself.  Newest
// entries of 8, 24, 64 sequences at d = 4096, two layers: 297 -> 261 us, 342 -> 307, 430 -> 395.
struct Parts {
  const float* partial;          // [ksplit][R][d], added up in order
  int ksplit, R;
  const float* bias;             // [d]
  const float* residual;         // [R, d]
};

// 4 columns from `col` of row r of the layer's output: sum of the parts, bias, residual.
__device__ __forceinline__ float4 sum_parts(const Parts& p, int r, int col, int d) {
  const size_t at = (size_t)r * d + col, plane = (size_t)p.R * d;
  const float4 rv = *reinterpret_cast<const float4*>(p.residual + at);
  const float4 b = p.bias ? *reinterpret_cast<const float4*>(p.bias + col) : float4{0.f, 0.f, 0.f, 0.f};
  float4 x = *reinterpret_cast<const float4*>(p.partial + at);
#pragma unroll 8
  for (int k = 1; k < p.ksplit; ++k) {
    const float4 y = *reinterpret_cast<const float4*>(p.partial + (size_t)k * plane + at);
    x.x += y.x;
    x.y += y.y;
    x.z += y.z;
    x.w += y.w;
  }
  return float4{x.x + b.x + rv.x, x.y + b.y + rv.y, x.z + b.z + rv.z, x.w + b.w + rv.w};
}

constexpr int E_FEW_ROWS = 2048;
constexpr int E_ROW_THREADS = 1024;    // 4 columns each: d <= 4096
static_assert(4 * E_ROW_THREADS >= 64 * 8 * E_KCH, "a row fits the workgroup");

__device__ __forceinline__ float row_sum(float v, float* xch) {      // over the workgroup; xch: 16 floats of its own
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) xch[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int w = 0; w < E_ROW_THREADS / 64; ++w) t += xch[w];
  return t;
}

// enc_norm_kernel for few rows: X[r] = E[token] + P[slot] (GATHER) or the finished sum of a K-split layer, then A[r].
template <bool GATHER>
__global__ void __launch_bounds__(E_ROW_THREADS) enc_row_norm_kernel(RowMap m, const uint16_t* E, const uint16_t* P, Parts parts,
                                                                     float* X, uint16_t* A, const float* gamma,
                                                                     const float* beta, int n_units) {
  __shared__ float xch[2][E_ROW_THREADS / 64];
  const int r = blockIdx.x;
  if (r >= m.row0[n_units]) return;
  const int col = 4 * (int)threadIdx.x;
  const bool in = col < m.d;
  float4 g = {0.f, 0.f, 0.f, 0.f}, bt = g, x = g;
  if (in) {
    g = *reinterpret_cast<const float4*>(gamma + col);
    bt = *reinterpret_cast<const float4*>(beta + col);
  }
  if (GATHER) {
    const int rs = m.row_slot[r];
    const int i = rs & 7;
    const int bu = rs >> 3;
    const int b = bu / m.un, u = bu % m.un;
    int C;
    const int e = entry_of(m, b, u, &C);
    const int tok = min(max(m.ent_tokens[((size_t)b * m.cap + e) * m.M + i], 0), m.V - 1);
    if (in) {
      const uint2 ev = *reinterpret_cast<const uint2*>(E + (size_t)tok * m.d + col);
      const uint2 pv = P ? *reinterpret_cast<const uint2*>(P + (size_t)i * m.d + col) : uint2{0u, 0u};
      x.x = __uint_as_float(ev.x << 16) + __uint_as_float(pv.x << 16);
      x.y = __uint_as_float(ev.x & 0xFFFF0000u) + __uint_as_float(pv.x & 0xFFFF0000u);
      x.z = __uint_as_float(ev.y << 16) + __uint_as_float(pv.y << 16);
      x.w = __uint_as_float(ev.y & 0xFFFF0000u) + __uint_as_float(pv.y & 0xFFFF0000u);
    }
  } else if (in) {
    x = sum_parts(parts, r, col, m.d);
  }
  if (in) *reinterpret_cast<float4*>(X + (size_t)r * m.d + col) = x;
  const float mean = row_sum((x.x + x.y) + (x.z + x.w), xch[0]) / (float)m.d;
  const float dx = x.x - mean, dy = x.y - mean, dz = x.z - mean, dw = x.w - mean;
  const float rstd = rsqrtf(row_sum(in ? (dx * dx + dy * dy) + (dz * dz + dw * dw) : 0.f, xch[1]) / (float)m.d + E_EPS);
  if (in) {
    uint2 o;
    o.x = bf16_bits_rne(dx * rstd * g.x + bt.x) | (bf16_bits_rne(dy * rstd * g.y + bt.y) << 16);
    o.y = bf16_bits_rne(dz * rstd * g.z + bt.z) | (bf16_bits_rne(dw * rstd * g.w + bt.w) << 16);
    *reinterpret_cast<uint2*>(A + (size_t)r * m.d + col) = o;
  }
}

// enc_pool_kernel behind a K-split last layer: grid (entries, ceil(d / 256)), a lane per 4 columns, a wave per slot
// (the first adds the slots up, in order).
__global__ void __launch_bounds__(64 * Z2Z_MAX_M) enc_sum_pool_kernel(RowMap m, Parts parts, uint16_t* W, int zero_missing) {
  __shared__ float4 xch[Z2Z_MAX_M][64];
  const int bu = blockIdx.x, lane = threadIdx.x & 63, i = threadIdx.x >> 6;
  const int col = 4 * (int)(blockIdx.y * 64 + lane);
  const int b = bu / m.un, u = bu % m.un;
  int C;
  const int e = entry_of(m, b, u, &C);
  if (e >= m.cap) return;                            // (the whole workgroup)
  uint2* w = reinterpret_cast<uint2*>(W + ((size_t)b * m.cap + e) * m.d + col);
  if (e >= C) {
    if (zero_missing && i == 0 && col < m.d) *w = uint2{0u, 0u};
    return;
  }
  const int r0 = m.row0[bu], L = m.row0[bu + 1] - r0;
  if (i < L && col < m.d) xch[i][lane] = sum_parts(parts, r0 + i, col, m.d);
  __syncthreads();
  if (i > 0 || col >= m.d) return;
  float4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int j = 0; j < L; ++j) {
    acc.x += xch[j][lane].x;
    acc.y += xch[j][lane].y;
    acc.z += xch[j][lane].z;
    acc.w += xch[j][lane].w;
  }
  const float invL = 1.0f / (float)L;
  uint2 o;
  o.x = bf16_bits_rne(acc.x * invL) | (bf16_bits_rne(acc.y * invL) << 16);
  o.y = bf16_bits_rne(acc.z * invL) | (bf16_bits_rne(acc.w * invL) << 16);
  *w = o;
}

// Attention among the slots of one entry.  QKV [rows, 3d] holds q | k | v of every real slot; a wave takes
// one entry and 512 consecutive features (whole heads: the head width is a power of two of at most 512), lane
// l the 8 features of chunk l.  Scores are reduced over the lanes_per_head lanes of a head; the softmax runs
// over the entry's L rows.
template <int MM>
__global__ void __launch_bounds__(256) enc_attention_kernel(RowMap m, const uint4* QKV, uint4* O, int lanes_per_head,
                                                            float scale, int groups, int n_units) {
  const int lane = threadIdx.x & 63;
  const long long wid = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int g = (int)(wid % groups);
  const long long bu = wid / groups;
  if (bu >= n_units) return;
  const int n_chunks = m.d / 8;
  const int c = g * 64 + lane;
  const bool active = c < n_chunks;
  const size_t r0 = (size_t)m.row0[bu];
  const int L = m.row0[bu + 1] - m.row0[bu];
  // (an entry's keys and values: all asked for at once, and once; 24 entries, d = 4096: 8.7 -> 6.6 us)
  uint4 kv[2][MM];
#pragma unroll
  for (int j = 0; j < MM; ++j)
#pragma unroll
    for (int h = 0; h < 2; ++h) kv[h][j] = load_if(active && j < L, QKV + (r0 + j) * 3 * n_chunks + (h + 1) * n_chunks + c);
  for (int i = 0; i < L; ++i) {
    float q[8];
    unpack8(load_if(active, QKV + (r0 + i) * 3 * n_chunks + c), q);
    float s[MM];
    float smax = -INFINITY;
#pragma unroll
    for (int j = 0; j < MM; ++j) {
      s[j] = -INFINITY;
      if (j < L) {
        float k[8];
        unpack8(kv[0][j], k);
        float dot = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) dot += q[t] * k[t];
        for (int off = 1; off < lanes_per_head; off <<= 1) dot += __shfl_xor(dot, off);
        s[j] = dot * scale;
        smax = fmaxf(smax, s[j]);
      }
    }
    float den = 0.f;
#pragma unroll
    for (int j = 0; j < MM; ++j) {
      s[j] = j < L ? __expf(s[j] - smax) : 0.f;
      den += s[j];
    }
    const float inv = 1.0f / den;
    float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < MM; ++j) {
      if (j < L) {
        float v[8];
        unpack8(kv[1][j], v);
        const float p = s[j] * inv;
#pragma unroll
        for (int t = 0; t < 8; ++t) o[t] += p * v[t];
      }
    }
    if (active) O[(r0 + i) * n_chunks + c] = pack8(o);
  }
}

// h = mean of the entry's real slots of Z -> W_hyper[b, e]; one wave per entry.  Passes that start at entry 0
// (full mode) also zero the rows of missing entries.
__global__ void __launch_bounds__(256) enc_pool_kernel(RowMap m, const float* Z, uint4* W, int n_units, int zero_missing) {
  const int lane = threadIdx.x & 63;
  const long long bu = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (bu >= n_units) return;
  const int b = (int)(bu / m.un), u = (int)(bu % m.un);
  const int n_chunks = m.d / 8;
  int C;
  const int e = entry_of(m, b, u, &C);
  if (e >= m.cap) return;
  uint4* wrow = W + ((size_t)b * m.cap + e) * n_chunks;
  if (e >= C) {
    if (zero_missing) {
      const uint4 z = {0u, 0u, 0u, 0u};
      for (int c = lane; c < n_chunks; c += 64) wrow[c] = z;
    }
    return;
  }
  const int L = m.row0[bu + 1] - m.row0[bu];
  const float invL = 1.0f / (float)L;
  const size_t r0 = (size_t)m.row0[bu];
  for (int c = lane; c < n_chunks; c += 64) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < L; ++i) {
      float z[8];
      load8(Z + (r0 + i) * m.d + c * 8, z);
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] += z[t];
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] *= invL;
    wrow[c] = pack8(acc);
  }
}

// ---------------------------------------------------------------------------------------------------------
// Backward pass (training f_phi: the loss reaches the encoder through every hypertoken vector, section 2.4).
// Reverse mode over the forward steps above.  Every product with a weight matrix, and every weight gradient
// (a product over the rows of the pass), runs on the same MFMA kernel, which reads the operands as they are; the kernels
// below are the bandwidth-bound rest.  Gradients between kernels are bf16, sums fp32.
// ---------------------------------------------------------------------------------------------------------

// The vector gradients, cleared in one launch (17 of them took 77 us): grid (64, pieces).
struct Pieces {
  static constexpr int kMax = 8 * Z2Z_MAX_ENCODER_LAYERS + 1;
  int n;
  float* p[kMax];
  int32_t len[kMax];
};
__global__ void __launch_bounds__(256) enc_fill_kernel(Pieces z) {
  float* p = z.p[blockIdx.y];
  const int n = z.len[blockIdx.y];
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += 64 * 256) p[i] = 0.f;
}

// dX[r] = dW_hyper[b, e] / L for the L rows of every entry (h = mean of the real slots); one wave per entry.
__global__ void __launch_bounds__(256) enc_pool_backward_kernel(RowMap m, const uint4* dW, uint4* dX, int n_units) {
  const int lane = threadIdx.x & 63;
  const long long bu = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (bu >= n_units) return;
  const int L = m.row0[bu + 1] - m.row0[bu];
  if (L < 1) return;
  const int b = (int)(bu / m.un), u = (int)(bu % m.un);
  const int n_chunks = m.d / 8;
  int C;
  const int e = entry_of(m, b, u, &C);
  const uint4* wrow = dW + ((size_t)b * m.cap + e) * n_chunks;
  const float invL = 1.0f / (float)L;
  const size_t r0 = (size_t)m.row0[bu];
  for (int c = lane; c < n_chunks; c += 64) {
    float g[8];
    unpack8(wrow[c], g);
#pragma unroll
    for (int t = 0; t < 8; ++t) g[t] *= invL;
    const uint4 o = pack8(g);
    for (int i = 0; i < L; ++i) dX[(r0 + i) * n_chunks + c] = o;
  }
}

// (Float sums that several workgroups add to go through the hardware's float atomic add: every target here is
// ordinary device memory.)
// Column sums over the pass's rows: a thread owns the 8 columns of its lane's chunk and, of the stripe's rows, those of its wave
// (every fourth); the waves' sums meet in LDS, and a stripe adds once to every column, lane by lane.  Grid (ceil(N / 512), stripes); as
// many stripes work as have 8 rows a wave.  (Four adds a column and stripe, 32 bytes between lanes: 240 rows x 3072 27 us, 35404 x 4096 110.)
constexpr int E_CS_STRIPES = 64;
__device__ __forceinline__ int cs_stripes(int rows) { return min(max((rows + 31) / 32, 1), E_CS_STRIPES); }

// acc: this thread's sums; out[512 blockIdx.x + column] += all waves'.  xch: 4 x 512 floats.  (The whole workgroup calls.)
__device__ __forceinline__ void cs_add(const float (&acc)[8], float* xch, float* out, int n) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  store8(xch + wave * 512 + lane * 8, acc);
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int t = threadIdx.x + 256 * h, col = blockIdx.x * 512 + t;
    if (col < n) unsafeAtomicAdd(out + col, (xch[t] + xch[512 + t]) + (xch[1024 + t] + xch[1536 + t]));
  }
}

// out[n] += sum over the pass's rows of G[r, n] (bias gradients).
__global__ void __launch_bounds__(256) enc_colsum_kernel(const uint4* G, int n_chunks, int pitch,
                                                         const int32_t* rows_dev, float* out) {
  __shared__ __align__(16) float xch[4 * 512];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int rows = *rows_dev, stripes = cs_stripes(rows);
  if ((int)blockIdx.y >= stripes) return;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const int step = 4 * stripes;
  for (int r = blockIdx.y * 4 + (threadIdx.x >> 6); c < n_chunks && r < rows; r += 4 * step) {   // four loads in flight
    const uint4 q0 = G[(size_t)r * pitch + c];
    const uint4 q1 = load_if(r + step < rows, G + (size_t)(r + step) * pitch + c);
    const uint4 q2 = load_if(r + 2 * step < rows, G + (size_t)(r + 2 * step) * pitch + c);
    const uint4 q3 = load_if(r + 3 * step < rows, G + (size_t)(r + 3 * step) * pitch + c);
    float g[8];
    unpack8(q0, g);
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] += g[t];
    unpack8(q1, g);
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] += g[t];
    unpack8(q2, g);
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] += g[t];
    unpack8(q3, g);
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] += g[t];
  }
  cs_add(acc, xch, out, n_chunks * 8);
}

__device__ __forceinline__ float gelu_exact(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_slope(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.3989422804014327f * __expf(-0.5f * x * x);
}

// F = GELU(U) over the pass's rows (the training pass keeps U for the slope).
__global__ void __launch_bounds__(256) enc_gelu_kernel(const uint4* U, uint4* F, int n_chunks, const int32_t* rows_dev) {
  const size_t n = (size_t)*rows_dev * n_chunks;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    float u[8];
    unpack8(U[i], u);
#pragma unroll
    for (int t = 0; t < 8; ++t) u[t] = gelu_exact(u[t]);
    F[i] = pack8(u);
  }
}

// dU = dF * GELU'(U), in place over dF, and its column sums (the bias gradient) on the way: the stripes of enc_colsum_kernel, two rows at
// a time.
__global__ void __launch_bounds__(256) enc_gelu_backward_kernel(uint4* dF, const uint4* U, int n_chunks, int pitch,
                                                                const int32_t* rows_dev, float* out) {
  __shared__ __align__(16) float xch[4 * 512];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int rows = *rows_dev, stripes = cs_stripes(rows);
  if ((int)blockIdx.y >= stripes) return;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const int step = 4 * stripes;
  for (int r = blockIdx.y * 4 + (threadIdx.x >> 6); c < n_chunks && r < rows; r += 2 * step) {
    const bool two = r + step < rows;
    const size_t at = (size_t)r * pitch + c, at2 = at + (size_t)step * pitch;
    const uint4 u0 = U[at], g0 = dF[at];
    const uint4 u1 = load_if(two, U + at2), g1 = load_if(two, dF + at2);
    float u[8], g[8];
    unpack8(u0, u);
    unpack8(g0, g);
#pragma unroll
    for (int t = 0; t < 8; ++t) g[t] *= gelu_slope(u[t]);
    uint4 o = pack8(g);
    dF[at] = o;
    unpack8(o, g);                                   // (what the products read is what is summed)
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] += g[t];
    if (two) {
      unpack8(u1, u);
      unpack8(g1, g);
#pragma unroll
      for (int t = 0; t < 8; ++t) g[t] *= gelu_slope(u[t]);
      o = pack8(g);
      dF[at2] = o;
      unpack8(o, g);
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] += g[t];
    }
  }
  cs_add(acc, xch, out, n_chunks * 8);
}

// LayerNorm backward: N = (x - mean) * rstd * gamma + beta.  out[r] = dres[r] + dx[r] with
//   g = dN * gamma;  dx = rstd * (g - mean(g) - xh * mean(g * xh)),  xh = (x - mean) * rstd.
// One wave per row as in the forward kernel: the row of X stays in registers, dN is streamed twice (the second
// time from cache).  The row's mean and rstd are left in stats[r] for the parameter gradients.
__global__ void __launch_bounds__(256) enc_norm_backward_kernel(const int32_t* rows_dev, int d, const uint4* dN,
                                                                const float* X, const float* gamma, const uint4* dres,
                                                                uint4* out, float2* stats) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= *rows_dev) return;
  const int n_chunks = d / 8;
  const float inv_d = 1.0f / (float)d;
  float x[E_KCH][8];
  float sum = 0.f;
#pragma unroll
  for (int k = 0; k < E_KCH; ++k) {
    const int c = lane + 64 * k;
    if (c < n_chunks) {
      load8(X + (size_t)r * d + c * 8, x[k]);
#pragma unroll
      for (int t = 0; t < 8; ++t) sum += x[k][t];
    }
  }
  const float mean = wave_sum(sum) * inv_d;
  float sq = 0.f;
#pragma unroll
  for (int k = 0; k < E_KCH; ++k)
    if (lane + 64 * k < n_chunks) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float dv = x[k][t] - mean;
        sq += dv * dv;
      }
    }
  const float rstd = rsqrtf(wave_sum(sq) * inv_d + E_EPS);
  if (lane == 0) stats[r] = float2{mean, rstd};
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int k = 0; k < E_KCH; ++k) {
    const int c = lane + 64 * k;
    if (c < n_chunks) {
      float g[8];
      unpack8(dN[(size_t)r * n_chunks + c], g);
      const float4 g0 = *reinterpret_cast<const float4*>(gamma + c * 8), g1 = *reinterpret_cast<const float4*>(gamma + c * 8 + 4);
      const float gm[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float xh = (x[k][t] - mean) * rstd;
        x[k][t] = xh;
        s1 += g[t] * gm[t];
        s2 += g[t] * gm[t] * xh;
      }
    }
  }
  const float m1 = wave_sum(s1) * inv_d, m2 = wave_sum(s2) * inv_d;
#pragma unroll
  for (int k = 0; k < E_KCH; ++k) {
    const int c = lane + 64 * k;
    if (c < n_chunks) {
      float g[8], o[8];
      unpack8(dN[(size_t)r * n_chunks + c], g);
      unpack8(dres[(size_t)r * n_chunks + c], o);
      const float4 g0 = *reinterpret_cast<const float4*>(gamma + c * 8), g1 = *reinterpret_cast<const float4*>(gamma + c * 8 + 4);
      const float gm[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
#pragma unroll
      for (int t = 0; t < 8; ++t) o[t] += rstd * (g[t] * gm[t] - m1 - x[k][t] * m2);
      out[(size_t)r * n_chunks + c] = pack8(o);
    }
  }
}

// dgamma[n] += sum_r dN[r, n] * xh[r, n],  dbeta[n] += sum_r dN[r, n],  xh = (X - mean[r]) * rstd[r]: column sums as in
// enc_colsum_kernel.
__global__ void __launch_bounds__(256) enc_norm_param_grad_kernel(const uint4* dN, const float* X, const float2* stats,
                                                                  int n_chunks, const int32_t* rows_dev, float* dgamma,
                                                                  float* dbeta) {
  __shared__ __align__(16) float xch[2][4 * 512];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int rows = *rows_dev, stripes = cs_stripes(rows);
  if ((int)blockIdx.y >= stripes) return;
  float ag[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, ab[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const int step = 4 * stripes;
  for (int r = blockIdx.y * 4 + (threadIdx.x >> 6); c < n_chunks && r < rows; r += 2 * step) {   // two rows in flight
    const bool two = r + step < rows;
    const int r2 = two ? r + step : r;
    const uint4 qg0 = dN[(size_t)r * n_chunks + c], qg1 = dN[(size_t)r2 * n_chunks + c];
    float g[8], x[8], x1[8];
    load8(X + ((size_t)r * n_chunks + c) * 8, x);
    load8(X + ((size_t)r2 * n_chunks + c) * 8, x1);
    const float2 st0 = stats[r], st1 = stats[r2];
    unpack8(qg0, g);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      ag[t] += g[t] * ((x[t] - st0.x) * st0.y);
      ab[t] += g[t];
    }
    if (two) {
      unpack8(qg1, g);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        ag[t] += g[t] * ((x1[t] - st1.x) * st1.y);
        ab[t] += g[t];
      }
    }
  }
  cs_add(ag, xch[0], dgamma, n_chunks * 8);
  cs_add(ab, xch[1], dbeta, n_chunks * 8);
}

// Attention backward for one entry and 512 features (same split as the forward kernel).  Per query row i the
// probabilities p[i][.] are formed again from q and k; with dP[i][j] = dO_i . v_j and
// dS[i][j] = p[i][j] (dP[i][j] - sum_j' dP[i][j'] p[i][j']):  dq_i = scale * sum_j dS[i][j] k_j;
// dk_j += scale * dS[i][j] q_i;  dv_j += p[i][j] dO_i.  dQKV has the layout of QKV.
template <int MM>          // slots per entry the registers are sized for: 4 (the usual M = 3) or Z2Z_MAX_M
__global__ void __launch_bounds__(256) enc_attention_backward_kernel(RowMap m, const uint4* QKV, const uint4* dO,
                                                                     uint4* dQKV, int lanes_per_head, float scale,
                                                                     int groups, int n_units) {
  const int lane = threadIdx.x & 63;
  const long long wid = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int g = (int)(wid % groups);
  const long long bu = wid / groups;
  if (bu >= n_units) return;
  const int n_chunks = m.d / 8;
  const int c = g * 64 + lane;
  const bool active = c < n_chunks;
  const size_t r0 = (size_t)m.row0[bu];
  const int L = m.row0[bu + 1] - m.row0[bu];
  float dk[MM][8], dv[MM][8];
#pragma unroll
  for (int j = 0; j < MM; ++j)
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      dk[j][t] = 0.f;
      dv[j][t] = 0.f;
    }
  for (int i = 0; i < L; ++i) {
    float q[8], go[8];
    unpack8(load_if(active, QKV + (r0 + i) * 3 * n_chunks + c), q);
    unpack8(load_if(active, dO + (r0 + i) * n_chunks + c), go);
    float s[MM], dp[MM];
    float smax = -INFINITY;
#pragma unroll
    for (int j = 0; j < MM; ++j) {
      s[j] = -INFINITY;
      dp[j] = 0.f;
      if (j < L) {
        float k[8], v[8];
        unpack8(load_if(active, QKV + (r0 + j) * 3 * n_chunks + n_chunks + c), k);
        unpack8(load_if(active, QKV + (r0 + j) * 3 * n_chunks + 2 * n_chunks + c), v);
        float dot = 0.f, dot2 = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          dot += q[t] * k[t];
          dot2 += go[t] * v[t];
        }
        for (int off = 1; off < lanes_per_head; off <<= 1) {
          dot += __shfl_xor(dot, off);
          dot2 += __shfl_xor(dot2, off);
        }
        s[j] = dot * scale;
        dp[j] = dot2;
        smax = fmaxf(smax, s[j]);
      }
    }
    float den = 0.f;
#pragma unroll
    for (int j = 0; j < MM; ++j) {
      s[j] = j < L ? __expf(s[j] - smax) : 0.f;
      den += s[j];
    }
    const float inv = 1.0f / den;
    float dot_pp = 0.f;
#pragma unroll
    for (int j = 0; j < MM; ++j) {
      s[j] *= inv;                                   // p[i][j]
      dot_pp += s[j] * dp[j];
    }
    float dq[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < MM; ++j) {
      if (j < L) {
        const float ds = s[j] * (dp[j] - dot_pp) * scale;
        float k[8];
        unpack8(load_if(active, QKV + (r0 + j) * 3 * n_chunks + n_chunks + c), k);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          dq[t] += ds * k[t];
          dk[j][t] += ds * q[t];
          dv[j][t] += s[j] * go[t];
        }
      }
    }
    if (active) dQKV[(r0 + i) * 3 * n_chunks + c] = pack8(dq);
  }
#pragma unroll
  for (int j = 0; j < MM; ++j) {
    if (j < L && active) {
      dQKV[(r0 + j) * 3 * n_chunks + n_chunks + c] = pack8(dk[j]);
      dQKV[(r0 + j) * 3 * n_chunks + 2 * n_chunks + c] = pack8(dv[j]);
    }
  }
}

// The gradient at the encoder's input: dE[token of row r] += dX[r] (float atomics: tokens recur), and
// dP[slot of row r] += dX[r], the latter summed per slot over a stripe of rows in registers first.
// Grid (ceil(d / 512), input_stripes): 128 stripes of the rows that exist, or stripes of 16 or of 256 (240 rows x 3072: one stripe of 256
// 149 us, 15 of 16 17; 35404 x 4096: 139 of 256 536 us, 192 of 185 659); a thread owns features f0 + lane + 64 t (t < 8) of a block of 512,
// so that the 64 lanes of one atomic instruction cover 256 consecutive bytes, and every fourth row of the stripe.
__global__ void __launch_bounds__(256) enc_input_backward_kernel(RowMap m, const uint16_t* dX, float* dE, float* dP,
                                                                 int n_units) {
  const int f0 = blockIdx.x * 512 + (threadIdx.x & 63);
  const int rows = m.row0[n_units];
  const int per = min(max((rows + 127) / 128, 16), 256);
  const int r_begin = (int)blockIdx.y * per + (threadIdx.x >> 6), r_end = min(rows, (int)(blockIdx.y + 1) * per);
  if (r_begin >= r_end) return;
  float acc[Z2Z_MAX_M][8];
#pragma unroll
  for (int j = 0; j < Z2Z_MAX_M; ++j)
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[j][t] = 0.f;
  for (int r = r_begin; r < r_end; r += 4) {
    const int rs = m.row_slot[r];
    const int i = rs & 7;
    const int bu = rs >> 3;
    const int b = bu / m.un, u = bu % m.un;
    int C;
    const int e = entry_of(m, b, u, &C);
    const int tok = min(max(m.ent_tokens[((size_t)b * m.cap + e) * m.M + i], 0), m.V - 1);
    float g[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int f = f0 + 64 * t;
      g[t] = f < m.d ? __uint_as_float((uint32_t)dX[(size_t)r * m.d + f] << 16) : 0.f;
    }
    float* er = dE + (size_t)tok * m.d;
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (f0 + 64 * t < m.d) unsafeAtomicAdd(er + f0 + 64 * t, g[t]);
#pragma unroll
    for (int j = 0; j < Z2Z_MAX_M; ++j)
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[j][t] += (i == j) ? g[t] : 0.f;
  }
  if (dP) {
#pragma unroll
    for (int j = 0; j < Z2Z_MAX_M; ++j)
      if (j < m.M) {
#pragma unroll
        for (int t = 0; t < 8; ++t)
          if (f0 + 64 * t < m.d) unsafeAtomicAdd(dP + (size_t)j * m.d + f0 + 64 * t, acc[j][t]);
      }
  }
}

__global__ void __launch_bounds__(256) enc_to_bf16_kernel(const float* in, uint16_t* out, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
    out[i] = (uint16_t)bf16_bits_rne(in[i]);
}

}  // namespace

// Row pitch of the feed-forward activations of a call that takes `units` entries per sequence, u_step a pass: the padded
// one if every pass, the last and shortest too, runs their products on kernels that take it.
static int ffn_pitch(const z2z_ctx* c, int B, int M, int units, int u_step, int d, int dff) {
  const int last = (units - 1) % u_step + 1;
  for (int u : {u_step, last})
    if (dff == 0 || !z2z_linear_takes_pitch(c, B * u * M, dff, d) || !z2z_linear_takes_pitch(c, B * u * M, d, dff)) return dff;
  return z2z_activation_pitch(dff);
}

bool z2z_hyper_encode_ok(const z2z_ctx* c, const z2z_encoder* enc) {
  const int d = c->cfg.d;
  if (c->cfg.dtype != Z2Z_BF16 || !c->fast_ready || d % 64 != 0 || d > 64 * 8 * E_KCH) return false;
  if (enc->n_heads < 1 || d % enc->n_heads != 0) return false;
  const int dh = d / enc->n_heads;
  if (dh < 8 || dh > 512 || (dh & (dh - 1)) != 0) return false;
  if (!enc->attention_only && (enc->d_ff < 64 || enc->d_ff % 64 != 0)) return false;
  return true;
}

int z2z_launch_hyper_encode(z2z_ctx* c, const void* E, const z2z_encoder* enc, void* W_hyper, const int32_t* first,
                            int32_t max_new, hipStream_t s) {
  const int B = c->cfg.B, M = c->cfg.M, cap = c->cfg.cap, d = c->cfg.d;
  if (cap == 0) return Z2Z_OK;
  const bool incremental = first || max_new > 0;
  const int units = incremental ? (max_new < 1 ? cap : (max_new < cap ? max_new : cap)) : cap;
  const int dff = enc->attention_only ? 0 : enc->d_ff;
  // (few rows: does anything of the weights stay in the memory-side cache until the next call?)
  const bool once = (size_t)enc->n_layers * ((size_t)4 * d + (size_t)2 * dff) * d * sizeof(uint16_t) > z2z_logits::kKeepBytes;
  // rows per pass: all sequences, u_step entries each, M slots per entry
  long long u_step = 0;
  size_t R_max = 0, n_units_max = 0, index_bytes = 0;
  int dffp = 0;
  auto layout = [&](long long rows) -> size_t {
    u_step = rows / ((long long)B * M);
    if (u_step < 1) u_step = 1;
    if (u_step > units) u_step = units;
    R_max = (size_t)B * (size_t)u_step * M;
    dffp = ffn_pitch(c, B, M, units, (int)u_step, d, dff);
    n_units_max = (size_t)B * (size_t)u_step;
    index_bytes = ((n_units_max + 1 + R_max) * sizeof(int32_t) + 255) & ~(size_t)255;
    // per row: the stream X and Y in fp32 (2 x 4 bytes x d), A, O (d), QKV (3d) and F (d_ff) in bf16
    return R_max * ((size_t)8 * d + ((size_t)2 * d + (size_t)3 * d + (size_t)dffp) * 2) + index_bytes;
  };
  auto room = [&](size_t need) -> int {
    if (need <= c->enc_ws_bytes) return Z2Z_OK;
    Z2Z_TRY_GROW(s);
    if (c->enc_ws) (void)hipFree(c->enc_ws);
    c->enc_ws = nullptr;
    c->enc_ws_bytes = 0;
    if (!z2z_device_malloc(&c->enc_ws, need)) return Z2Z_ENOMEM;
    c->enc_ws_bytes = need;
    return Z2Z_OK;
  };
  // (where the buffer cannot grow that far, or not at all under capture, passes of half as many rows.  What the device has refused is not asked
  // for again: every call would free the buffer that does)
  size_t need = layout(131072);
  int rc = c->enc_ws_refused && need >= c->enc_ws_refused && need > c->enc_ws_bytes ? Z2Z_ENOMEM : room(need);
  if (rc != Z2Z_OK) {
    if (rc == Z2Z_ENOMEM) c->enc_ws_refused = need;
    need = layout(65536);
    rc = room(need);
  }
  if (rc != Z2Z_OK) return rc;
  int32_t* index = reinterpret_cast<int32_t*>(c->enc_ws);
  float* X = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(c->enc_ws) + index_bytes);
  float* Y = X + R_max * d;
  uint16_t* A = reinterpret_cast<uint16_t*>(Y + R_max * d);
  uint16_t* O = A + R_max * d;
  uint16_t* QKV = O + R_max * d;
  uint16_t* F = QKV + R_max * 3 * d;

  RowMap m;
  m.size = c->st.size;
  m.ent_tokens = c->st.ent_tokens;
  m.ent_len = c->st.ent_len;
  m.first = first;
  m.last_n = (!first && max_new > 0) ? max_new : 0;
  m.B = B;
  m.V = c->cfg.V;
  m.M = M;
  m.cap = cap;
  m.d = d;
  m.row0 = index;
  m.row_slot = index + n_units_max + 1;
  const int dh = d / enc->n_heads;
  const int groups = (d + 511) / 512;
  const float scale = 1.0f / sqrtf((float)dh);
  for (int u0 = 0; u0 < units; u0 += (int)u_step) {
    m.u0 = u0;
    m.un = (int)(u0 + u_step <= units ? u_step : units - u0);
    const int n_units = B * m.un;
    const int R = n_units * M;                      // upper bound; the pass's row count is row0[n_units], on the device
    const int32_t* rows_dev = m.row0 + n_units;
    const unsigned row_blocks = (unsigned)((R + 3) / 4);
    hipLaunchKernelGGL(enc_rows_kernel, dim3(1), dim3(1024), 0, s, m, n_units);
    float* x = X;
    float* y = Y;
    bool normed = false;                            // A holds the layer's normalised input already
    bool pooled = false;
    // A dense layer that adds to the residual stream: out = in A^T + bias + residual, then the LayerNorm that follows
    // (gamma, beta -> A) or, behind the last layer, the mean over an entry's rows.  Where K is split those
    // add up the partial tiles themselves; else *fused stays false and only `out` is written.
    auto layer_out = [&](const uint16_t* in, const void* w, const float* bias, const float* residual, float* out, int K,
                         const float* gamma, const float* beta, bool* fused) -> int {
      Parts parts = {};
      *fused = false;
      const z2z_linear_pitch pitch = {dffp, dff, d};
      const bool padded = in == F && dffp != dff;
      int ret = Z2Z_OK;
      // (with more rows -- K is split there too in a narrow encoder -- a wave per row is the better LayerNorm: 6144 rows,
      // d = 256: the pass 275 us fused, 267 in launches of their own)
      if (!padded && R <= E_FEW_ROWS)
        ret = z2z_launch_linear_parts(c, in, w, R, rows_dev, d, K, &parts.partial, &parts.ksplit, s, once);
      if (ret != Z2Z_OK) return ret;
      if (parts.ksplit == 0)
        return z2z_launch_linear(c, in, w, bias, residual, 0, out, R, rows_dev, d, K, s, true, padded ? &pitch : nullptr, once);
      parts.R = R;
      parts.bias = bias;
      parts.residual = residual;
      *fused = true;
      if (gamma)
        hipLaunchKernelGGL(enc_row_norm_kernel<false>, dim3((unsigned)R), dim3(E_ROW_THREADS), 0, s, m, nullptr, nullptr, parts, out,
                           A, gamma, beta, n_units);
      else
        hipLaunchKernelGGL(enc_sum_pool_kernel, dim3((unsigned)n_units, (unsigned)((d + 255) / 256)), dim3((unsigned)(64 * M)), 0, s, m,
                           parts, reinterpret_cast<uint16_t*>(W_hyper), incremental ? 0 : 1);
      return Z2Z_OK;
    };
    for (int l = 0; l < enc->n_layers; ++l) {
      const z2z_encoder_layer& lay = enc->layers[l];
      const z2z_encoder_layer* next = l + 1 < enc->n_layers ? &enc->layers[l + 1] : nullptr;
      if (l == 0 && R <= E_FEW_ROWS) {              // (few rows: a workgroup each, 24 entries, 52 rows: 14 -> 5 us)
        hipLaunchKernelGGL(enc_row_norm_kernel<true>, dim3((unsigned)R), dim3(E_ROW_THREADS), 0, s, m,
                           reinterpret_cast<const uint16_t*>(E), reinterpret_cast<const uint16_t*>(enc->pos), Parts{}, x, A,
                           lay.ln1_g, lay.ln1_b, n_units);
      } else if (l == 0) {
        hipLaunchKernelGGL(enc_norm_kernel<true>, dim3(row_blocks), dim3(256), 0, s, m,
                           reinterpret_cast<const uint4*>(E), reinterpret_cast<const uint4*>(enc->pos), x,
                           reinterpret_cast<uint4*>(A), lay.ln1_g, lay.ln1_b, n_units);
      } else if (!normed) {
        hipLaunchKernelGGL(enc_norm_kernel<false>, dim3(row_blocks), dim3(256), 0, s, m, nullptr, nullptr, x,
                           reinterpret_cast<uint4*>(A), lay.ln1_g, lay.ln1_b, n_units);
      }
      rc = z2z_launch_linear(c, A, lay.w_qkv, lay.b_qkv, nullptr, 0, QKV, R, rows_dev, 3 * d, d, s, false, nullptr, once);
      if (rc != Z2Z_OK) return rc;
      const long long att_waves = (long long)n_units * groups;
      hipLaunchKernelGGL(M <= 4 ? enc_attention_kernel<4> : enc_attention_kernel<Z2Z_MAX_M>, dim3((unsigned)((att_waves + 3) / 4)), dim3(256), 0, s, m,
                         reinterpret_cast<const uint4*>(QKV), reinterpret_cast<uint4*>(O), dh / 8, scale, groups,
                         n_units);
      bool fused = false;
      if (enc->attention_only) {
        rc = layer_out(O, lay.w_o, lay.b_o, x, y, d, next ? next->ln1_g : nullptr, next ? next->ln1_b : nullptr, &fused);
        if (rc != Z2Z_OK) return rc;
        float* t = x;
        x = y;
        y = t;
      } else {
        rc = layer_out(O, lay.w_o, lay.b_o, x, y, d, lay.ln2_g, lay.ln2_b, &fused);
        if (rc != Z2Z_OK) return rc;
        if (!fused)
          hipLaunchKernelGGL(enc_norm_kernel<false>, dim3(row_blocks), dim3(256), 0, s, m, nullptr, nullptr, y,
                             reinterpret_cast<uint4*>(A), lay.ln2_g, lay.ln2_b, n_units);
        const z2z_linear_pitch to_wide = {d, d, dffp};
        rc = z2z_launch_linear(c, A, lay.w_1, lay.b_1, nullptr, 1, F, R, rows_dev, dff, d, s, false,
                               dffp != dff ? &to_wide : nullptr, once);
        if (rc != Z2Z_OK) return rc;
        rc = layer_out(F, lay.w_2, lay.b_2, y, x, dff, next ? next->ln1_g : nullptr, next ? next->ln1_b : nullptr, &fused);
        if (rc != Z2Z_OK) return rc;
      }
      normed = fused && next;
      pooled = fused && !next;
    }
    if (!pooled)
      hipLaunchKernelGGL(enc_pool_kernel, dim3((unsigned)((n_units + 3) / 4)), dim3(256), 0, s, m, x,
                         reinterpret_cast<uint4*>(W_hyper), n_units, incremental ? 0 : 1);
  }
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

namespace {

struct LayerSave {                   // what the training pass keeps of one layer: the stream (Xin, Y) [rows, d] fp32,
  float *Xin, *Y;                    // the operands of the matrix products [rows, .] bf16
  uint16_t *A, *QKV, *O, *N2, *U, *F;
};

void colsum_to(const void* G, int N, int ld, const int32_t* rows_dev, float* out, hipStream_t s) {
  hipLaunchKernelGGL(enc_colsum_kernel, dim3((N / 8 + 63) / 64, E_CS_STRIPES), dim3(256), 0, s,
                     reinterpret_cast<const uint4*>(G), N / 8, ld / 8, rows_dev, out);
}

unsigned input_stripes(int R) {
  const int most = (R + 15) / 16, of256 = (R + 255) / 256;
  return (unsigned)(of256 > 128 ? of256 : (most < 128 ? most : 128));
}

unsigned flat_grid(size_t n) {
  const size_t blocks = (n + 255) / 256;
  return (unsigned)(blocks < 1 ? 1 : (blocks > 65536 ? 65536 : blocks));
}

}  // namespace

// mode 0: forward (rows kept) + backward, pass by pass; mode 1: the forward alone, W_hyper written and the rows
// left in the work space; mode 2: the backward alone on the rows mode 1 left.  Modes 1 and 2 need all slot rows
// in one pass.
int z2z_launch_hyper_encode_train(z2z_ctx* c, int mode, const void* E, const z2z_encoder* enc, void* W_hyper,
                                  const void* dW_hyper, const z2z_encoder* grad, float* dE, hipStream_t s) {
  const int B = c->cfg.B, M = c->cfg.M, cap = c->cfg.cap, d = c->cfg.d;
  if (cap == 0) return Z2Z_OK;
  if (mode != 0 && (long long)B * cap * M > 65536) return Z2Z_EUNSUPPORTED;
  const int nl = enc->n_layers;
  const bool ffn = !enc->attention_only;
  const int dff = ffn ? enc->d_ff : 0;
  long long u_step = 65536 / ((long long)B * M);
  if (u_step < 1) u_step = 1;
  if (u_step > cap) u_step = cap;
  const size_t R_max = (size_t)B * (size_t)u_step * M;
  const int dffp = ffn_pitch(c, B, M, cap, (int)u_step, d, dff);
  const size_t n_units_max = (size_t)B * (size_t)u_step;
  const size_t index_bytes = ((n_units_max + 1 + R_max) * sizeof(int32_t) + 255) & ~(size_t)255;
  const size_t pos_bytes = ((size_t)Z2Z_MAX_M * d * sizeof(float) + 255) & ~(size_t)255;
  // in units of bf16 elements (an fp32 element counts as two): per layer what LayerSave names (Xin and Y fp32);
  // the last layer's output (fp32); the running gradients dX dY dN dO (d each), dQKV (3d), dF (d_ff)
  const size_t per_layer = R_max * ((size_t)10 * d + (size_t)2 * dffp);
  const size_t elems = (size_t)nl * per_layer + R_max * ((size_t)7 * d + dffp) + R_max * 2 * d;
  const size_t nb_bytes = (R_max * sizeof(float2) + 255) & ~(size_t)255;   // mean and rstd of every row of a LayerNorm
  const size_t need = index_bytes + pos_bytes + nb_bytes + elems * 2;
  if (need > ((size_t)200 << 30)) return Z2Z_ENOMEM;
  // the rows a mode-1 call left are those of this encoder's shape only if the layout is the same
  if (mode == 2 && (!c->enc_kept || c->enc_kept_need != need || c->enc_kept_E != E)) return Z2Z_EINVAL;
  c->enc_kept = false;
  if (need > c->enc_bwd_ws_bytes) {
    Z2Z_TRY_GROW(s);
    if (c->enc_bwd_ws) (void)hipFree(c->enc_bwd_ws);
    c->enc_bwd_ws = nullptr;
    c->enc_bwd_ws_bytes = 0;
    if (!z2z_device_malloc(&c->enc_bwd_ws, need)) return Z2Z_ENOMEM;
    c->enc_bwd_ws_bytes = need;
  }
  unsigned char* base = reinterpret_cast<unsigned char*>(c->enc_bwd_ws);
  int32_t* index = reinterpret_cast<int32_t*>(base);
  float* dP = reinterpret_cast<float*>(base + index_bytes);
  float2* ln_stats = reinterpret_cast<float2*>(base + index_bytes + pos_bytes);
  uint16_t* p = reinterpret_cast<uint16_t*>(base + index_bytes + pos_bytes + nb_bytes);
  auto take = [&](size_t n) {
    uint16_t* r = p;
    p += n;
    return r;
  };
  auto take_f32 = [&](size_t n) { return reinterpret_cast<float*>(take(2 * n)); };   // (every size is a multiple of 64 elements)
  LayerSave sv[Z2Z_MAX_ENCODER_LAYERS];
  for (int l = 0; l < nl; ++l) {
    sv[l].Xin = take_f32(R_max * d);
    sv[l].Y = take_f32(R_max * d);
    sv[l].A = take(R_max * d);
    sv[l].QKV = take(R_max * 3 * d);
    sv[l].O = take(R_max * d);
    sv[l].N2 = take(R_max * d);
    sv[l].U = take(R_max * (size_t)dffp);
    sv[l].F = take(R_max * (size_t)dffp);
  }
  float* Xout = take_f32(R_max * d);
  uint16_t* dX = take(R_max * d);
  uint16_t* dY = take(R_max * d);
  uint16_t* dN = take(R_max * d);
  uint16_t* dO = take(R_max * d);
  uint16_t* dQKV = take(R_max * 3 * d);
  uint16_t* dF = take(R_max * (size_t)dffp);

  RowMap m;
  m.size = c->st.size;
  m.ent_tokens = c->st.ent_tokens;
  m.ent_len = c->st.ent_len;
  m.first = nullptr;
  m.last_n = 0;
  m.B = B;
  m.V = c->cfg.V;
  m.M = M;
  m.cap = cap;
  m.d = d;
  m.row0 = index;
  m.row_slot = index + n_units_max + 1;
  const int dh = d / enc->n_heads;
  const int groups = (d + 511) / 512;
  const float scale = 1.0f / sqrtf((float)dh);

  // vector gradients are sums over all passes: cleared once, added to by every pass
  Pieces zero = {};
  auto clear = [&](const float* q, int n) {
    zero.p[zero.n] = const_cast<float*>(q);
    zero.len[zero.n++] = n;
  };
  for (int l = 0; l < nl && mode != 1; ++l) {
    const z2z_encoder_layer& g = grad->layers[l];
    clear(g.ln1_g, d);
    clear(g.ln1_b, d);
    clear(g.b_qkv, 3 * d);
    clear(g.b_o, d);
    if (ffn) {
      clear(g.ln2_g, d);
      clear(g.ln2_b, d);
      clear(g.b_1, dff);
      clear(g.b_2, d);
    }
  }
  if (mode != 1) {
    clear(dP, Z2Z_MAX_M * d);
    hipLaunchKernelGGL(enc_fill_kernel, dim3(64, (unsigned)zero.n), dim3(256), 0, s, zero);
  }

  int rc;
#define Z2Z_TRY_RC(expr)      \
  do {                        \
    rc = (expr);              \
    if (rc != Z2Z_OK) return rc; \
  } while (0)

  // pitches of the products into and out of the feed-forward width
  const z2z_linear_pitch into = {d, d, dffp}, out_of = {dffp, dff, d};
  const z2z_linear_pitch *to_wide = dffp != dff ? &into : nullptr, *from_wide = dffp != dff ? &out_of : nullptr;
  int pass = 0;
  for (int u0 = 0; u0 < cap; u0 += (int)u_step, ++pass) {
    m.u0 = u0;
    m.un = (int)(u0 + u_step <= cap ? u_step : cap - u0);
    const int n_units = B * m.un;
    const int R = n_units * M;                       // upper bound; the real count is on the device
    const int32_t* rows_dev = m.row0 + n_units;
    const unsigned row_blocks = (unsigned)((R + 3) / 4);
    if (mode != 2) hipLaunchKernelGGL(enc_rows_kernel, dim3(1), dim3(1024), 0, s, m, n_units);

    // ---- forward, keeping every layer's intermediate rows ----
    for (int l = 0; l < nl && mode != 2; ++l) {
      const z2z_encoder_layer& lay = enc->layers[l];
      const LayerSave& v = sv[l];
      float* next = l + 1 < nl ? sv[l + 1].Xin : Xout;
      if (l == 0)
        hipLaunchKernelGGL(enc_norm_kernel<true>, dim3(row_blocks), dim3(256), 0, s, m,
                           reinterpret_cast<const uint4*>(E), reinterpret_cast<const uint4*>(enc->pos), v.Xin,
                           reinterpret_cast<uint4*>(v.A), lay.ln1_g, lay.ln1_b, n_units);
      else
        hipLaunchKernelGGL(enc_norm_kernel<false>, dim3(row_blocks), dim3(256), 0, s, m, nullptr, nullptr, v.Xin,
                           reinterpret_cast<uint4*>(v.A), lay.ln1_g, lay.ln1_b, n_units);
      Z2Z_TRY_RC(z2z_launch_linear(c, v.A, lay.w_qkv, lay.b_qkv, nullptr, 0, v.QKV, R, rows_dev, 3 * d, d, s));
      const long long att_waves = (long long)n_units * groups;
      hipLaunchKernelGGL(M <= 4 ? enc_attention_kernel<4> : enc_attention_kernel<Z2Z_MAX_M>, dim3((unsigned)((att_waves + 3) / 4)), dim3(256), 0, s, m,
                         reinterpret_cast<const uint4*>(v.QKV), reinterpret_cast<uint4*>(v.O), dh / 8, scale, groups,
                         n_units);
      float* y = ffn ? v.Y : next;
      Z2Z_TRY_RC(z2z_launch_linear(c, v.O, lay.w_o, lay.b_o, v.Xin, 0, y, R, rows_dev, d, d, s, true));
      if (ffn) {
        hipLaunchKernelGGL(enc_norm_kernel<false>, dim3(row_blocks), dim3(256), 0, s, m, nullptr, nullptr, v.Y,
                           reinterpret_cast<uint4*>(v.N2), lay.ln2_g, lay.ln2_b, n_units);
        Z2Z_TRY_RC(z2z_launch_linear(c, v.N2, lay.w_1, lay.b_1, nullptr, 0, v.U, R, rows_dev, dff, d, s, false, to_wide));
        hipLaunchKernelGGL(enc_gelu_kernel, dim3(flat_grid((size_t)R * dffp / 8)), dim3(256), 0, s,
                           reinterpret_cast<const uint4*>(v.U), reinterpret_cast<uint4*>(v.F), dffp / 8, rows_dev);
        Z2Z_TRY_RC(z2z_launch_linear(c, v.F, lay.w_2, lay.b_2, v.Y, 0, next, R, rows_dev, d, dff, s, true, from_wide));
      }
    }

    if (mode == 1) {
      hipLaunchKernelGGL(enc_pool_kernel, dim3((unsigned)((n_units + 3) / 4)), dim3(256), 0, s, m, Xout,
                         reinterpret_cast<uint4*>(W_hyper), n_units, 1);
      continue;
    }

    // ---- backward ----
    hipLaunchKernelGGL(enc_pool_backward_kernel, dim3((unsigned)((n_units + 3) / 4)), dim3(256), 0, s, m,
                       reinterpret_cast<const uint4*>(dW_hyper), reinterpret_cast<uint4*>(dX), n_units);
    auto norm_backward = [&](const uint16_t* dn, const float* x, const float* gamma, const uint16_t* dres,
                             uint16_t* out, const float* dgamma, const float* dbeta) {
      hipLaunchKernelGGL(enc_norm_backward_kernel, dim3(row_blocks), dim3(256), 0, s, rows_dev, d,
                         reinterpret_cast<const uint4*>(dn), x, gamma,
                         reinterpret_cast<const uint4*>(dres), reinterpret_cast<uint4*>(out), ln_stats);
      hipLaunchKernelGGL(enc_norm_param_grad_kernel, dim3((d / 8 + 63) / 64, E_CS_STRIPES), dim3(256), 0, s,
                         reinterpret_cast<const uint4*>(dn), x, ln_stats, d / 8, rows_dev,
                         const_cast<float*>(dgamma), const_cast<float*>(dbeta));
    };
    for (int l = nl - 1; l >= 0; --l) {
      const z2z_encoder_layer& lay = enc->layers[l];
      const z2z_encoder_layer& g = grad->layers[l];
      const LayerSave& v = sv[l];
      const void* acc = nullptr;                     // weight gradients of later passes add to the earlier ones
      uint16_t* dy = dX;                             // gradient at Y (attention layers: the layer's output)
      if (ffn) {
        colsum_to(dX, d, d, rows_dev, const_cast<float*>(g.b_2), s);
        Z2Z_TRY_RC(z2z_launch_linear_input(c, dX, d, lay.w_2, dff, d, nullptr, dF, dffp, R, rows_dev, dff, d, s));
        acc = pass > 0 ? g.w_2 : nullptr;
        Z2Z_TRY_RC(z2z_launch_linear_weight(c, dX, d, v.F, dffp, R, rows_dev, acc, const_cast<void*>(g.w_2), d, dff, s));
        hipLaunchKernelGGL(enc_gelu_backward_kernel, dim3((dff / 8 + 63) / 64, E_CS_STRIPES), dim3(256), 0, s,
                           reinterpret_cast<uint4*>(dF), reinterpret_cast<const uint4*>(v.U), dff / 8, dffp / 8, rows_dev,
                           const_cast<float*>(g.b_1));
        acc = pass > 0 ? g.w_1 : nullptr;
        Z2Z_TRY_RC(z2z_launch_linear_weight(c, dF, dffp, v.N2, d, R, rows_dev, acc, const_cast<void*>(g.w_1), dff, d, s));
        Z2Z_TRY_RC(z2z_launch_linear_input(c, dF, dffp, lay.w_1, d, dff, nullptr, dN, d, R, rows_dev, d, dff, s));
        norm_backward(dN, v.Y, lay.ln2_g, dX, dY, g.ln2_g, g.ln2_b);
        dy = dY;
      }
      colsum_to(dy, d, d, rows_dev, const_cast<float*>(g.b_o), s);
      Z2Z_TRY_RC(z2z_launch_linear_input(c, dy, d, lay.w_o, d, d, nullptr, dO, d, R, rows_dev, d, d, s));
      acc = pass > 0 ? g.w_o : nullptr;
      Z2Z_TRY_RC(z2z_launch_linear_weight(c, dy, d, v.O, d, R, rows_dev, acc, const_cast<void*>(g.w_o), d, d, s));
      const long long att_waves = (long long)n_units * groups;
      if (M <= 4)
        hipLaunchKernelGGL(enc_attention_backward_kernel<4>, dim3((unsigned)((att_waves + 3) / 4)), dim3(256), 0, s, m,
                           reinterpret_cast<const uint4*>(v.QKV), reinterpret_cast<const uint4*>(dO),
                           reinterpret_cast<uint4*>(dQKV), dh / 8, scale, groups, n_units);
      else
        hipLaunchKernelGGL(enc_attention_backward_kernel<Z2Z_MAX_M>, dim3((unsigned)((att_waves + 3) / 4)), dim3(256), 0,
                           s, m, reinterpret_cast<const uint4*>(v.QKV), reinterpret_cast<const uint4*>(dO),
                           reinterpret_cast<uint4*>(dQKV), dh / 8, scale, groups, n_units);
      colsum_to(dQKV, 3 * d, 3 * d, rows_dev, const_cast<float*>(g.b_qkv), s);
      acc = pass > 0 ? g.w_qkv : nullptr;
      Z2Z_TRY_RC(z2z_launch_linear_weight(c, dQKV, 3 * d, v.A, d, R, rows_dev, acc, const_cast<void*>(g.w_qkv), 3 * d, d, s));
      Z2Z_TRY_RC(z2z_launch_linear_input(c, dQKV, 3 * d, lay.w_qkv, d, 3 * d, nullptr, dN, d, R, rows_dev, d, 3 * d, s));
      norm_backward(dN, v.Xin, lay.ln1_g, dy, dX, g.ln1_g, g.ln1_b);
    }
    hipLaunchKernelGGL(enc_input_backward_kernel, dim3((d + 511) / 512, input_stripes(R)), dim3(256), 0, s, m, dX, dE,
                       enc->pos ? dP : nullptr, n_units);
  }
#undef Z2Z_TRY_RC
  if (mode == 1) {
    Z2Z_HIP_TRY(hipGetLastError());
    c->enc_kept = true;
    c->enc_kept_need = need;
    c->enc_kept_E = E;
    return Z2Z_OK;
  }
  if (enc->pos)
    hipLaunchKernelGGL(enc_to_bf16_kernel, dim3(flat_grid((size_t)M * d)), dim3(256), 0, s, dP,
                       reinterpret_cast<uint16_t*>(const_cast<void*>(grad->pos)), (size_t)M * d);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

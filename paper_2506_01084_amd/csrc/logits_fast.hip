// extended_logits, bf16 MFMA kernel for gfx950 (d a multiple of 64), one wave per SIMD.
//
// Workgroup tile 256 (vocabulary rows, MFMA "A") x 256 (hidden rows, MFMA "B"), 4 waves in a 2 x 2 grid,
// each wave 128 x 128 = 8 x 8 blocks of v_mfma_f32_16x16x32_bf16 (256 accumulator registers per lane):
// per 32-deep k-step a wave reads 16 operand fragments from LDS for 64 MFMAs.  What bounds it is the power limit
// (the clock falls to 1.5-1.8 GHz under it), so the form of the matrix instruction counts: 32 x 32 x 16 moves the
// accumulators once per 16 of K, 16 x 16 x 32 once per 32, for the same operand bytes.  32768 x 4096 outputs, K = 128256:
// 25.4 ms with 32 x 32 x 16 in this schedule, 23.2 with 16 x 16 x 32 (27.2 with 32 x 32 x 16 and one hand-over per slab).
//
// K advances in slabs of 64 elements (128 bytes per row, two k-steps): the global -> LDS stream moves
// whole 128-byte lines, which it does markedly faster than half lines (measured on a bare streaming
// kernel: 14-22 TB/s against 12-15 TB/s out of L2).  Both operand tiles of a slab (2 x 32 KiB) go straight
// from global memory into LDS (16-byte global_load ... lds), two stages.  With one wave per SIMD all overlap is
// inside the instruction stream.  A slab's 128 MFMAs are slots, and between them go, each at a slot of its own
// (Schedule below):
//   - the 16 fragment reads of the second k-step, then a barrier (everybody holds the rest of slab s in registers:
//     its stage is free) and the 16 requests for slab s+2, six MFMAs apart;
//   - late in the second k-step a wait for slab s+1 and a second barrier (it has landed for everybody), then the 16
//     fragment reads of its first k-step.
// Freeing the stage that early gives a request more than a slab's time to land; with one barrier per slab for both
// purposes the same product takes 26.0-26.4 ms.  Taking the waits or the barriers out changes nothing any more (23.1-23.4
// ms, in a build for timing): fewer stall cycles are answered by a lower clock.  Requests closer together are slower (every
// 3 MFMAs 25.3 ms, every 4 24.8, 5 24.4, 6 24.1 in one run), and so are the fragment reads spread over twice the slots.
// The stream runs on across the vocabulary tiles of a strip.
//
// LDS layout of an operand tile: row r = 128 bytes = 8 chunks of 16 B; chunk c is stored at position
// c ^ ((r >> 1) & 7).  The LDS has 64 four-byte banks and serves a 16-byte-per-lane read 16 lanes at a
// time; an MFMA operand read has 16 consecutive lanes on 16 consecutive rows at one logical chunk, whose
// bank group is (r & 1) * 8 + position -- all 16 distinct with this swizzle.
//
// Gradient products contract over what their operands have as rows (dW = dY^T X, dX = dY W): such an operand is read as it
// is, K-major.  A slab is then 64 rows of 512 bytes (the tile's 256 columns), two whole rows a request, and a fragment
// comes out of LDS by transposing reads (ds_read_b64_tr_b16: 16 lanes read 4 rows x 16 columns, a lane gets 4 rows of one column), two
// for one plain read and the same bytes.  The 32-byte piece b of row k is stored at b ^ f(k), f = 3 low bits out of k's bits
// 0, 1 and 3: the 8 pieces that 32 lanes read at a time are on different banks.  Rows behind the last one read as zeros by the buffer
// descriptor's range, so that nothing is copied or padded.  One read per MFMA, its address in a register of its own (two per MFMA with an
// addition each: dW 20 % slower, dX 8 %).  32768 x 4096 over 128256 and 128256 x 4096 over 32768: 22.0 and 23.3 ms, against 22.4 and 22.2 on
// transposed copies that took 3.6 ms to make; a training step of 8 x 4096 tokens 169.3 -> 164.6 ms, 1 x 65 tokens, d = 3072 4.2 -> 2.4 (with the cut
// along K).
//
// In the 16 x 16 result block a lane holds 4 vocabulary entries of one hidden row (of 8 rows and 32 entries each in the
// whole tile), so the running (max, sum-exp, argmax) of the joint softmax (zip2zip paper, section 2.3, step 8) lives in
// registers and crosses lanes once per strip.
#include "logits_common.h"

#include <utility>

namespace {

using namespace z2z_logits;

constexpr int FT = 256;                   // tile edge, vocabulary and hidden rows
constexpr int F_SLAB = 128;               // bytes per row per K slab (64 bf16)
constexpr int F_OPER = FT * F_SLAB;       // one operand tile of one slab: 32 KiB
constexpr int F_STAGE = 2 * F_OPER;       // A + B
constexpr int F_LDS_STAGES = 2 * F_STAGE; // 128 KiB
constexpr int F_LDS = F_LDS_STAGES + FT * (int)(sizeof(Triple) + sizeof(Draw));     // + what the waves exchange at the end of a strip
constexpr int F_THREADS = 256;
// with the hyper part along: items ahead of every sequence's, and sizes (of up to F_HYP_SEQS of them), sums of the four waves
constexpr int F_HYP_SEQS = 2048;
constexpr int F_HYP_LDS = F_LDS + (2 * F_HYP_SEQS + 4) * (int)sizeof(int32_t);
static_assert(F_HYP_LDS <= 160 * 1024 && F_HYP_SEQS <= 64 * 64 && F_LDS % 16 == 0, "");
constexpr int F_N = 8;                    // MFMA blocks of a wave along either side (128 x 128)
constexpr int F_PAIRS = 8;                // request pairs (8 rows of A + 8 rows of B) per wave and slab
constexpr int F_SLOTS = 2 * F_N * F_N;    // MFMAs of a wave per slab
constexpr int F_KROW = 2 * FT;            // bytes of a row of a K-major operand's tile

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;

// What goes out after which MFMA of a slab (barriers: ahead of it).
template <bool TW, bool TH>
struct Schedule {
  static constexpr int reads = F_N * (1 + TW) + F_N * (1 + TH);      // of a k-step: 16 fragments, those of a K-major operand in two
  static constexpr bool long_reads = reads > 16;
  static constexpr int read2 = 0;                              // the second k-step's reads, one per MFMA
  static constexpr int free_ = read2 + reads + 8;              // barrier: slab s is in registers
  static constexpr int request = free_ + 2;                    // 16 requests for slab s+2 ...
  static constexpr int request_every = long_reads ? 5 : 6;     // ... this far apart
  static constexpr int landed = F_SLOTS - reads - 2;           // wait + barrier: slab s+1 is there
  static constexpr int read1 = landed;                         // its first k-step's reads, one per MFMA
  static constexpr int out_at_landed = (landed - request + request_every - 1) / request_every;     // requests out ahead of that wait
  static_assert(request + 15 * request_every < F_SLOTS && read1 + reads <= F_SLOTS && landed > F_SLOTS / 2 && out_at_landed <= 2 * F_PAIRS, "");
  // read e: fragment (in the order the MFMAs first need them: b0, a0, b1 .. b7, a1 .. a7) and half
  static constexpr bool is_a(int n) { return n == 1 || n > F_N; }
  static constexpr int parts(int n) { return 1 + (is_a(n) ? TW : TH); }
  static constexpr int fragment(int e) {
    int n = 0;
    while (e >= parts(n)) e -= parts(n++);
    return n;
  }
  static constexpr int half(int e) {
    int n = 0;
    while (e >= parts(n)) e -= parts(n++);
    return e;
  }
};
static_assert(Schedule<false, false>::free_ == 24 && Schedule<false, false>::request == 26 && Schedule<false, false>::landed == 110, "");

// f(0) ... f(N - 1) with the index a constant.
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// acc += a * b, or a * b where nothing has been accumulated yet.  Spelled as an instruction: left to the compiler the
// accumulators are copied about (it knows 16 x 16 blocks of four registers, and allots them anew between the uses),
// and MFMAs drift across the barriers and requests between which they were put.  The compiler does not know then that an
// MFMA's result takes its time: see wait_for_mfma.
template <bool FIRST>
__device__ __forceinline__ void mfma(f32x4& acc, const uint4& a, const uint4& b) {
  if (FIRST)
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(__builtin_bit_cast(bf16x8, a)), "v"(__builtin_bit_cast(bf16x8, b)));
  else
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(__builtin_bit_cast(bf16x8, a)), "v"(__builtin_bit_cast(bf16x8, b)));
}

// Ahead of the first read of an accumulator: more wait states than any MFMA's result needs.
__device__ __forceinline__ void wait_for_mfma() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

// Waves of the workgroup meet.  (Not __syncthreads, which waits for all outstanding requests as well.)
__device__ __forceinline__ void barrier_after_lds() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Half of a fragment out of a K-major operand: four rows of a column.
template <int OFFSET, int HALF>
__device__ __forceinline__ void read_transposed(uint4& f, uint32_t at) {
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  const uint2 v = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(uintptr_t)(at + OFFSET)));
  if (HALF == 0) {
    f.x = v.x;
    f.y = v.y;
  } else {
    f.z = v.x;
    f.w = v.y;
  }
}

// Descriptor of the rows from p on, of which `rows` exist (none: an empty range); p is `col` bytes into its row.
__device__ __forceinline__ u32x4 k_rows_rsrc(const unsigned char* p, int rows, size_t pitch, int col) {
  const int n = min(max(rows, 0), 64);
  const uint32_t range = n > 0 ? (uint32_t)n * (uint32_t)pitch - (uint32_t)col : 0u;
  const uint64_t at = (uint64_t)p;
  return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at), (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(at >> 32) & 0xFFFFu)),
               (uint32_t)__builtin_amdgcn_readfirstlane((int)range), 0x00020000u};
}

constexpr int vmcnt_imm(int n) { return (n & 0xF) | ((n >> 4) << 14) | 0x0F70; }

// 16 bytes per lane, global -> LDS without passing through registers: address = 64-bit scalar base +
// 32-bit per-lane offset; the LDS address is the wave-uniform byte offset in M0 plus 16 * lane.  Inline
// assembly on purpose: the compiler cannot tell the LDS stages apart and would make every LDS read wait
// for all outstanding direct loads.  Completion is awaited explicitly (s_waitcnt vmcnt) before the
// barrier that publishes a stage.  One wait state is required between the write of M0 and its use.
// M0 is written as stage base + constant in one scalar instruction: with one wave per SIMD every
// instruction issued between two MFMAs counts, and the request stream is the bulk of them.
template <int LDS_IMM>
__device__ __forceinline__ void load16_to_lds(const unsigned char* base, uint32_t lane_offset, uint32_t lds_stage_base) {
  asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(lane_offset), "s"(base), "s"(lds_stage_base), "n"(LDS_IMM)
               : "memory", "scc");   // M0 is reserved: the compiler keeps nothing in it across statements
}

// The same through a buffer descriptor: lanes at or beyond its range put zeros into LDS.
template <int LDS_IMM>
__device__ __forceinline__ void load16_to_lds(const u32x4& rsrc, uint32_t lane_offset, uint32_t lds_stage_base) {
  asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(lane_offset), "s"(rsrc), "s"(lds_stage_base), "n"(LDS_IMM)
               : "memory", "scc");
}

__device__ __forceinline__ uint32_t lds_offset_of(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// Position j of XCD xcd's list of work -> (row tile, strip) for the base part and dense layers; false behind its end.
// Workgroup ids go round-robin over the 8 XCDs, and the 32 workgroups of one take consecutive positions, so what is
// consecutive shares operand tiles through the XCD's L2.  One side of the output, P tiles (map_p_rows: the row tiles,
// otherwise the strips), is walked in blocks of map_lp, dealt out map_xp ways; inside a block all Q of the other side's that are this XCD's
// (q mod map_xq) follow: 32 workgroups work on map_lp x 32 / map_lp outputs, and all of them on 16 x 16 (the memory-side cache
// serves an operand tile to several XCDs).  The P tiles behind whole blocks of map_lp * map_xp go, with all of Q, in eight
// equal runs, so that the XCDs' lists differ by a run's rounding.  Lists without holes, in sizes that the device works
// out itself: the row count may be known there only.
// `more` items of another kind lie behind the P tiles' last and are dealt out with them: *extra is the index of one of those, else -1.
__device__ __forceinline__ bool locate_base(const LogitsArgs& a, int row_tiles, int xcd, int j, int* rt, int* st, int more = 0, int* extra = nullptr) {
  const int P = a.map_p_rows ? row_tiles : a.n_strips, Q = a.map_p_rows ? a.n_strips : row_tiles;
  const int xpi = xcd % a.map_xp, xqi = xcd / a.map_xp;
  const int blocks = P / (a.map_lp * a.map_xp);                    // whole blocks of each XCD along P
  const int own_q = (Q - xqi + a.map_xq - 1) / a.map_xq;
  const int main_items = blocks * a.map_lp * own_q;
  int pi, qi;
  if (extra) *extra = -1;
  if (j < main_items) {
    const int w = j / a.map_lp, blk = w / own_q;
    pi = (blk * a.map_xp + xpi) * a.map_lp + (j - w * a.map_lp);
    qi = (w - blk * own_q) * a.map_xq + xqi;
  } else {
    const int p0 = blocks * a.map_lp * a.map_xp, T = P - p0, total = T * Q + more;
    const int t = j - main_items + (int)((long long)total * xcd / 8);
    if (t >= (int)((long long)total * (xcd + 1) / 8)) return false;
    if (extra) {
      *extra = t < T * Q ? -1 : t - T * Q;
      if (t >= T * Q) return true;
    }
    qi = t / T;
    pi = p0 + (t - qi * T);
  }
  *rt = a.map_p_rows ? pi : qi;
  *st = a.map_p_rows ? qi : pi;
  return true;
}

// Length of that list.
__host__ __device__ __forceinline__ int list_length(const LogitsArgs& a, int row_tiles, int xcd) {
  const int P = a.map_p_rows ? row_tiles : a.n_strips, Q = a.map_p_rows ? a.n_strips : row_tiles;
  const int blocks = P / (a.map_lp * a.map_xp);
  const int own_q = (Q - xcd / a.map_xp + a.map_xq - 1) / a.map_xq;
  const long long total = (long long)(P - blocks * a.map_lp * a.map_xp) * Q;
  return blocks * a.map_lp * own_q + (int)(total * (xcd + 1) / 8) - (int)(total * xcd / 8);
}

// The lengths of an XCD's list and of the longest.  (On the device every lane works out one of them: the whole wave calls.)
__host__ __device__ __forceinline__ void list_lengths(const LogitsArgs& a, int row_tiles, int xcd, int* own, int* longest) {
#ifdef __HIP_DEVICE_COMPILE__
  int len = list_length(a, row_tiles, (int)(threadIdx.x & 7));
  *own = __builtin_amdgcn_readlane(len, xcd);
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) len = max(len, __shfl_xor(len, o));
  *longest = __builtin_amdgcn_readfirstlane(len);
#else
  *own = list_length(a, row_tiles, xcd);
  *longest = 0;
  for (int x = 0; x < 8; ++x) {
    const int len = list_length(a, row_tiles, x);
    *longest = *longest < len ? len : *longest;
  }
#endif
}

// A dense layer's last round.  The 32 workgroups of an XCD take 32 output tiles of its list at a time; the `rem` tiles that are
// left may be too few for them, and then every one of those is cut along K into `ways` parts of `per` slabs: position
// full + part * rem + t is part `part` of tile full + t.  Where all tiles together are at most half a round and the XCD with the most of them
// would keep the others from another part, they are cut over all workgroups instead (`whole`): position 0 of workgroup g, counted XCD by XCD,
// is part g / tiles of tile g % tiles (84 tiles, 10 or 11 an XCD, K = 151936: three parts instead of two, 1698 -> 1118 us; with as many parts either
// way the XCDs' own tiles are the better ones, 70 tiles, K = 14336 146 against 160 us: a weight tile is fetched by one XCD).  The fp32 sums of a part go to the tile buffer of its workgroup, and
// tile_sum_kernel adds the parts up, in order, with the layer's epilogue.  Decided here, where the row count is known: the host lays
// out rows for codebooks that are full.  A part is worth it from 16 slabs saved on (17-20 us; the sum reads at most 64 MB, about 10), in the XCD
// with the most tiles: the launch ends with that one.  (132 tiles, 16 or 17 an XCD, 48 slabs: whole 78 us, 102 with the sum where those of
// 16 were cut; 144 tiles of 64 slabs 87 and 106, 704, the last round half full on some, 310 and 330.)
// (Runs of slabs as long as each other, across tiles, keep every CU busy but not at one place of K: 1.10 times the time at 2644 rows.)
struct LastRound {
  int full, rem, ways, per, whole;
};
constexpr int F_XCD_WGS = 32;                // workgroups of an XCD that a dense layer is launched with where it may be cut
constexpr int F_WGS = 8 * F_XCD_WGS;
constexpr int F_MIN_SAVED = 16;              // slabs
constexpr int F_MIN_PART = 4;
// Slabs of a part where `tiles` tiles of n_slabs share `wgs` workgroups.
__host__ __device__ __forceinline__ int part_slabs(int wgs, int tiles, int n_slabs) {
  const int most = n_slabs / F_MIN_PART > 1 ? n_slabs / F_MIN_PART : 1, ways = wgs / tiles < most ? wgs / tiles : most;
  return (n_slabs + ways - 1) / ways;
}
__host__ __device__ __forceinline__ LastRound last_round(const LogitsArgs& a, int row_tiles, int xcd, int n_slabs) {
  const int tiles = row_tiles * a.n_strips;
  int len, longest;
  list_lengths(a, row_tiles, xcd, &len, &longest);
  LastRound r;
  r.whole = tiles > 0 && tiles <= F_WGS / 2 && F_WGS / tiles > F_XCD_WGS / longest;
  r.full = r.whole ? 0 : len & ~(F_XCD_WGS - 1);
  r.rem = r.whole ? tiles : len - r.full;
  r.ways = 1;
  r.per = n_slabs;
  // (what the XCD with the most tiles left gains decides: the launch ends with that one)
  const int wgs = r.whole ? F_WGS : F_XCD_WGS, most = r.whole ? tiles : longest - r.full;
  if (r.rem > 0 && most <= wgs / 2 && n_slabs - part_slabs(wgs, most, n_slabs) >= F_MIN_SAVED) {
    r.per = part_slabs(wgs, r.rem, n_slabs);
    r.ways = (n_slabs + r.per - 1) / r.per;    // no empty parts
  }
  return r;
}

// Tile t of a dense layer that is cut over all workgroups: the longer side in blocks of four, all of the other side inside.
__device__ __forceinline__ void locate_whole(const LogitsArgs& a, int row_tiles, int t, int* rt, int* st) {
  const int P = a.map_p_rows ? row_tiles : a.n_strips, Q = a.map_p_rows ? a.n_strips : row_tiles;
  const int blk = t / (4 * Q), in = t - blk * 4 * Q, wide = min(4, P - blk * 4);
  const int q = in / wide, p = blk * 4 + in - q * wide;
  *rt = a.map_p_rows ? p : q;
  *st = a.map_p_rows ? q : p;
}

// Slabs of a dense layer's contraction (k_dev: its length is known on the device only).
__device__ __forceinline__ int dense_slabs(const LogitsArgs& a) {
  const int n = (a.d * 2) / F_SLAB;
  return a.k_dev ? max(1, min(n, (__builtin_amdgcn_readfirstlane(*a.k_dev) * 2 + F_SLAB - 1) / F_SLAB)) : n;
}

struct Frags {
  uint4 a[F_N];
  uint4 b[F_N];
};

typedef f32x4 Acc[F_N][F_N];

// ---- epilogues: acc[i][j] is a 16 x 16 result block, register e of this lane is the value of hidden row
// row_base + j * 16 + (lane & 15) and column col_base + i * 16 + e, where col_base already holds the tile origin, the wave's
// offset and (lane >> 4) * 4.

// Columns at and beyond n_valid do not exist: they read as -inf.  (A pass of its own over the accumulators of the one
// tile of a matrix that has such columns: with the tests in the fold, or a second fold with them, the registers of
// both are more than there are.)
__device__ __forceinline__ void mask_tail16(Acc& acc, int col_base, int n_valid) {
#pragma unroll
  for (int i = 0; i < F_N; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = col_base + i * 16 + e < n_valid;
#pragma unroll
      for (int j = 0; j < F_N; ++j) {
        const float x = read_acc(acc[i][j][e]);
        float y;
        asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(y) : "v"(ok ? x : kNegInf));
        acc[i][j][e] = y;
      }
    }
}

// Fold one finished tile into the running triples, 16 values of a row at a time, in increasing column order per lane, so
// strict comparisons keep the lowest column among equal maxima.  The running sum is kept against the running maximum in
// base-2 units: exp(x - m) is one multiply-add and one hardware exponential.
__device__ __forceinline__ void fold_tile16(const Acc& acc, Triple (&run)[F_N], int col_base, int col0, int n_valid) {
  constexpr float kLog2e = 1.4426950408889634f;
#pragma unroll
  for (int j = 0; j < F_N; ++j) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float x[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) x[v] = read_acc(acc[h * 4 + (v >> 2)][j][v & 3]);
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
        run[j].i = col0 + col_base + h * 64 + (targ >> 2) * 16 + (targ & 3);
      }
      if (col_base + h * 64 < n_valid) {
        // (where nothing has been above -inf yet, columns that do not exist add 0 and a hidden row's NaN stay NaN.  The branch keeps
        // the groups apart: without it they are scheduled together and spill 48 bytes a lane.)
        const float m2 = run[j].m == kNegInf ? 0.f : -run[j].m * kLog2e;
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

// The same for a filtered sampled pick: x = logit * inv_temperature enters the running triple and is stored,
// fp32, at logits[row, col0 + column] (the selection kernels read the rows back); 16-byte stores where the four
// columns of a group all exist.
__device__ __forceinline__ void fold_store16(const Acc& acc, Triple (&run)[F_N], const LogitsArgs& a, int row_base, int r_end,
                                             int col_base, int n_valid) {
  const int lane15 = threadIdx.x & 15;
#pragma unroll
  for (int j = 0; j < F_N; ++j) {
    const int row = row_base + j * 16 + lane15;
    float* out = a.logits + (size_t)min(row, r_end - 1) * a.ld + a.col0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float x[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int col = col_base + h * 64 + (v >> 2) * 16 + (v & 3);
        const float z = read_acc(acc[h * 4 + (v >> 2)][j][v & 3]);
        x[v] = col < n_valid ? z * a.inv_temperature : kNegInf;
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
        run[j].i = a.col0 + col_base + h * 64 + (targ >> 2) * 16 + (targ & 3);
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
          const int col = col_base + h * 64 + q * 16;
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

// The same for a sampled pick: x = logit * inv_temperature enters the running triple, and x + Gumbel(u[row, col]) the
// running draw.  A lane's columns come in aligned fours (one generator call each) and in increasing order, so a strict
// comparison keeps the lowest column among equal values.  The four groups of 16 values are a real loop (the generator
// is long: unrolled 64 times per tile it would not fit the register file next to the accumulators).
__device__ __forceinline__ void fold_sample16(const Acc& acc, Triple (&run)[F_N], Draw (&draw)[F_N], const LogitsArgs& a,
                                              int row_base, int col_base, int n_valid) {
  const int lane15 = threadIdx.x & 15;
#pragma unroll
  for (int j = 0; j < F_N; ++j) {
    const uint32_t row = (uint32_t)(row_base + j * 16 + lane15);
    Triple t = run[j];
    Draw dr = draw[j];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float x[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) x[v] = read_acc(acc[h * 4 + (v >> 2)][j][v & 3]);
#pragma unroll 1
      for (int q = 0; q < 4; ++q) {
        const int c0 = a.col0 + col_base + h * 64 + q * 16;
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
        const float m = t.m == kNegInf ? 0.f : t.m;  // (a hidden row's NaN stay NaN, as in fold_tile16)
        t.s += (__expf(z[0] - m) + __expf(z[1] - m)) + (__expf(z[2] - m) + __expf(z[3] - m));
        // (the next four move up: picked by q, the values go through scratch memory -- draws of 256 sequences over 128256
        // columns 735 -> 644 us, 300: 1136 -> 949; the plain picks' kernel gains 27 and 22 of that as well)
#pragma unroll
        for (int v = 0; v < 12; ++v) x[v] = x[v + 4];
      }
    }
    run[j] = t;
    draw[j] = dr;
  }
}

// Eight consecutive columns per lane from two blocks' fours: lanes of the even quarter-waves (lane >> 4) get block i's
// columns, the odd ones block i + 1's, the lower half of the wave columns 0-7 and the upper 8-15 of it.  `lo`, `hi`: this
// lane's four bf16 of block i and of block i + 1.
__device__ __forceinline__ uint4 eight_columns(uint2 lo, uint2 hi) {
  const auto x = __builtin_amdgcn_permlane16_swap(lo.x, hi.x, false, false);
  const auto y = __builtin_amdgcn_permlane16_swap(lo.y, hi.y, false, false);
  return uint4{x[0], y[0], x[1], y[1]};
}

// Stores two blocks' bf16 (columns col_base + i * 16 ..., and the next 16) of one row in 16-byte pieces; columns come in
// fours, and n_valid and the row pitch are multiples of 8 (the layers' widths are).
__device__ __forceinline__ void store_two_blocks(uint16_t* out_row, bool row_ok, int col_base, int i, uint2 lo, uint2 hi,
                                                 int n_valid) {
  const uint4 v = eight_columns(lo, hi);
  const int quarter = (threadIdx.x >> 4) & 3;
  const int col = col_base - quarter * 4 + (i + (quarter & 1)) * 16 + (quarter >> 1) * 8;
  if (row_ok && col < n_valid) *reinterpret_cast<uint4*>(out_row + col) = v;
}

// Store one finished tile of a gradient product, rounded once to bf16: nothing is added.  (Over few rows such a product is its stores: with
// the dense layers' epilogue 128256 x 4096 over 244 rows 581 us, 457 with this one, 537 past the caches; 32064 x 3072 over 109 105, 64, 73.)
__device__ __forceinline__ void store_plain16(const Acc& acc, const LogitsArgs& a, int row_base, int r_end, int col_base, int n_valid) {
  const int lane15 = threadIdx.x & 15;
#pragma unroll
  for (int j = 0; j < F_N; ++j) {
    const int row = row_base + j * 16 + lane15;
    uint16_t* out_row = reinterpret_cast<uint16_t*>(a.out) + (size_t)row * a.ldo;
#pragma unroll
    for (int i = 0; i < F_N; i += 2) {
      uint2 o[2];
#pragma unroll
      for (int h = 0; h < 2; ++h)
        o[h] = uint2{pack_bf16(read_acc(acc[i + h][j][0]), read_acc(acc[i + h][j][1])),
                     pack_bf16(read_acc(acc[i + h][j][2]), read_acc(acc[i + h][j][3]))};
      store_two_blocks(out_row, row < r_end, col_base, i, o[0], o[1], n_valid);
    }
  }
}

// Store one finished tile as a dense layer's output: out[row, col] = act(acc + bias[col]) + residual[row, col], rounded
// once to bf16.  The loads the epilogue needs are issued in batches ahead of their use (the bias of all the lane's
// columns once, the residual of 16 rows at a time): one memory round trip per batch, during which the matrix cores
// have nothing to do.
__device__ __forceinline__ void store_tile16(const Acc& acc, const LogitsArgs& a, int row_base, int r_end, int col_base,
                                             int n_valid) {
  const int lane15 = threadIdx.x & 15;
  float4 bias[F_N];
#pragma unroll
  for (int i = 0; i < F_N; ++i) {
    const int col = col_base + i * 16;
    bias[i] = (a.bias && col < n_valid) ? *reinterpret_cast<const float4*>(a.bias + col) : float4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int j = 0; j < F_N; ++j) {
    const int row = row_base + j * 16 + lane15;
    const bool row_ok = row < r_end;
    uint16_t* out_row = reinterpret_cast<uint16_t*>(a.out) + (size_t)row * a.ldo;
    uint2 res[F_N];
#pragma unroll
    for (int i = 0; i < F_N; ++i) {
      const int col = col_base + i * 16;
      res[i] = (a.residual && row_ok && col < n_valid)
                   ? *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(a.residual) + (size_t)row * a.ldo + col)
                   : uint2{0u, 0u};
    }
    uint2 o[F_N];
#pragma unroll
    for (int i = 0; i < F_N; ++i) {
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = read_acc(acc[i][j][e]);
      x[0] += bias[i].x;
      x[1] += bias[i].y;
      x[2] += bias[i].z;
      x[3] += bias[i].w;
      if (a.act == 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = gelu_erf(x[e]);
      }
      x[0] += __uint_as_float(res[i].x << 16);
      x[1] += __uint_as_float(res[i].x & 0xFFFF0000u);
      x[2] += __uint_as_float(res[i].y << 16);
      x[3] += __uint_as_float(res[i].y & 0xFFFF0000u);
      o[i] = uint2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
    }
#pragma unroll
    for (int i = 0; i < F_N; i += 2) store_two_blocks(out_row, row_ok, col_base, i, o[i], o[i + 1], n_valid);
  }
}

// The same with the residual and the output in fp32 (no rounding): 16-byte loads and stores.
__device__ __forceinline__ void store_tile16_f32(const Acc& acc, const LogitsArgs& a, int row_base, int r_end, int col_base,
                                                 int n_valid) {
  const int lane15 = threadIdx.x & 15;
  const float* res = reinterpret_cast<const float*>(a.residual);
  float* out = reinterpret_cast<float*>(a.out);
  float4 bias[F_N];
#pragma unroll
  for (int i = 0; i < F_N; ++i) {
    const int col = col_base + i * 16;
    bias[i] = (a.bias && col < n_valid) ? *reinterpret_cast<const float4*>(a.bias + col) : float4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int j = 0; j < F_N; ++j) {
    const int row = row_base + j * 16 + lane15;
    if (row >= r_end) continue;
    float4 rv[F_N];
#pragma unroll
    for (int i = 0; i < F_N; ++i) {
      const int col = col_base + i * 16;
      const bool ok = col < n_valid;
      rv[i] = (res && ok) ? *reinterpret_cast<const float4*>(res + (size_t)row * a.ldo + col) : float4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < F_N; ++i) {
      const int col = col_base + i * 16;
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = read_acc(acc[i][j][e]);
      x[0] += bias[i].x;
      x[1] += bias[i].y;
      x[2] += bias[i].z;
      x[3] += bias[i].w;
      if (a.act == 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = gelu_erf(x[e]);
      }
      if (col < n_valid)
        *reinterpret_cast<float4*>(out + (size_t)row * a.ldo + col) =
            float4{x[0] + rv[i].x, x[1] + rv[i].y, x[2] + rv[i].z, x[3] + rv[i].w};
    }
  }
}

// Store one finished tile as it is (fp32), for a dense layer whose K range is split over several workgroups.
__device__ __forceinline__ void store_partial16(const Acc& acc, float* part, int ld, int row_base, int r_end, int col_base,
                                                int n_valid) {
  const int lane15 = threadIdx.x & 15;
#pragma unroll
  for (int j = 0; j < F_N; ++j) {
    const int row = row_base + j * 16 + lane15;
#pragma unroll
    for (int i = 0; i < F_N; ++i) {
      const int col = col_base + i * 16;
      float4 x;
      x.x = read_acc(acc[i][j][0]);
      x.y = read_acc(acc[i][j][1]);
      x.z = read_acc(acc[i][j][2]);
      x.w = read_acc(acc[i][j][3]);
      if (row < r_end && col < n_valid) *reinterpret_cast<float4*>(part + (size_t)row * ld + col) = x;
    }
  }
}

// Store one finished tile as the gradient of the loss with respect to the logits (see LogitsArgs, probability mode).
// Columns come in fours; ldo is a multiple of 64.
__device__ __forceinline__ void store_prob16(const Acc& acc, const LogitsArgs& a, void* out, int ldo, int col0, int row_base, int r_end,
                                             int col_base, int n_valid) {
  const int lane15 = threadIdx.x & 15;
  float lse[F_N], g[F_N];
  int tgt[F_N];
#pragma unroll
  for (int j = 0; j < F_N; ++j) {
    const int row = row_base + j * 16 + lane15;
    const bool ok = row < r_end;
    lse[j] = ok ? a.lse[row] : 0.f;
    g[j] = ok ? a.row_grad[row] : 0.f;
    tgt[j] = ok ? a.targets[row] - col0 : -1;
  }
#pragma unroll
  for (int j = 0; j < F_N; ++j) {
    const int row = row_base + j * 16 + lane15;
    uint16_t* out_row = reinterpret_cast<uint16_t*>(out) + (size_t)row * ldo;
    uint2 o[F_N];
#pragma unroll
    for (int i = 0; i < F_N; ++i) {
      const int col = col_base + i * 16;
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float z = read_acc(acc[i][j][e]);
        const float p = __expf(z - lse[j]) - (col + e == tgt[j] ? 1.f : 0.f);
        x[e] = col + e < n_valid ? g[j] * p : 0.f;
      }
      o[i] = uint2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
    }
#pragma unroll
    for (int i = 0; i < F_N; i += 2) store_two_blocks(out_row, row < r_end, col_base, i, o[i], o[i + 1], ldo);
  }
}

// Lanes that hold the same rows, 16 or 32 apart, exchange halves: of a[k] and a[k + N] the lower lane of a pair keeps row k
// and the upper one row k + N, each with both lanes' values.
struct Swap16 {
  __device__ __forceinline__ void operator()(uint32_t& x, uint32_t& y) const {
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = r[0];
    y = r[1];
  }
};
struct Swap32 {
  __device__ __forceinline__ void operator()(uint32_t& x, uint32_t& y) const {
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = r[0];
    y = r[1];
  }
};
__device__ __forceinline__ void merge(Triple& a, const Triple& b) { merge_triple(a, b); }
__device__ __forceinline__ void merge(Draw& a, const Draw& b) { merge_draw(a, b); }

template <int N, typename R, typename S>
__device__ __forceinline__ void merge_rows(R (&a)[F_N], S swap) {
  static_assert(sizeof(R) == 12, "three words");
#pragma unroll
  for (int k = 0; k < N; ++k) {
    uint32_t x[3], y[3];
    __builtin_memcpy(x, &a[k], 12);
    __builtin_memcpy(y, &a[k + N], 12);
#pragma unroll
    for (int w = 0; w < 3; ++w) swap(x[w], y[w]);
    R other;
    __builtin_memcpy(&a[k], x, 12);
    __builtin_memcpy(&other, y, 12);
    merge(a[k], other);
  }
}

// MODE 8 and 9 are measurement probes of the base part (their results are NOT the logits' reduction): 8 stops
// requesting operands after the first two slabs (the matrix cores, the LDS reads and the fold run as usual on
// those two slabs' values), 9 also stops reading LDS and folds once per strip -- the MFMA stream alone.  They
// bracket what the operand stream costs and give the clock the matrix cores alone are left with.
// ROT (base part with a single row tile: up to 256 hidden rows): nobody shares a workgroup's weight tiles, so the
// strips walk K from different slabs, wrapping round.  With all of them at the same
// slab every request in flight goes to the same 128-byte column of rows a power of two apart, and with it to the
// same few memory channels.  (With many row tiles the workgroups that share operands through L2 and the
// memory-side cache must stay in step: there the rotation costs 1-2 %, and so does its arithmetic alone; with two
// row tiles it is level or 1 % slower.  A decode step of 256 sequences: 646 -> 634 us, with a filtered draw 704 -> 675.  With the hyper part
// along, V = 128256, d = 4096: 1 x 193 rows 250 us in step, 240 rotated; where its items open a third round, 3 x 65 with 2048 entries each,
// 317, 293, and 292 in two launches.)
//
// A workgroup walks its XCD's list (locate_base) from its own position on, in steps of the workgroups an XCD has: the
// operand stream runs on from one output tile to the next, and a tile's epilogue finds the next one's first two slabs on the
// way.  With a workgroup per tile instead, a launch and the first slabs' round trip stood before every tile and a
// store queue behind it: a training step of 8 x 4096 tokens (kernels only) 172.8 -> 168.9 ms, of it the order below 2.5.
// The hyper part alone and K-split layers (modes 1, 5) have a workgroup per item: what exists of them is known on the device.
// TW, TH (mode 2): the operand of that side is K-major, W [k_rows, ldw] and H [k_rows, ldh]; there may be a batch of such products,
// of a.rows output rows each, one below the other.
// HYP (modes 0 and 3): the items of the per-sequence hyper part (a.hyper) that exist are dealt out with the base part's last tiles.  In a launch
// of its own that part is one or two rounds of tiles on a few CUs (58 us at d = 3072): V = 32064, 8 x 86 rows 190 -> 146 us, 17 x 75 257 -> 204;
// V = 128256, d = 4096, 3 x 176 654 -> 597, 2 x 577 1090 -> 1043; level about 10000 rows (3 x 3577 7818 and 7826).
template <int MODE, bool ROT = false, bool TW = false, bool TH = false, bool HYP = false>
__global__ void __launch_bounds__(F_THREADS) logits_fast_kernel(LogitsArgs a) {
  static_assert((MODE == 2 || !TW) && (TW || !TH), "dense layers only, and H K-major only where W is");
  static_assert(!HYP || MODE == 0 || (MODE == 3 && !ROT), "");
  constexpr bool PROBE_NOREQ = MODE == 8 || MODE == 9;
  constexpr bool PROBE_MFMA = MODE == 9;
  constexpr bool LIST = MODE != 1 && MODE != 5;
  extern __shared__ __align__(1024) unsigned char lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wv = wave & 1;    // which 128 vocabulary rows of the tile
  const int wr = wave >> 1;   // which 128 hidden rows of the tile

  // ---- the work: positions first, first + step, ... of a list; item(j) gives its row tile and strip ----------------
  const int first = LIST ? (int)(blockIdx.x >> 3) : 0, step = LIST ? (int)(gridDim.x >> 3) : 1;
  const unsigned char* Wp = reinterpret_cast<const unsigned char*>(a.W);
  const unsigned char* Hm = reinterpret_cast<const unsigned char*>(a.H);
  const size_t row_bytes = (size_t)a.d * 2;
  // (pitches of their own: dense layers only)
  const size_t pitch_h = MODE == 2 && a.ldh ? (size_t)a.ldh * 2 : row_bytes;
  const size_t pitch_w = MODE == 2 && a.ldw ? (size_t)a.ldw * 2 : row_bytes;
  int r_end = a.rows;                                // one past the last row of the matrix, or of the sequence
  if ((MODE == 2 || MODE == 5) && a.rows_dev) r_end = min(r_end, __builtin_amdgcn_readfirstlane(*a.rows_dev));
  const int tiles_each = (r_end + FT - 1) / FT, row_tiles_now = TW && a.batch > 1 ? a.batch * tiles_each : tiles_each;
  int n_valid = a.w_rows;
  int one_rt = 0, one_st = 0, one_r0 = 0, ks = 0;    // modes 1, 5: the one item
  if (MODE == 1) {
    if ((int)blockIdx.x >= a.n_work) return;
    one_rt = blockIdx.x / a.n_strips;
    // workgroup ids go round-robin over the 8 XCDs, and the strips beyond a sequence's C_b are empty: with the
    // strip taken straight from the id, the XCDs that own the low strips would do all the work (config 5: 9 of 16
    // strips exist, XCD 0 owned two of them, the others one).  Rotating by the row tile deals them out evenly.
    one_st = (int)((blockIdx.x + (unsigned)one_rt) % (unsigned)a.n_strips);
    const int b = one_rt / a.row_tiles;
    one_r0 = b * a.rows_per_seq + (one_rt % a.row_tiles) * FT;
    r_end = (b + 1) * a.rows_per_seq;
    n_valid = min(max(a.size[b], 0), a.w_rows);
    Wp += (size_t)b * a.w_rows * row_bytes;
  } else if (MODE == 5) {
    // few tiles, K split: workgroup -> (K part, row tile, weight tile)
    const int t = blockIdx.x / a.ksplit;
    ks = (int)(blockIdx.x % a.ksplit);
    one_rt = t % a.row_tiles;
    one_st = t / a.row_tiles;
    if (one_st >= a.n_strips) return;
    one_r0 = one_rt * FT;
    if (one_r0 >= r_end) return;                     // a tile beyond the rows that exist
    Wp += (size_t)ks * a.slabs_per_part * F_SLAB;    // this part's slabs start here in every row
    Hm += (size_t)ks * a.slabs_per_part * F_SLAB;
  }
  const int n_vt = min(a.n_vtiles, (n_valid + FT - 1) / FT);
  const int strip = MODE == 2 ? 1 : a.strip;
  int n_slabs = MODE == 5 ? min(a.slabs_per_part, (int)(row_bytes / F_SLAB) - ks * a.slabs_per_part)
                          : (int)(row_bytes / F_SLAB);
  if (MODE == 2) n_slabs = dense_slabs(a);
  // the item's slabs [s0, s0 + sn) and, where it is a part of a tile, the buffer of its sums (else -1)
  const int k_rows = (TW || TH) && a.k_dev ? min(a.k_rows, max(__builtin_amdgcn_readfirstlane(*a.k_dev), 0)) : a.k_rows;     // of the K-major operands
  const LastRound last = MODE == 2 && a.split ? last_round(a, row_tiles_now, (int)(blockIdx.x & 7), n_slabs) : LastRound{0, 0, 1, n_slabs};

  struct Item {
    int r0, st, s0, sn, part;    // first row, strip, slabs, buffer
    int b;                       // product of a batch; sequence of an item of the hyper part, else (HYP) -1
  };
  // The hyper part's items lie sequence by sequence, those of one strip after strip.  How many each sequence has follows from its size, so a table of the
  // items ahead of every sequence is made in LDS first; an item's sequence is found in it by two reads of the wave.  (Counted out from
  // the first sequence on, a load and a wait for the whole operand stream a step: 2000 x 66 rows, V = 1024, d = 512 2419 us, 499 with the table,
  // 546 with the hyper part in a launch of its own; 1024 x 66, V = 4096, d = 1024 1302, 771, 815; 64 x 70, V = 32064, d = 3072 893, 868, 910.)
  int32_t* const items_before = reinterpret_cast<int32_t*>(lds + F_LDS);
  int32_t* const sizes = items_before + F_HYP_SEQS;
  int hyper_items = 0;
  auto strips_of = [&](int size) -> int { return (size + FT * a.hyper.strip - 1) / (FT * a.hyper.strip); };
  if (HYP) {
    int32_t* const wave_items = sizes + F_HYP_SEQS;
    const int each = (a.hyper.n_seq + F_THREADS - 1) / F_THREADS, b0 = tid * each, b1 = min(b0 + each, a.hyper.n_seq);
    int own = 0;
    for (int b = b0; b < b1; ++b) {
      sizes[b] = min(max(a.hyper.size[b], 0), a.hyper.cap);
      own += strips_of(sizes[b]) * a.hyper.row_tiles;
    }
    int upto = own;                                  // of this lane and those before it
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(upto, o);
      upto += lane >= o ? x : 0;
    }
    if (lane == 63) wave_items[wave] = upto;
    __syncthreads();
    int before = upto - own;
    for (int w = 0; w < 4; ++w) {
      before += w < wave ? wave_items[w] : 0;
      hyper_items += wave_items[w];
    }
    hyper_items = __builtin_amdgcn_readfirstlane(hyper_items);
    for (int b = b0; b < b1; ++b) {
      items_before[b] = before;
      before += strips_of(sizes[b]) * a.hyper.row_tiles;
    }
    __syncthreads();
  }
  // the last sequence with at most k items ahead of it (the one that has item k: those without items lie before it)
  auto sequence_of = [&](int k) -> int {
    const int each = (a.hyper.n_seq + 63) / 64;
    const int block = lane * each;
    const int c = __popcll(__ballot(block < a.hyper.n_seq && items_before[min(block, a.hyper.n_seq - 1)] <= k)) - 1;
    const int b = c * each + lane;
    return c * each + __popcll(__ballot(lane < each && b < a.hyper.n_seq && items_before[min(b, a.hyper.n_seq - 1)] <= k)) - 1;
  };
  // (where all strips are one tile the base part's last ones and the hyper items are dealt out as one; else every XCD goes on with every eighth
  // of these behind its base list: the longer strips of the base part have to be dealt out evenly by themselves, 9 x 263 rows 1930 us, 2155 as one)
  const bool together = HYP && strip == 1 && a.hyper.strip == 1;
  const int base_items = HYP && !together ? list_length(a, row_tiles_now, (int)(blockIdx.x & 7)) : 0;
  // (behind: j is not the workgroup's first position.  There are copies of this at every place where the operand stream may go on to another
  // item, and what a whole cut needs is left out of most of them)
  auto item = [&](int j, Item* it, bool behind) __attribute__((always_inline)) -> bool {
    it->s0 = 0;
    it->sn = n_slabs;
    it->part = -1;
    it->b = 0;
    if (!LIST) {
      it->r0 = one_r0;
      it->st = one_st;
      return j == 0;
    }
    int rt;
    const int xcd = (int)(blockIdx.x & 7);
    if (MODE == 2 && behind && last.whole && last.ways > 1) return false;
    if (MODE == 2 && last.ways > 1 && j >= last.full) {
      const int g = last.whole ? xcd * F_XCD_WGS + j : j - last.full, ks = __builtin_amdgcn_readfirstlane(g / last.rem);
      if (ks >= last.ways || (last.whole && j >= F_XCD_WGS)) return false;
      it->s0 = ks * last.per;
      it->sn = min(last.per, n_slabs - it->s0);
      it->part = last.whole ? g : xcd * F_XCD_WGS + g;
      j = last.full + g - ks * last.rem;
    }
    if (MODE == 2 && !behind && last.ways > 1 && last.whole)
      locate_whole(a, row_tiles_now, j, &rt, &it->st);
    else if (!locate_base(a, row_tiles_now, xcd, j, &rt, &it->st, HYP && together ? hyper_items : 0, HYP ? &it->b : nullptr)) {
      if (!HYP || together) return false;
      it->b = (j - base_items) * 8 + xcd;
      if (it->b >= hyper_items) return false;
    }
    if (HYP && it->b >= 0) {
      const int b = sequence_of(it->b), k = it->b - __builtin_amdgcn_readfirstlane(items_before[b]);
      const int n = strips_of(__builtin_amdgcn_readfirstlane(sizes[b]));
      rt = __builtin_amdgcn_readfirstlane(k / n);
      it->st = k - rt * n;
      it->b = b;
      it->r0 = b * a.rows_per_seq + rt * FT;
      return true;
    }
    it->r0 = rt * FT;
    if (TW && a.batch > 1) {
      it->b = __builtin_amdgcn_readfirstlane(rt / tiles_each);
      it->r0 = it->b * a.rows + (rt - it->b * tiles_each) * FT;
    }
    if (MODE == 2) {                         // (quotients come out of vector instructions; addresses follow from these)
      it->r0 = __builtin_amdgcn_readfirstlane(it->r0);
      it->st = __builtin_amdgcn_readfirstlane(it->st);
    }
    return true;
  };

  // what an item's tiles are cut from
  struct Part {
    const unsigned char* W;
    int n_valid, n_vt, r_end, strip;
  };
  auto part_of = [&](const Item& it) -> Part {
    if (HYP && it.b >= 0) {
      const int n = __builtin_amdgcn_readfirstlane(sizes[it.b]);
      return Part{reinterpret_cast<const unsigned char*>(a.hyper.W) + (size_t)it.b * a.hyper.cap * row_bytes, n, (n + FT - 1) / FT,
                  (it.b + 1) * a.rows_per_seq, a.hyper.strip};
    }
    return Part{TW ? Wp + (size_t)it.b * a.batch_w * 2 : Wp, n_valid, n_vt, TW && a.batch > 1 ? (it.b + 1) * a.rows : r_end, strip};
  };

  // ---- loader: lane l of wave w, instruction i moves the chunk that lands at LDS byte
  //      ((w * F_PAIRS + i) * 8 + (l >> 3)) * 128 + (l & 7) * 16 of the operand tile; offsets are relative to
  //      the first row of the tile, rows past the last valid one are clamped onto it ------------------
  const uint32_t lds_base = lds_offset_of(lds);
  const int ld_row = lane >> 3;                                  // row inside the 8-row group
  // per-lane global byte offsets of the 8 row groups a wave requests (swizzled chunk folded in); rows
  // past the last valid one are clamped onto it.  B's change with the item, A's with the tile.
  auto row_offset = [&](int i, int lim, size_t pitch) -> uint32_t {
    const int row = (wave * F_PAIRS + i) * 8 + ld_row;
    const int chunk16 = ((lane & 7) ^ ((row >> 1) & 7)) * 16;
    return (uint32_t)(min(row, lim) * (int)pitch + chunk16);
  };
  // (K-major: two rows of the slab a request, a lane's 16 bytes of its row's 512; columns past the last whole chunk of the matrix row are
  // clamped onto it)
  auto krow_offset = [&](int i, int chunks, size_t pitch) -> uint32_t {
    const int k = (wave * F_PAIRS + i) * 2 + (lane >> 5);
    const int chunk = (lane & 31) ^ (((k & 3) | ((k >> 3) & 1) << 2) << 1);
    return (uint32_t)(k * (int)pitch + min(chunk, chunks - 1) * 16);
  };
  uint32_t voffA[F_PAIRS], voffB[F_PAIRS];
  const unsigned char* Wtile = Wp;
  Part at = {Wp, n_valid, n_vt, r_end, strip};       // (one for all items but with the hyper part and in a batch)
  const unsigned char* Hp = Hm;
  // ---- the cursor of the operand stream: slab lslab of weight tile lvt of the item at position lj (none: !live) ----------
  int lj = first, lslab = 0, lslab_end = n_slabs, lvt = 0, lvt_end = 0, rot = 0;
  int w_col = 0, h_col = 0;                  // K-major: byte of the tile's first column in a row
  bool live = true;
  auto set_tile = [&](int vt) {
    if (TW) w_col = vt * F_KROW;
    Wtile = at.W + (TW ? (size_t)w_col : (size_t)vt * FT * pitch_w);
#pragma unroll
    for (int i = 0; i < F_PAIRS; ++i)
      voffA[i] = TW ? krow_offset(i, ((int)pitch_w - w_col) >> 4, pitch_w) : row_offset(i, at.n_valid - 1 - vt * FT, pitch_w);
  };
  auto open_item = [&](bool behind) __attribute__((always_inline)) {
    if (HYP) asm volatile("" : "+s"(lj));       // (what is worked out here is not worked out for every slab)
    Item it;
    live = item(lj, &it, behind);
    if (!live) return;
    if (HYP || TW) at = part_of(it);
    lvt = it.st * at.strip;
    lvt_end = min(lvt + at.strip, at.n_vt);
    const int r0 = it.r0, st = it.st;
    lslab = it.s0;
    lslab_end = it.s0 + it.sn;
    if (MODE != 2) live = lvt < lvt_end;       // (a tile of a dense layer exists)
    if (!live) return;
    if (TH) h_col = (r0 - it.b * a.rows) * 2;
    Hp = Hm + (TH ? (size_t)h_col : (size_t)r0 * pitch_h);
    if (TH) Hp += (size_t)it.b * a.batch_h * 2;
#pragma unroll
    for (int i = 0; i < F_PAIRS; ++i)
      voffB[i] = TH ? krow_offset(i, ((int)pitch_h - h_col) >> 4, pitch_h)
                    : row_offset(i, at.r_end - 1 - r0, pitch_h);
    if (ROT) rot = __builtin_amdgcn_readfirstlane(st % n_slabs);
    set_tile(lvt);
  };
  // request the slab that follows in the stream, if any, and advance the cursor.  A request is 16 instructions per
  // wave, so that the caller can place them between MFMAs.
  uint32_t isA = 0;                          // LDS destination (operand A) of the slab being requested
  const unsigned char* is_ga = Wp;
  const unsigned char* is_gb = Hm;
  int is_rows = 0, is_col_a = 0, is_col_b = 0;
  u32x4 is_ra, is_rb;                        // their descriptors where they are K-major
  auto issue_begin = [&](int stage) {
    isA = __builtin_amdgcn_readfirstlane(lds_base + stage * F_STAGE + wave * (F_PAIRS * 1024));
    if (live) {                              // else: keep the last valid source
      int sl = lslab;
      if (ROT) {
        sl += rot;
        if (sl >= n_slabs) sl -= n_slabs;
      }
      is_ga = Wtile + (size_t)sl * (TW ? 64 * pitch_w : F_SLAB);
      is_gb = Hp + (size_t)sl * (TH ? 64 * pitch_h : F_SLAB);
      is_col_a = w_col;
      is_col_b = h_col;
      is_rows = k_rows - sl * 64;
    }
    // (a descriptor's range ends with the matrix's last row)
    if (TW) is_ra = k_rows_rsrc(is_ga, is_rows, pitch_w, is_col_a);
    if (TH) is_rb = k_rows_rsrc(is_gb, is_rows, pitch_h, is_col_b);
    // (five wait states between v_readfirstlane and the load that reads its register: the compiler does not know that the requests are loads)
    if (TW && TH)
      asm volatile("s_nop 4" : "+s"(is_ra), "+s"(is_rb));
    else if (TW)
      asm volatile("s_nop 4" : "+s"(is_ra));
  };
  // request n of the 16 of a slab: 8 rows of the vocabulary tile (n even) or of the hidden rows' (n odd)
  auto request = [&](auto n_) __attribute__((always_inline)) {
    constexpr int n = decltype(n_)::value;
    if constexpr (n & 1) {
      if constexpr (TH)
        load16_to_lds<F_OPER + (n >> 1) * 1024>(is_rb, voffB[n >> 1], isA);
      else
        load16_to_lds<F_OPER + (n >> 1) * 1024>(is_gb, voffB[n >> 1], isA);
    } else {
      if constexpr (TW)
        load16_to_lds<(n >> 1) * 1024>(is_ra, voffA[n >> 1], isA);
      else
        load16_to_lds<(n >> 1) * 1024>(is_ga, voffA[n >> 1], isA);
    }
  };
  auto issue_end = [&]() {
    if (live && ++lslab == lslab_end) {
      lslab = 0;                               // (a strip of several tiles is never a part)
      if (MODE != 2 && ++lvt < lvt_end) {
        set_tile(lvt);
      } else {
        lj += step;
        open_item(true);
      }
    }
  };
  // ---- MFMA operand addresses (bytes inside an operand tile), swizzle folded in ---------------------
  const int sw = (lane >> 1) & 7;   // ((row >> 1) & 7) of every row this lane reads
  const int quarter = lane >> 4;    // which 8 of a k-step's 32 elements
  const int offA0 = (wv * 128 + (lane & 15)) * F_SLAB;
  const int offB0 = (wr * 128 + (lane & 15)) * F_SLAB;
  // (K-major: lane l reads 8 bytes of row k = 8 quarter + ((l & 15) >> 2) of the k-step, and of row k + 4, in the piece of block idx of its
  // wave's 8; idx only meets the low 3 bits of the piece)
  const uint32_t tr0 = (uint32_t)((8 * quarter + ((lane & 15) >> 2)) * F_KROW + ((((lane & 15) >> 2) | (quarter & 1) << 2) * 32) + (lane & 3) * 8);
  // (addresses of the eight blocks in the stage that is read: everything else is an instruction's own offset)
  uint32_t trA[F_N], trB[F_N];
#pragma unroll
  for (int i = 0; i < F_N; ++i) {
    trA[i] = lds_base + ((tr0 + wv * 256) ^ (i * 32));
    trB[i] = lds_base + ((tr0 + wr * 256) ^ (i * 32));
  }
  // read e (Schedule) of k-step q of the slab in a stage
  using Sched = Schedule<TW, TH>;
  auto read_one = [&](Frags& f, int stage, auto q_, auto e_, auto next_) __attribute__((always_inline)) {
    constexpr bool next = decltype(next_)::value;
    constexpr int q = decltype(q_)::value, e = decltype(e_)::value, n = Sched::fragment(e), half = Sched::half(e);
    constexpr bool is_a = Sched::is_a(n);
    constexpr int idx = n <= 1 ? 0 : (n <= F_N ? n - 1 : n - F_N);
    const int base = stage * F_STAGE + (((4 * q + quarter) ^ sw) << 4);
    // (the first k-step's reads go over to the other stage)
    if constexpr (next && half == 0 && (is_a ? TW : TH)) {
      if constexpr (is_a)
        asm volatile("v_add_u32 %0, %1, %0" : "+v"(trA[idx]) : "s"(stage ? (uint32_t)F_STAGE : 0u - (uint32_t)F_STAGE));
      else
        asm volatile("v_add_u32 %0, %1, %0" : "+v"(trB[idx]) : "s"(stage ? (uint32_t)F_STAGE : 0u - (uint32_t)F_STAGE));
    }
    if constexpr (is_a && TW)
      read_transposed<q * 32 * F_KROW + half * 4 * F_KROW, half>(f.a[idx], trA[idx]);
    else if constexpr (!is_a && TH)
      read_transposed<F_OPER + q * 32 * F_KROW + half * 4 * F_KROW, half>(f.b[idx], trB[idx]);
    else if constexpr (is_a)
      f.a[idx] = *reinterpret_cast<const uint4*>(lds + base + offA0 + idx * 16 * F_SLAB);
    else
      f.b[idx] = *reinterpret_cast<const uint4*>(lds + base + F_OPER + offB0 + idx * 16 * F_SLAB);
  };

  constexpr std::integral_constant<int, 0> kZero{};
  constexpr std::integral_constant<int, 1> kOne{};
  Acc acc;
  Frags f[2];                                        // the two k-steps of a slab
  int g = 0;                                         // slabs behind
  // one slab: 128 MFMAs, and what goes out between them; FIRST: nothing has been accumulated yet.  The hand-overs
  // are the same for every slab, the last ones included: past the end of the stream the requests re-read the last slab
  // into a stage nobody reads again.
  auto slab_step = [&](auto first_) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(first_)::value;
    const int stage = g & 1;
    static_for<F_SLOTS>([&](auto m_) __attribute__((always_inline)) {
      constexpr int m = decltype(m_)::value;
      constexpr int q = m / (F_N * F_N), i = m / F_N % F_N;
      constexpr int j = i & 1 ? F_N - 1 - m % F_N : m % F_N;      // (to and fro: one operand stays from MFMA to MFMA, 1 %)
      if constexpr (m == Sched::free_) {
        __builtin_amdgcn_sched_barrier(0);
        barrier_after_lds();
        if (!PROBE_NOREQ) issue_begin(stage);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (m == Sched::landed) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(PROBE_NOREQ ? 0 : Sched::out_at_landed));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      mfma<FIRST && q == 0>(acc[i][j], f[q].a[i], f[q].b[j]);
      if constexpr (!PROBE_MFMA && m >= Sched::read2 && m < Sched::read2 + Sched::reads) {
        __builtin_amdgcn_sched_barrier(0);
        read_one(f[1], stage, kOne, std::integral_constant<int, m - Sched::read2>{}, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (!PROBE_MFMA && m >= Sched::read1 && m < Sched::read1 + Sched::reads) {
        __builtin_amdgcn_sched_barrier(0);
        read_one(f[0], stage ^ 1, kZero, std::integral_constant<int, m - Sched::read1>{}, std::true_type{});
        __builtin_amdgcn_sched_barrier(0);
      }
      constexpr int rq = m - Sched::request;
      if constexpr (!PROBE_NOREQ && rq >= 0 && rq % Sched::request_every == 0 && rq / Sched::request_every < 2 * F_PAIRS) {
        __builtin_amdgcn_sched_barrier(0);
        request(std::integral_constant<int, rq / Sched::request_every>{});
        if constexpr (rq / Sched::request_every == 2 * F_PAIRS - 1) issue_end();
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    ++g;
  };

  if (HYP && MODE == 0) {
    // strips of the hyper part that do not exist leave empty triples (ahead of the loop: divergent code in it, and the compiler keeps
    // the loop's state in vector registers)
    for (int h = blockIdx.x; h < a.hyper.n_work; h += gridDim.x) {
      const int rt = h / a.hyper.n_strips, st = h % a.hyper.n_strips, b = rt / a.hyper.row_tiles;
      const int row = b * a.rows_per_seq + (rt % a.hyper.row_tiles) * FT + tid;
      if (st * a.hyper.strip * FT < a.hyper.size[b] || row >= (b + 1) * a.rows_per_seq) continue;
      const size_t q = (size_t)row * a.n_parts + a.hyper.part0 + st;
      a.part_m[q] = kNegInf;
      a.part_s[q] = 0.f;
      a.part_i[q] = kNoColumn;
    }
  }
  open_item(false);
  if (live) {
    // prologue: the first two slabs of the stream requested; the first landed and visible, the fragments of its first
    // k-step on the way
    issue_begin(0);
    static_for<2 * F_PAIRS>(request);
    issue_end();
    issue_begin(1);
    static_for<2 * F_PAIRS>(request);
    issue_end();
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(PROBE_NOREQ ? 0 : 2 * F_PAIRS));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    static_for<Sched::reads>([&](auto e) __attribute__((always_inline)) { read_one(f[0], 0, kZero, e, std::false_type{}); });
    if (PROBE_MFMA) static_for<Sched::reads>([&](auto e) __attribute__((always_inline)) { read_one(f[1], 0, kOne, e, std::false_type{}); });
  }
  Item it;
  for (int j = first; item(j, &it, false); j += step) {
    const int r0 = it.r0, st = it.st;
    const Part p = part_of(it);
    const bool hyper = HYP && it.b >= 0;
    const int r_end = p.r_end, n_valid = p.n_valid;
    const int vt0 = st * p.strip, vt_end = min(vt0 + p.strip, p.n_vt);      // (hyper part: possibly no tile)
    Triple run[F_N];
    Draw draw[F_N];                                  // MODE 6 only
#pragma unroll
    for (int i = 0; i < F_N; ++i) {
      run[i] = empty_triple();
      draw[i] = empty_draw();
    }
    for (int vt = vt0; vt < vt_end; ++vt) {
      slab_step(std::true_type{});
      for (int slab = 1; slab < it.sn; ++slab) slab_step(std::false_type{});
      if (PROBE_MFMA && vt + 1 < vt_end) continue;
      wait_for_mfma();
      // ---- this vocabulary tile is complete: fold its 128 x 128 logits into the running triples, or store it ------
      int row_base = r0 + wr * 128, col_base = vt * FT + wv * 128 + quarter * 4;
      asm volatile("" : "+v"(col_base), "+v"(row_base));   // (what follows from them is not worked out ahead of the K loop and kept)
      if (MODE == 2) {
        if (it.part >= 0)
          store_partial16(acc, a.split + (ptrdiff_t)it.part * (FT * FT) - ((ptrdiff_t)r0 * FT + vt * FT), FT, row_base, r_end, col_base, n_valid);
        else if (TW && !a.residual)
          store_plain16(acc, a, row_base, r_end, col_base, n_valid);
        else if (!TW && a.stream_f32)
          store_tile16_f32(acc, a, row_base, r_end, col_base, n_valid);
        else
          store_tile16(acc, a, row_base, r_end, col_base, n_valid);
      } else if (MODE == 5) {
        store_partial16(acc, a.partial + (size_t)ks * a.rows * a.ldo, a.ldo, row_base, r_end, col_base, n_valid);
      } else if (MODE == 3) {
        store_prob16(acc, a, hyper ? a.hyper.out : a.out, hyper ? a.hyper.ldo : a.ldo, hyper ? a.hyper.col0 : a.col0, row_base, r_end, col_base,
                     n_valid);
      } else if (MODE == 6) {
        fold_sample16(acc, run, draw, a, row_base, col_base, n_valid);
      } else if (MODE == 7) {
        fold_store16(acc, run, a, row_base, r_end, col_base, n_valid);
      } else {
        if ((vt + 1) * FT > n_valid) mask_tail16(acc, col_base, n_valid);
        fold_tile16(acc, run, col_base, hyper ? a.hyper.col0 : a.col0, n_valid);
      }
    }
    if (MODE >= 2 && MODE <= 5) continue;
    // ---- end of strip: the four quarter-waves hold the same hidden rows; then the two vocabulary halves ------
    // (each exchange halves a lane's rows: 6 merges and no shuffles, where every row merged in all lanes took 16 and 48 and three
    // lanes in four idled behind them.  32000 columns, 300 / 3500 rows, d = 64 33.1 -> 28.2, 92.4 -> 80.1 us, d = 1024 66.0 -> 61.4,
    // 246.9 -> 232.4)
    merge_rows<4>(run, Swap16{});
    merge_rows<2>(run, Swap32{});
    if (MODE == 6) {
      merge_rows<4>(draw, Swap16{});
      merge_rows<2>(draw, Swap32{});
    }
    // (now lane l holds rows (l & 15) + 16 (4 (bit 4 of l) + 2 (bit 5) + e), e = 0, 1)
    const int hrow0 = wr * 128 + (lane & 15) + 16 * (4 * ((lane >> 4) & 1) + 2 * (lane >> 5));
    // (one barrier: the next strip's writes lie behind the barriers of its slabs, and these reads ahead of them)
    Triple* xch = reinterpret_cast<Triple*>(lds + F_LDS_STAGES);    // [256 hidden rows of the tile]
    Draw* xdr = reinterpret_cast<Draw*>(xch + FT);
    if (wv == 1) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        xch[hrow0 + e * 16] = run[e];
        if (MODE == 6) xdr[hrow0 + e * 16] = draw[e];
      }
    }
    barrier_after_lds();
    if (wv == 0) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        merge_triple(run[e], xch[hrow0 + e * 16]);
        const int hrow = r0 + hrow0 + e * 16;
        if (hrow < r_end) {
          const size_t q = (size_t)hrow * a.n_parts + (hyper ? a.hyper.part0 : a.part0) + st;
          a.part_m[q] = run[e].m;
          a.part_s[q] = run[e].s;
          if (MODE == 6) {
            merge_draw(draw[e], xdr[hrow0 + e * 16]);
            a.part_v[q] = draw[e].v;
            a.part_l[q] = draw[e].l;
            a.part_i[q] = draw[e].i;
          } else {
            a.part_i[q] = run[e].i;
          }
        }
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): the requests past the end of the stream land in LDS
}

// The tiles of a dense layer's last round that were cut along K (last_round): out = act(sum of the parts + bias) + residual, 8 rows of a tile
// at a time, a thread 4 columns of 2 of them and eight parts asked for at once.  A workgroup takes pieces of its XCD's tiles, or of all;
// pieces of 16 rows leave CUs without one where 12 tiles have 21 parts each (27 us instead of 17), 4096 workgroups cost 1.5 us where nothing was cut.
constexpr int F_SUM_WGS = 1024;
__global__ void __launch_bounds__(256) tile_sum_kernel(LogitsArgs a) {
  const int rows = a.rows_dev ? min(a.rows, *a.rows_dev) : a.rows;
  const int tiles_each = (rows + FT - 1) / FT, row_tiles = max(a.batch, 1) * tiles_each;
  const int xcd = blockIdx.x & 7;
  const LastRound last = last_round(a, row_tiles, xcd, dense_slabs(a));
  if (last.ways < 2) return;
  const int first = last.whole ? (int)blockIdx.x : (int)(blockIdx.x >> 3), step = last.whole ? F_SUM_WGS : F_SUM_WGS / 8;
  for (int u = first; u < last.rem * (FT / 8); u += step) {
    const int t = u / (FT / 8), trow = u % (FT / 8) * 8 + (int)(threadIdx.x >> 6);
    int rt, st;
    if (last.whole)
      locate_whole(a, row_tiles, t, &rt, &st);
    else if (!locate_base(a, row_tiles, xcd, last.full + t, &rt, &st))
      return;
    const int b = rt / tiles_each, r0 = b * rows + (rt - b * tiles_each) * FT, r_end = (b + 1) * rows;
    const int tcol = 4 * (int)(threadIdx.x & 63), col = st * FT + tcol;
    if (col >= a.w_rows || r0 + trow >= r_end) continue;
    const float4 bias = a.bias ? *reinterpret_cast<const float4*>(a.bias + col) : float4{0.f, 0.f, 0.f, 0.f};
    const float* from = a.split + (size_t)((last.whole ? 0 : xcd * F_XCD_WGS) + t) * (FT * FT) + trow * FT + tcol;
    // (rows that do not exist were not stored: what their place in a buffer holds is read and dropped)
    float4 x[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) x[i] = *reinterpret_cast<const float4*>(from + i * 4 * FT);
#pragma unroll 8
    for (int k = 1; k < last.ways; ++k) {
      from += (size_t)last.rem * (FT * FT);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float4 y = *reinterpret_cast<const float4*>(from + i * 4 * FT);
        x[i] = float4{x[i].x + y.x, x[i].y + y.y, x[i].z + y.z, x[i].w + y.w};
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (r0 + trow + i * 4 < r_end)
        finish_linear(x[i], bias, a.act, a.residual, a.out, a.stream_f32, (size_t)(r0 + trow + i * 4) * a.ldo + col);
  }
}

}  // namespace

unsigned z2z_logits_fast_order(LogitsArgs& a, int forced) {
  // The longer side is walked in blocks, the shorter one inside them: it is the one that the memory-side cache can hold
  // meanwhile.  Both ways 2 x 4 or 4 x 2 for the XCDs is within 1 % (26616 rows x 128256, d = 4096: 19.9 ms, rows in blocks
  // 20.2-20.4; 8 ways along one side 20.9); what counts is 4 x 8 outputs for an XCD's 32 workgroups (2 x 16: 21.4), and that
  // a short side is not dealt out unevenly.  (Up to 4 row tiles meet a weight tile on one XCD, which fetches it once: 300 rows 482 -> 471
  // us, 800 rows 850 -> 839; 6 and 14 row tiles lose 1.5 % that way.)  Against blocks with holes at the edges and one strip of four tiles per
  // workgroup: 128256 x 4096 outputs over K = 32896 27.2 -> 23.3 ms, 35404 x 4096 over 16384 3.60 -> 3.14.
  a.map_p_rows = a.row_tiles > a.n_vtiles;
  const int q = a.map_p_rows ? a.n_strips : a.row_tiles;
  a.map_lp = 4;
  a.map_xq = q > 4 && (q % 2 == 0 || q >= 64) ? 2 : 1;
  if (forced) {
    a.map_p_rows = 1;
    a.map_lp = forced & 0xFF;
    a.map_xq = (forced >> 24) & 0xFF;
  }
  a.map_xp = 8 / a.map_xq;
  // 32 workgroups per XCD (one per CU) walk its list; a short list has fewer
  const int P = a.map_p_rows ? a.row_tiles : a.n_strips;
  const long long main_items = (long long)(P / (a.map_lp * a.map_xp)) * a.map_lp * ((q + a.map_xq - 1) / a.map_xq);
  const long long tail = (long long)(P % (a.map_lp * a.map_xp)) * q;
  const long long longest = main_items + (tail + 7) / 8 + (a.hyper.n_work + 7) / 8;
  return 8u * (unsigned)(longest < 32 ? longest : 32);
}

bool z2z_logits_fast_cuts(const LogitsArgs& a) {
  if (a.rows_dev || a.k_dev) return true;
  for (int xcd = 0; xcd < 8; ++xcd)
    if (last_round(a, a.row_tiles, xcd, a.d * 2 / F_SLAB).ways > 1) return true;
  return false;
}

int z2z_launch_linear_kmajor(const LogitsArgs& a, bool rows_too, unsigned grid, hipStream_t s) {
  if (rows_too)
    hipLaunchKernelGGL((logits_fast_kernel<2, false, true, true>), dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else
    hipLaunchKernelGGL((logits_fast_kernel<2, false, true, false>), dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

int z2z_launch_logits_fast(int mode, const LogitsArgs& a, unsigned grid, hipStream_t s) {
  const bool rot = a.row_tiles == 1;
  if (a.hyper.n_work > 0) {
    if (a.hyper.n_seq > F_HYP_SEQS) return Z2Z_EUNSUPPORTED;
    if (mode == 3)
      hipLaunchKernelGGL((logits_fast_kernel<3, false, false, false, true>), dim3(grid), dim3(F_THREADS), F_HYP_LDS, s, a);
    else if (mode != 0)
      return Z2Z_EUNSUPPORTED;
    else if (rot)
      hipLaunchKernelGGL((logits_fast_kernel<0, true, false, false, true>), dim3(grid), dim3(F_THREADS), F_HYP_LDS, s, a);
    else
      hipLaunchKernelGGL((logits_fast_kernel<0, false, false, false, true>), dim3(grid), dim3(F_THREADS), F_HYP_LDS, s, a);
    Z2Z_HIP_TRY(hipGetLastError());
    return Z2Z_OK;
  }
  if (rot && mode == 0)
    hipLaunchKernelGGL((logits_fast_kernel<0, true>), dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (rot && mode == 6)
    hipLaunchKernelGGL((logits_fast_kernel<6, true>), dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (rot && mode == 7)
    hipLaunchKernelGGL((logits_fast_kernel<7, true>), dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (mode == 9)
    hipLaunchKernelGGL(logits_fast_kernel<9>, dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (mode == 8)
    hipLaunchKernelGGL(logits_fast_kernel<8>, dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (mode == 7)
    hipLaunchKernelGGL(logits_fast_kernel<7>, dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (mode == 6)
    hipLaunchKernelGGL(logits_fast_kernel<6>, dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (mode == 5)
    hipLaunchKernelGGL(logits_fast_kernel<5>, dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (mode == 3)
    hipLaunchKernelGGL(logits_fast_kernel<3>, dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (mode == 2)
    hipLaunchKernelGGL(logits_fast_kernel<2>, dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else if (mode == 1)
    hipLaunchKernelGGL(logits_fast_kernel<1>, dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  else
    hipLaunchKernelGGL(logits_fast_kernel<0>, dim3(grid), dim3(F_THREADS), F_LDS, s, a);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

int z2z_launch_tile_sum(const LogitsArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(tile_sum_kernel, dim3(F_SUM_WGS), dim3(256), 0, s, a);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

int z2z_logits_fast_sequences() { return F_HYP_SEQS; }

int z2z_logits_fast_prepare(z2z_ctx* c) {
  if (c->lds_limit < F_HYP_LDS) return Z2Z_EUNSUPPORTED;
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<0>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<1>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<2>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<3>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<0, false, false, false, true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_HYP_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<0, true, false, false, true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_HYP_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<3, false, false, false, true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_HYP_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<5>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<6>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<7>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<8>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<9>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<2, false, true, false>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<2, false, true, true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<0, true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<6, true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(logits_fast_kernel<7, true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, F_LDS));
  return Z2Z_OK;
}

// Batched token-level LZW for gfx950: one workgroup per sequence, up to 16 waves.
//
// The parse of one sequence is a serial dependency chain (section 2.1 of the zip2zip paper: every
// step looks up "current phrase + next token" in the codebook built so far), so the unit of
// parallelism across workgroups is the sequence.  Inside a sequence a window of up to 1024 positions (encoder) or
// codes (decoder), one per thread, is looked up at once in the codebook as it stood when the window began, and what
// depends on entries made inside the window is found by iterating until nothing changes; the kernels' own comments
// give the argument why the result is that of the one-element-at-a-time loop.
//
// Measured, kernel time encode; decode (before: rounds of 256 elements, four waves, cut at the first element that depends
// on an entry of the round; inputs in the caches): 8 sequences of 4096 tokens, M = 3, cap 2048: 110 -> 44 -> 40 us; 89 -> 32 -> 28 us.
// 4 of 32768, M = 4, cap 8192: 691 -> 211 -> 210; 391 -> 125 -> 85.  16 of 16384, M = 5, cap 16384 (table in memory, its tags in LDS):
// 657 -> 284 -> 187; 449 -> 157 -> 76.  2048 of 1024 to 4096, cap 2048: 224 -> 149 (up to four workgroups on a CU); 163 -> 113 (three).
// 1 of 512: 24 -> 11; 22 -> 8.3.
//
// The codebook is a trie stored as a hash table over its edges: one 64-bit slot = parent code (24 bits)
// | token (24 bits) | entry index (16 bits), two slots per bucket, two buckets per probe step (Table).  The
// workgroup keeps the table of its sequence in LDS for the whole call when it fits (4 slots per entry
// when the 160 KiB of a CU allow, at least 1.25); the decoder also keeps (length, first token) of every
// entry there when it fits.  Tokens and codes are staged in LDS a window ahead.
#include "hyper_embed_common.h"

#include <algorithm>

#include <string.h>

namespace {

constexpr int kWave = 64;
typedef unsigned long long u64;
constexpr u64 kEmpty = ~0ull;

struct LzwArgs {
  LzwState st;
  const int32_t* in;       // tokens (encode) or codes (decode), [B, stride]
  const int32_t* in_len;   // [B] or nullptr
  int32_t stride;
  // APPEND or RESET, compared whole, never masked: the compiler (clang 22 for gfx950) turns `x & 1` that is asked for != 0 and
  // for == 0 in one basic block into one s_bitcmp0_b32 that both answers are read from, so that one of them is inverted (seen
  // in the tag kernels, which then cleared a table that a call continued and kept one that it emptied)
  int32_t flags;
  int32_t* out;            // codes (encode) or tokens (decode), [B, out_stride]
  int32_t* out_n;          // [B]
  int32_t out_stride;
  int32_t* status;         // [B]
  int32_t lds_ef;          // decode, LDS variant: 1 = (length, first token) of the entries live in LDS too
  int32_t by_length;       // window kernels: workgroups take the sequences longest first
  int32_t tail_min;        // decode: codes left behind a full codebook that lzw_decode_tail_kernel takes over
  int32_t in_step;         // one-code-at-a-time decoder only: > 0 = row distance of `in` (else `stride`)
};

// (parents and tokens have at most 24 bits: the 24-bit multiplier runs at full rate, a 32-bit product at a quarter)
__device__ __forceinline__ uint32_t edge_hash(int32_t parent, int32_t tok) {
  uint32_t h = __umul24((uint32_t)parent, 0x9E3779u) + __umul24((uint32_t)tok, 0xC2B2AFu);
  h ^= h >> 15;
  return h * 0x2C1B3C6Du;              // (the upper bits are the well mixed ones)
}

__device__ __forceinline__ u64 edge_bits(int32_t parent, int32_t tok) {
  return ((u64)(uint32_t)parent << 40) | ((u64)(uint32_t)tok << 16);
}

extern __shared__ __align__(16) u64 lds_slots[];   // the sequence's hash table (+ entry info), or its tags

// The hash table of one sequence: in LDS for the length of a call (indexes the shared array directly so that probes
// are ds_read_b128), in global memory (huge capacities, and short appends that touch a few slots), or in global memory
// with a tag of every slot in LDS: 16 bits of the edge's hash.  What a probe in memory costs is requests, two
// of 16 bytes, hit or miss; with the tags a miss is a matter of LDS and a hit one request of 8 bytes, the slot itself.
// (Tags of 32 bits, with the entry's index, left LDS for 28100 slots only, and calls that go to the table in memory all the
// same met it fuller: 2000 tokens appended to a full codebook of 22000 entries, 16 sequences, 44000 -> 28100 slots 13 -> 20 us.)
// 16 sequences of 16384 tokens, cap 16384, M = 5: encode 272 -> 187 us, decode 156 -> 100 (76 by now); 100 of 8192, cap 12000,
// M = 3: 134 -> 91; 109 -> 69 (54).
enum { kMem, kLds, kTag };
template <int WHERE>
struct Table {
  static constexpr bool LDS = WHERE == kLds;
  u64* g;           // global slots of this sequence
  uint32_t n;       // number of slots

  struct Probe {
    uint32_t b0, b1, step, i;
  };
  static __device__ __forceinline__ uint32_t* tags() { return reinterpret_cast<uint32_t*>(lds_slots); }   // a word per bucket
  static __device__ __forceinline__ uint32_t tag_of(uint32_t h) {           // (all ones: no entry has it)
    return min((h >> 2) & 0xFFFFu, 0xFFFEu);
  }
  // The tags of two buckets (slot 0 of a bucket in the low half), and which of them agree with an edge's (bit i: slot i of the four).
  struct Tags {
    uint32_t a, b;
  };
  __device__ __forceinline__ Tags load_tags(uint32_t b0, uint32_t b1) const { return {tags()[b0], tags()[b1]}; }
  static __device__ __forceinline__ uint32_t agree(const Tags& t, uint32_t tag) {
    const uint32_t x = t.a ^ (tag * 0x10001u), y = t.b ^ (tag * 0x10001u);
    return ((x & 0xFFFFu) == 0 ? 1u : 0u) | (x < 0x10000u ? 2u : 0u) | ((y & 0xFFFFu) == 0 ? 4u : 0u) | (y < 0x10000u ? 8u : 0u);
  }
  // Claims slot `at`, empty in the tags read: fails when another lane has claimed a slot of the bucket since.
  static __device__ __forceinline__ bool claim(const Probe& p, const Tags& t, int at, uint32_t tag) {
    const uint32_t old = (uint32_t)(at >> 1) == p.b0 ? t.a : t.b, shift = (at & 1) * 16;
    return atomicCAS(&tags()[at >> 1], old, old ^ ((tag ^ 0xFFFFu) << shift)) == old;
  }

  // Two slots are a bucket (n is even): one 16-byte read.  A probe step looks at two buckets at once, and a new
  // edge goes into the emptier one (slot 0 of a bucket first), so hardly any look-up needs a second step: with the
  // table half full the longest of 64 simultaneous probes takes two, where a one-bucket probe sequence took six.  The
  // first kJumps buckets of a sequence are `step` (a second hash) apart, the rest follow one by one, which reaches
  // every bucket whatever n is.  A look-up ends at the first step with an empty slot.
  static constexpr uint32_t kJumps = 8;
  __device__ __forceinline__ uint32_t hop(uint32_t bucket, uint32_t by) const {
    bucket += by;
    return min(bucket, bucket - (n >> 1));          // (unsigned: the subtraction wraps unless bucket is past the end)
  }
  __device__ __forceinline__ Probe probe_init(uint32_t h) const {
    Probe p;
    p.step = 1 + ((h >> 4) & 30);                   // odd, at most 31 < n / 2 (n >= 64)
    p.b0 = __umulhi(h, n >> 1);
    p.b1 = hop(p.b0, p.step);
    p.i = 0;
    return p;
  }
  __device__ __forceinline__ bool probe_next(Probe* p) const {
    p->i += 2;
    const uint32_t by = p->i < kJumps ? p->step : 1;
    p->b0 = hop(p->b1, by);
    p->b1 = hop(p->b0, by);
    return p->i < (n >> 1) + kJumps + 2;
  }
  // (the global table is read past the vector L1 everywhere: slots are claimed with atomics, which do not
  // update that cache, so a line it holds can be stale)
  // A bucket is one 16-byte request (atomic loads have 8 bytes at most; what a probe in memory costs is requests).
  __device__ __forceinline__ void load(const Probe& p, ulonglong2* a, ulonglong2* b) const {
    if (LDS) {
      *a = *reinterpret_cast<const ulonglong2*>(&lds_slots[2 * p.b0]);
      *b = *reinterpret_cast<const ulonglong2*>(&lds_slots[2 * p.b1]);
      return;
    }
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 x, y;
    asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %3, off sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(x), "=&v"(y)
                 : "v"(g + 2 * p.b0), "v"(g + 2 * p.b1)
                 : "memory");
    a->x = ((u64)x[1] << 32) | x[0];
    a->y = ((u64)x[3] << 32) | x[2];
    b->x = ((u64)y[1] << 32) | y[0];
    b->y = ((u64)y[3] << 32) | y[2];
  }
  __device__ __forceinline__ void store(uint32_t pos, u64 v) const {
    if (WHERE == kTag) {
      reinterpret_cast<uint16_t*>(tags())[pos] = (uint16_t)tag_of(edge_hash((int32_t)(v >> 40), (int32_t)((v >> 16) & 0xFFFFFFu)));
      g[pos] = v;
    } else if (LDS)
      lds_slots[pos] = v;
    else
      __hip_atomic_store(&g[pos], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // Slot of the emptier of two buckets, -1 if both are full.
  static __device__ __forceinline__ int free_slot(const Probe& p, const ulonglong2& a, const ulonglong2& b) {
    if (a.x == kEmpty) return (int)(2 * p.b0);
    if (b.x == kEmpty) return (int)(2 * p.b1);
    if (a.y == kEmpty) return (int)(2 * p.b0 + 1);
    if (b.y == kEmpty) return (int)(2 * p.b1 + 1);
    return -1;
  }
  static __device__ __forceinline__ int free_slot(const Probe& p, const Tags& t) {
    if ((t.a & 0xFFFFu) == 0xFFFFu) return (int)(2 * p.b0);
    if ((t.b & 0xFFFFu) == 0xFFFFu) return (int)(2 * p.b1);
    if (t.a >= 0xFFFF0000u) return (int)(2 * p.b0 + 1);
    if (t.b >= 0xFFFF0000u) return (int)(2 * p.b1 + 1);
    return -1;
  }
  // The entry of an edge whose tag some slots of a probe have, or -1: the slots themselves decide.
  __device__ __forceinline__ int confirm(const Probe& p, uint32_t which, u64 key) const {
    for (; which != 0; which &= which - 1) {
      const int i = __builtin_ctz(which);
      const u64 slot = g[2 * (i < 2 ? p.b0 : p.b1) + (i & 1)];
      if (holds(slot, key)) return (int)((uint32_t)slot & 0xFFFFu);
    }
    return -1;
  }
  static __device__ __forceinline__ bool holds(u64 slot, u64 key) {
    return (uint32_t)(slot >> 32) == (uint32_t)(key >> 32) && ((uint32_t)slot ^ (uint32_t)key) < 0x10000u;
  }
  static __device__ __forceinline__ int match(const ulonglong2& a, const ulonglong2& b, u64 key) {
    int idx = -1;
    if (holds(a.x, key)) idx = (int)((uint32_t)a.x & 0xFFFFu);
    if (holds(a.y, key)) idx = (int)((uint32_t)a.y & 0xFFFFu);
    if (holds(b.x, key)) idx = (int)((uint32_t)b.x & 0xFFFFu);
    if (holds(b.y, key)) idx = (int)((uint32_t)b.y & 0xFFFFu);
    return idx;
  }
  static __device__ __forceinline__ u64 uniform(u64 v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((u64)hi << 32) | lo;
  }
  // Wave-uniform look-up (every lane reads the same address; the chain stays in scalar registers).  Returns the
  // entry index, or -1 with *free_pos = the slot the edge would get (-1 if the table has no empty slot, which
  // cannot happen while n > cap).
  __device__ __forceinline__ int find(int32_t parent, int32_t tok, int* free_pos) const {
    const u64 key = edge_bits(parent, tok);
    Probe p = probe_init(edge_hash(parent, tok));
    do {
      if (WHERE == kTag) {
        const Tags t = load_tags(p.b0, p.b1);
        const int idx = __builtin_amdgcn_readfirstlane(confirm(p, agree(t, tag_of(edge_hash(parent, tok))), key));
        if (idx >= 0) return idx;
        *free_pos = __builtin_amdgcn_readfirstlane(free_slot(p, t));
        if (*free_pos >= 0) return -1;
        continue;
      }
      ulonglong2 a, b;
      load(p, &a, &b);
      a.x = uniform(a.x);
      a.y = uniform(a.y);
      b.x = uniform(b.x);
      b.y = uniform(b.y);
      const int idx = match(a, b, key);
      if (idx >= 0) return idx;
      *free_pos = free_slot(p, a, b);
      if (*free_pos >= 0) return -1;
    } while (probe_next(&p));
    return -1;
  }
  // The same look-up per lane (each lane its own edge; h = edge_hash(parent, tok)).
  __device__ __forceinline__ int find_lane(int32_t parent, int32_t tok, uint32_t h) const {
    const u64 key = edge_bits(parent, tok);
    Probe p = probe_init(h);
    do {
      if (WHERE == kTag) {
        const Tags t = load_tags(p.b0, p.b1);
        const uint32_t which = agree(t, tag_of(h));
        if (which != 0) {
          const int idx = confirm(p, which, key);
          if (idx >= 0) return idx;
        }
        if (t.a >= 0xFFFF0000u || t.b >= 0xFFFF0000u) return -1;
        continue;
      }
      ulonglong2 a, b;
      load(p, &a, &b);
      const int idx = match(a, b, key);
      if (idx >= 0) return idx;
      if (a.y == kEmpty || b.y == kEmpty) return -1;
    } while (probe_next(&p));
    return -1;
  }
  __device__ __forceinline__ int find_lane(int32_t parent, int32_t tok) const {
    return find_lane(parent, tok, edge_hash(parent, tok));
  }
  // Per-lane insertion of an edge that may be there, or be inserted by another lane at the same time: of several lanes with
  // one edge, one claims a slot (returned) and the others find it (-1; with tags also, now and then, where it is not so: the
  // slot of a tag claimed in this phase may not be readable yet).  -2: no empty slot, which cannot happen while n > cap.
  __device__ __forceinline__ int insert_new(int32_t parent, int32_t tok, int idx) const {
    const u64 key = edge_bits(parent, tok), val = key | (u64)(uint32_t)idx;
    const uint32_t h = edge_hash(parent, tok);
    Probe p = probe_init(h);
    do {
      for (int tries = 0; tries < 5; ++tries) {     // (a claim is lost when one of the four slots has filled: at most four times)
        int at;
        if (WHERE == kTag) {
          const Tags t = load_tags(p.b0, p.b1);
          for (uint32_t which = agree(t, tag_of(h)); which != 0; which &= which - 1) {
            const int i = __builtin_ctz(which);
            const u64 slot = g[2 * (i < 2 ? p.b0 : p.b1) + (i & 1)];
            if (slot == kEmpty || holds(slot, key)) return -1;
          }
          at = free_slot(p, t);
          if (at < 0) break;
          if (claim(p, t, at, tag_of(h))) {
            g[at] = val;
            return at;
          }
        } else {
          ulonglong2 a, b;
          load(p, &a, &b);
          if (match(a, b, key) >= 0) return -1;
          at = free_slot(p, a, b);
          if (at < 0) break;
          if (atomicCAS(LDS ? &lds_slots[at] : &g[at], kEmpty, val) == kEmpty) return at;
        }
      }
    } while (probe_next(&p));
    return -2;
  }
  __device__ __forceinline__ void remove(int at) const {
    if (WHERE == kTag) atomicOr(&tags()[at >> 1], 0xFFFFu << ((at & 1) * 16));
    if (LDS)
      lds_slots[at] = kEmpty;
    else
      __hip_atomic_store(&g[at], kEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // Per-lane insertion of an edge known to be absent (several lanes insert at once: a slot is claimed with a
  // compare-and-swap, and the buckets are looked at again when it was lost).
  __device__ __forceinline__ void insert_lane(int32_t parent, int32_t tok, int idx) const {
    const u64 val = edge_bits(parent, tok) | (u64)(uint32_t)idx;
    const uint32_t h = edge_hash(parent, tok);
    Probe p = probe_init(h);
    do {
      for (int tries = 0; tries < 5; ++tries) {     // (a claim is lost when one of the four slots has filled: at most four times)
        if (WHERE == kTag) {
          const Tags t = load_tags(p.b0, p.b1);
          const int at = free_slot(p, t);
          if (at < 0) break;
          if (claim(p, t, at, tag_of(h))) {
            g[at] = val;
            return;
          }
          continue;
        }
        ulonglong2 a, b;
        load(p, &a, &b);
        const int at = free_slot(p, a, b);
        if (at < 0) break;
        if (atomicCAS(LDS ? &lds_slots[at] : &g[at], kEmpty, val) == kEmpty) return;
      }
    } while (probe_next(&p));
  }
};

// A workgroup barrier that other waves' reads PAST the vector L1 may rely on.  Between the waves of a workgroup
// plain stores and plain loads are ordered by the L1 they share, and the barrier does not wait for the stores
// to leave it; a load that goes straight to L2 (the table's) could overtake a store of another wave that is still on
// its way there.  So the stores are awaited before the barrier.  (Slots claimed with atomics need no such wait: the
// claiming thread has waited for the old value.)
__device__ __forceinline__ void sync_after_global_stores() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// The one-wave helpers (table_open / table_close, lzw_decode_serial_body) are run by exactly one
// wave: the whole workgroup of the 64-thread kernels, or wave 0 of the step-update kernel.  What they need between their steps is that the lanes' earlier LDS and
// global accesses have completed, not a meeting of waves, so they never execute a workgroup barrier: a fence at
// workgroup scope (the waits for the outstanding memory operations) and a wave barrier (keeps the compiler from
// moving memory operations across).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

template <int LDS>
__device__ __forceinline__ void table_open(const LzwArgs& a, int b, int lane, bool reset, Table<LDS>* t) {
  const LzwState& st = a.st;
  t->g = st.slots + (size_t)b * st.nslots;
  t->n = (uint32_t)st.nslots;
  if (LDS) {
    if (reset) {
      for (int i = lane; i < st.nslots; i += kWave) lds_slots[i] = kEmpty;
    } else {
      for (int i = lane; i < st.nslots; i += kWave) lds_slots[i] = t->g[i];
    }
    wave_sync();
  } else if (reset) {
    // plain stores; the probes read past the L1 (atomic loads), so the stores are awaited first
    for (int i = lane; i < st.nslots; i += kWave) t->g[i] = kEmpty;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    wave_sync();
  }
}

// The same by all THREADS threads of a workgroup; no barrier inside.  (probed: whether a look-up can come)
template <int WHERE, int THREADS>
__device__ __forceinline__ void table_open_all(const LzwArgs& a, int b, int tid, bool reset, Table<WHERE>* t, bool probed = true) {
  t->g = a.st.slots + (size_t)b * a.st.nslots;
  t->n = (uint32_t)a.st.nslots;
  ulonglong2* g2 = reinterpret_cast<ulonglong2*>(t->g);             // (nslots is even, the rows 16-byte aligned)
  ulonglong2* l2 = reinterpret_cast<ulonglong2*>(lds_slots);
  const int pairs = a.st.nslots >> 1;
  const ulonglong2 empty = {kEmpty, kEmpty};
  if (WHERE == kLds) {
    for (int i = tid; i < pairs; i += THREADS) l2[i] = reset ? empty : g2[i];
  } else if (reset) {
    for (int i = tid; i < pairs; i += THREADS) g2[i] = empty;
  }
  if (WHERE == kTag && probed) {
    uint32_t* tags = t->tags();
    if (reset) {
      for (int i = tid; i < pairs; i += THREADS) tags[i] = ~0u;
    } else {
      auto tag = [&](u64 v) -> uint32_t {
        return v == kEmpty ? 0xFFFFu : t->tag_of(edge_hash((int32_t)(v >> 40), (int32_t)((v >> 16) & 0xFFFFFFu)));
      };
      for (int i = tid; i < pairs; i += THREADS) tags[i] = tag(g2[i].x) | tag(g2[i].y) << 16;
    }
  }
}
template <int WHERE, int THREADS>
__device__ __forceinline__ void table_close_all(int tid, const Table<WHERE>& t) {
  if (WHERE == kLds) {
    ulonglong2* g2 = reinterpret_cast<ulonglong2*>(t.g);
    const ulonglong2* l2 = reinterpret_cast<const ulonglong2*>(lds_slots);
    for (int i = tid; i < (int)(t.n >> 1); i += THREADS) g2[i] = l2[i];
  }
}

template <int LDS>
__device__ __forceinline__ void table_close(const LzwArgs& a, int lane, const Table<LDS>& t) {
  if (LDS) {
    wave_sync();
    for (int i = lane; i < a.st.nslots; i += kWave) t.g[i] = lds_slots[i];
  }
}

// Add the edge (parent, tok) as entry C.  `ph` holds, in lane j, token j of the parent phrase (plen
// tokens); the new entry's flattened row is that phrase followed by tok.
template <int LDS>
__device__ __forceinline__ void table_insert(const LzwArgs& a, int b, int lane, const Table<LDS>& t, int free_pos,
                                             int C, int32_t parent, int32_t tok, int32_t ph, int plen) {
  const LzwState& st = a.st;
  if (lane == 0) {
    t.store((uint32_t)free_pos, edge_bits(parent, tok) | (u64)(uint32_t)C);
    st.ent_len[(size_t)b * st.cap + C] = plen + 1;
  }
  if (lane < st.M) {
    const int32_t v = lane < plen ? ph : (lane == plen ? tok : -1);
    st.ent_tokens[((size_t)b * st.cap + C) * st.M + lane] = v;
  }
}

// ------------------------------------------------------------------------------------------------
// encode
//
// The greedy parse is the solution of a recurrence over positions: the match at a phrase start is the longest one
// in the codebook as it stood when the round began plus the entries that earlier starts of the round make, and
// the starts are the positions reached from the first by start -> start + length.  A round takes a window of one
// position per thread and finds that solution by iteration, instead of cutting the window at the first start that
// depends on an entry made inside it:
//   1. every position follows its chain of lookups token -> (code, next token) -> ... in the table as it stands
//      (at most M-1 probes): (L0, c0), the match without this round's entries.
//   2. starts from lengths.  "Positions still to skip" is a state in 0..M-1 and position i a function of it:
//      s -> s-1, 0 -> L-1.  A function is M bytes and v_perm_b32 composes two of them (one instruction up to
//      M = 4, two up to 8), so the starts are a DPP scan over the wave's lanes, one LDS exchange of the waves'
//      compositions, and a scan over those.
//   3. every start whose match may grow puts its edge (its code, next token) into an LDS hash set that keeps the
//      lowest position per edge; an entry of this round is named by the position of the start that makes it.
//   4. every position extends (L0, c0) through the set by edges of lower positions.  If no start's match
//      changed, lengths, starts and edges satisfy the recurrence and are the parse (by induction over the
//      positions: each depends on lower ones only); else back to 2.  The lowest start that is not final yet
//      becomes final with every iteration, so the loop ends; one to three iterations are usual, as a parse falls
//      back into step soon after a changed length.
//   5. publish: entry numbers are ranks of the proposing starts; codes, table insertions (compare-and-swap) and
//      flattened rows from the staged tokens.
// A window is cut only by a token out of range, the end of the output row and the entry that fills the codebook;
// with the codebook full the iteration is a single scan.  Order of entries and matches are those of the
// one-token-at-a-time parse.
//
// What bounds it: instruction issue and LDS latency of one CU (a window of 1024 is four waves per SIMD, so an
// instruction costs 16 cycles; chains ~3500 cycles a window, an iteration ~5000, publishing ~4000).  Wider windows have
// fewer rounds and hardly more iterations: a 4096-token sequence at M = 3 takes 28 rounds of 256 positions cut at the
// first repeat, but 5 windows of 1024 with 13 iterations in all.
// ------------------------------------------------------------------------------------------------
constexpr int kShortAppend = 64;
// Tags of a table in memory have to be made from all of its slots when a call continues a codebook (256 KB for a CU to
// read at cap 16384), which only entries to come make up for: an appended call has them made from kTagAppendTokens tokens
// (kTagAppendCodes codes) on, and where the codebook has room for so many codes' entries.  Table in memory -> tags, us:
//   room   200 sequences, cap 16384: encode 513 tokens 20 -> 26, 1024 27 -> 32, 1500 37 -> 39, 2048 44 -> 42, 4096 75 -> 64; decode of their
//          codes (280, 560, 830, 1130, 2260) 14 -> 21, 19 -> 23, 27 -> 24, 33 -> 29, 52 -> 37
//          16 sequences, cap 22000: encode 1024 22 -> 23, 1500 31 -> 30, 2048 35 -> 32; decode 16 -> 18, 17 -> 18, 24 -> 22
//   full   16 sequences, cap 12000: encode 1024 tokens 11 -> 14, 4096 27 -> 31, 16384 88 -> 93; decode 8 -> 12, 14 -> 17 (nothing is
//          looked up there: the tag kernel without tags, 8 and 13)
// (An emptied codebook has its tags for nothing: 513 tokens 42 -> 37 and 30 -> 24.)
constexpr int kTagAppendTokens = 2048, kTagAppendCodes = 1024;

// Number of elements of sequence b in this call.
__device__ __forceinline__ int call_length(const LzwArgs& a, int b) {
  return a.in_len ? min(max(__builtin_amdgcn_readfirstlane(a.in_len[b]), 0), a.stride) : a.stride;
}

// The sequence workgroup r of a window kernel works on.  With a few rounds of workgroups on every CU the last ones to
// start decide when a call with ragged lengths ends, so they should be the shortest: the r-th in the order of 16 classes
// of length, longest first, and inside a class in the order (wave, turn, lane) of the threads that look at the lengths.
// Every workgroup finds its own (about 2 us of the 50 and more that a long document takes; as a launch of its own it would be 5).
// Short rows end together and only pay for it: 2048 rows of up to 400 tokens, as they come -> in order, 38 -> 41 us, of 700 52 -> 51, of
// 1000 63 -> 59; decode of 1000 46 -> 49.
// 2048 documents of 1024 to 4096 tokens, cap 2048, three workgroups per CU: 199 -> 181 us.
// Every workgroup looks at all lengths, so that the cost of a call grows with B squared, where the gain is a share of the last
// round of workgroups.  Lengths from 0 to N, as they come -> in order, us:
//   encode  N = 700   B = 2048 54 -> 52    3072 71 -> 72    16384 294 -> 503    32768 561 -> 1422
//           N = 2100      2048 99 -> 85    4096 162 -> 155  16384 508 -> 707 (from N / 4 on)
//           N = 4096      2048 164 -> 127  4096 265 -> 232
//   decode  N = 2100      2048 72 -> 67    3072 94 -> 97    16384 371 -> 668
//           N = 4096      2048 121 -> 98   3072 160 -> 145  4096 200 -> 192 (from N / 4 on: 234 -> 237)
// Hence up to eight (decode: four) sequences per CU and half the row's length more, sixteen per CU at most.
constexpr int kLengthBins = 16;
struct BlockOrder {
  int32_t bin[kLengthBins];
  int32_t count[16];                           // of each wave, in the class that holds r
  int32_t seq;
};
template <int NW>
__device__ __forceinline__ int sequence_of_block(const LzwArgs& a, BlockOrder& sh) {
  if (!a.by_length) return blockIdx.x;
  constexpr int THREADS = NW * kWave;
  const int B = gridDim.x, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float scale = (float)kLengthBins / ((float)a.stride + 1.0f);
  auto bin_of = [&](int i) -> int {            // -1 past the end
    if (i >= B) return -1;
    const int len = min(max(a.in_len[i], 0), a.stride);
    return kLengthBins - 1 - min((int)((float)len * scale), kLengthBins - 1);
  };
  if (tid < kLengthBins) sh.bin[tid] = 0;
  if (tid == 0) sh.seq = blockIdx.x;           // (found below as long as nobody writes to the lengths meanwhile: see plan)
  __syncthreads();
  for (int i = tid; i < B; i += THREADS) atomicAdd(&sh.bin[bin_of(i)], 1);
  __syncthreads();
  int mine = 0, rank = blockIdx.x;
  while (mine < kLengthBins - 1 && rank >= sh.bin[mine]) rank -= sh.bin[mine++];
  mine = __builtin_amdgcn_readfirstlane(mine);
  rank = __builtin_amdgcn_readfirstlane(rank);
  int count = 0;
  for (int base = 0; base < B; base += THREADS) count += (int)__popcll(__ballot(bin_of(base + tid) == mine));
  if (lane == 0) sh.count[w] = count;
  __syncthreads();
  for (int j = 0; j < w; ++j) rank -= sh.count[j];
  if (rank >= 0 && rank < count) {
    for (int base = 0; base < B; base += THREADS) {
      const unsigned long long m = __ballot(bin_of(base + tid) == mine);
      const int c = (int)__popcll(m);
      if (rank < c) {
        if (bin_of(base + tid) == mine && (int)__popcll(m & ((1ull << lane) - 1)) == rank) sh.seq = base + tid;
        break;
      }
      rank -= c;
    }
  }
  __syncthreads();
  const int b = __builtin_amdgcn_readfirstlane(sh.seq);
  __syncthreads();                             // (the kernel's own shared memory may lie over this)
  return b;
}

// The skip function of one position or of a run of positions: byte s = state after it, for state s before it.
struct SkipFn {
  uint32_t lo, hi;
};
constexpr uint32_t kSkipIdLo = 0x03020100u, kSkipIdHi = 0x07060504u;

template <bool M4>
__device__ __forceinline__ SkipFn skip_then(SkipFn first, SkipFn second) {
  SkipFn r;
  r.lo = __builtin_amdgcn_perm(second.hi, second.lo, first.lo);
  r.hi = M4 ? kSkipIdHi : __builtin_amdgcn_perm(second.hi, second.lo, first.hi);
  return r;
}

// One step of a scan over lanes: every lane that has a source under the DPP control composes it before its own.
template <bool M4, int CTRL, int ROW_MASK>
__device__ __forceinline__ SkipFn skip_scan_step(SkipFn f) {
  SkipFn g;
  g.lo = __builtin_amdgcn_update_dpp(kSkipIdLo, f.lo, CTRL, ROW_MASK, 0xf, false);
  g.hi = M4 ? kSkipIdHi : __builtin_amdgcn_update_dpp(kSkipIdHi, f.hi, CTRL, ROW_MASK, 0xf, false);
  return skip_then<M4>(g, f);
}
template <bool M4>
__device__ __forceinline__ SkipFn skip_scan16(SkipFn f) {         // inclusive, inside each row of 16 lanes
  f = skip_scan_step<M4, 0x111, 0xf>(f);                          // row_shr:1, 2, 4, 8
  f = skip_scan_step<M4, 0x112, 0xf>(f);
  f = skip_scan_step<M4, 0x114, 0xf>(f);
  return skip_scan_step<M4, 0x118, 0xf>(f);
}
template <bool M4>
__device__ __forceinline__ SkipFn skip_scan64(SkipFn f) {         // inclusive, over the wave
  f = skip_scan16<M4>(f);
  f = skip_scan_step<M4, 0x142, 0xa>(f);                          // row_bcast:15 into rows 1 and 3
  return skip_scan_step<M4, 0x143, 0xc>(f);                       // row_bcast:31 into rows 2 and 3
}

template <int CTRL>
__device__ __forceinline__ uint32_t row_add_step(uint32_t v) {
  return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
// Sums over the waves of a workgroup of up to 16: every lane l < NW holds wave l's value in, the sum of waves 0..l out.
__device__ __forceinline__ uint32_t row_scan_add(uint32_t v) {
  v = row_add_step<0x111>(v);
  v = row_add_step<0x112>(v);
  v = row_add_step<0x114>(v);
  return row_add_step<0x118>(v);
}

// The per-round set of proposed edges: for every edge the lowest position that proposes it.  A slot is 32 bits,
// 21 bits of the edge's hash | 11 bits of position (all ones: empty); four slots are a group, read at once, and an
// edge lives in one of two groups that its hash names, so a look-up is two 16-byte reads whatever the load, no loop.
// key[position] is the edge itself (parent: a code, or kRoundEntry | position for an entry of this round).
constexpr int32_t kRoundEntry = 1 << 24;
constexpr uint32_t kRoundPos = 0x7FFu, kRoundEmpty = ~0u;
__device__ __forceinline__ u64 round_key(int32_t parent, int32_t tok) { return ((u64)(uint32_t)parent << 32) | (uint32_t)tok; }
template <int SLOTS>
struct RoundSet {
  static constexpr int kGroups = SLOTS / 4;
  static constexpr int kGroupBits = __builtin_ctz(kGroups);
  static __device__ __forceinline__ void groups(uint32_t h, uint32_t* a, uint32_t* b) {
    *a = h >> (32 - kGroupBits);
    *b = *a ^ (((h >> 2) & (kGroups - 1)) | 1);
  }
  // Insert; returns the slot this thread claimed (it empties it later), -1 when the edge was there already, and -2 when
  // both groups are full of other edges.
  static __device__ __forceinline__ int insert(uint32_t* set, u64* key, uint32_t h, u64 kk, int pos) {
    uint32_t ga, gb;
    groups(h, &ga, &gb);
    key[pos] = kk;
    asm volatile("" ::: "memory");             // (a wave's LDS operations execute in order: the key is there before the slot)
    const uint32_t val = (h << 11) | (uint32_t)pos;
    uint32_t at = 4 * ga;
    for (uint32_t i = 0; i < 8; ++i) {
      const uint32_t idx = at + ((h + i) & 3);
      const uint32_t old = atomicCAS(&set[idx], kRoundEmpty, val);
      if (old == kRoundEmpty) return (int)idx;
      if ((old ^ val) <= kRoundPos && key[old & kRoundPos] == kk) {
        atomicMin(&set[idx], val);
        return -1;
      }
      if (i == 3) at = 4 * gb;
    }
    return -2;
  }
  // The lowest position below `pos` that proposes the edge, or -1.
  static __device__ __forceinline__ int find(const uint32_t* set, const u64* key, uint32_t h, u64 kk, int pos) {
    uint32_t ga, gb;
    groups(h, &ga, &gb);
    const uint4 a = reinterpret_cast<const uint4*>(set)[ga], b = reinterpret_cast<const uint4*>(set)[gb];
    const uint32_t tag = h << 11;
    const uint32_t x[8] = {a.x ^ tag, a.y ^ tag, a.z ^ tag, a.w ^ tag, b.x ^ tag, b.y ^ tag, b.z ^ tag, b.w ^ tag};
    const uint32_t m = min(min(min(x[0], x[1]), min(x[2], x[3])), min(min(x[4], x[5]), min(x[6], x[7])));
    if (m >= (uint32_t)pos) return -1;         // (an empty slot reads as a position of 2047 at least)
    if (key[m] == kk) return (int)m;
    int best = -1;                             // 21 bits agree, the edges differ: look at every slot
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (x[i] < (uint32_t)pos && (best < 0 || x[i] < (uint32_t)best) && key[x[i]] == kk) best = (int)x[i];
    return best;
  }
};

constexpr int kMaxWaves = 16;
template <int NW, int SETS, int PER = 4>
struct EncShared {
  static constexpr int W = NW * kWave;       // positions of a window
  static constexpr int kSet = PER * W;       // slots of a set
  uint32_t set[SETS][kSet];                  // edges proposed (two sets: in an even / odd iteration)
  u64 key[W];
  u64 skip[kMaxWaves];                       // skip function of each wave's positions
  int32_t tok[2 * W];                        // ring of token classes: position p at p & (2 W - 1)
  uint32_t count[kMaxWaves];                 // starts | proposals << 16 of each wave
  uint32_t count_valid[kMaxWaves];           // the same below the window's limit (cut windows only)
  int32_t changed[2];
  int32_t cut_asked;                         // the window holds a token out of range, or an edge found no slot
  int32_t bad_pos, ovf_pos, full_pos, spill_pos;   // where a window is cut
  int32_t last_code, last_len, last_end;     // the last phrase of the window
  uint16_t rank[W];                          // of the proposing starts
};

// What a kernel has of its own in LDS, for the room it leaves to a table: the size of its shared structure, and alignment.
constexpr int own_lds(size_t shared) { return (int)shared + 256; }
constexpr int kParseStaticLds = own_lds(sizeof(EncShared<kMaxWaves, 2>));
constexpr int kWideSets16 = own_lds(sizeof(EncShared<16, 2, 8>)), kWideSets8 = own_lds(sizeof(EncShared<8, 2, 8>));

template <int NW, int SETS, int PER, int WHERE, bool M4>
__device__ __forceinline__ void lzw_encode_windows(const LzwArgs& a, int b, EncShared<NW, SETS, PER>& sh) {
  constexpr int W = NW * kWave;
  constexpr int kSet = EncShared<NW, SETS, PER>::kSet, kRing = 2 * W;
  typedef RoundSet<kSet> Set;
  const LzwState& st = a.st;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int V = st.V, M = st.M, cap = st.cap;
  const bool reset = a.flags == Z2Z_RESET;

  const int size0 = __builtin_amdgcn_readfirstlane(st.size[b]);
  int C = reset ? 0 : size0;
  int prev = reset ? -1 : __builtin_amdgcn_readfirstlane(st.prev_code[b]);
  int prev_len = reset ? 0 : __builtin_amdgcn_readfirstlane(st.prev_len[b]);
  const int n = call_length(a, b);
  const int32_t* in = a.in + (size_t)b * a.stride;
  int32_t* out = a.out + (size_t)b * a.out_stride;
  int32_t* ent_tokens = st.ent_tokens + (size_t)b * cap * M;
  int32_t* ent_len = st.ent_len + (size_t)b * cap;

  Table<WHERE> t;
  table_open_all<WHERE, W>(a, b, tid, reset, &t);
  if (C < cap) {                      // (behind a full codebook nothing is proposed)
    for (int i = tid; i < SETS * kSet; i += W) sh.set[0][i] = kRoundEmpty;
  }
  // tokens: the ring holds [fill - kRing, fill); the next W of them wait in a register
  auto classify = [&](int32_t v) -> int32_t { return (v >= 0 && v < V) ? v : -2; };
  int fill = kRing;
  for (int i = tid; i < kRing; i += W) sh.tok[i] = i < n ? classify(in[i]) : -1;
  int32_t ahead = fill + tid < n ? in[fill + tid] : 0;
  if (tid == 0) sh.changed[0] = sh.changed[1] = 0;
  sync_after_global_stores();        // (a table cleared in global memory is read past the L1)

  int status = 0;
  int n_out = 0;

  // An appended call: the entry "last emitted phrase + first token of this call", which the earlier
  // flush could not add, is added now if it is legal and absent.
  if (n > 0 && prev >= 0 && prev_len < M && C < cap) {
    const int32_t c = __builtin_amdgcn_readfirstlane(in[0]);
    if (c >= 0 && c < V) {
      int free_pos = -1;
      const int idx = t.find(prev, c, &free_pos);
      __syncthreads();     // every wave has looked before wave 0 inserts (else a late wave finds the new edge)
      if (idx < 0 && free_pos >= 0) {
        if (w == 0) {
          int32_t ph = -1;        // lane j = token j of the previous phrase
          if (prev < V) {
            ph = lane == 0 ? prev : -1;
          } else if (lane < M) {
            ph = ent_tokens[(size_t)(prev - V) * M + lane];
          }
          table_insert<WHERE>(a, b, lane, t, free_pos, C, prev, c, ph, prev_len);
        }
        ++C;
      }
    }
    sync_after_global_stores();
  }

  bool stop = false;
  int pos = 0;                        // first position not yet covered by an emitted phrase
  int n_rounds = 0;
  while (pos < n && !stop) {
    auto tk = [&](int d) -> int32_t {           // token class at this thread's position + d, -1 past the end
      const int p = pos + tid + d;
      return p < n ? sh.tok[p & (kRing - 1)] : -1;
    };
    if (tid == 0) {
      sh.bad_pos = sh.ovf_pos = sh.full_pos = sh.spill_pos = W;
      sh.cut_asked = 0;               // (this window's: set behind the barrier below, read in step 5)
    }

    // ---- 1. chains against the table of the round's start -------------------------------------------
    const int32_t tok0 = tk(0);
    int L0 = tok0 >= 0 ? 1 : 0;
    int32_t c0 = tok0;
    int32_t nxt0 = tk(1);             // always the token that follows this position's match
    uint32_t h0 = edge_hash(c0, nxt0);
    for (int d = 1; d < M; ++d) {
      const int32_t after = tk(d + 1);
      int idx = -1;
      if (L0 == d && nxt0 >= 0) idx = t.find_lane(c0, nxt0, h0);
      if (__ballot(idx >= 0) == 0) break;
      if (idx >= 0) {
        c0 = V + idx;
        L0 = d + 1;
        nxt0 = after;
        h0 = edge_hash(c0, nxt0);
      }
    }

    const int avail = min(W, n - pos);
    const int room = cap - C;
    int L = L0;
    int32_t code = c0, nxt = nxt0;
    uint32_t h = h0;
    bool start = false, cand = false;
    u64 start_mask = 0, cand_mask = 0;
    int overrun = 0;                  // positions of the next window that the last phrase covers
    int own = -1;                     // the slot this thread claimed in the set of this iteration
    SkipFn before;                    // skip function of the lanes below
    auto skip_functions = [&]() {
      SkipFn f = {0x02010000u | (uint32_t)(max(L, 1) - 1), 0x06050403u};
      f = skip_scan64<M4>(f);
      if (lane == kWave - 1) sh.skip[w] = ((u64)f.hi << 32) | f.lo;
      before.lo = __builtin_amdgcn_update_dpp(kSkipIdLo, f.lo, 0x138, 0xf, 0xf, false);        // wave_shr:1
      before.hi = M4 ? kSkipIdHi : __builtin_amdgcn_update_dpp(kSkipIdHi, f.hi, 0x138, 0xf, 0xf, false);
    };
    skip_functions();
    __syncthreads();
    if (__ballot(tok0 == -2) != 0 && lane == 0) sh.cut_asked = 1;
    for (int it = 0; it <= W; ++it) {           // (a start becomes final with every iteration: the bound is never met)
      ++n_rounds;
      // ---- 2. starts ---------------------------------------------------------------------------------
      SkipFn g = {kSkipIdLo, kSkipIdHi};
      if (lane < NW) {
        const u64 v = sh.skip[lane];
        g.lo = (uint32_t)v;
        g.hi = (uint32_t)(v >> 32);
      }
      g = skip_scan16<M4>(g);
      overrun = __builtin_amdgcn_readlane((int)g.lo, NW - 1) & 0xFF;
      const uint32_t s0 = w == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)g.lo, w == 0 ? 0 : w - 1) & 0xFFu;
      const uint32_t state = ((s0 < 4 ? before.lo : before.hi) >> (8 * (s0 & 3))) & 0xFFu;
      start = state == 0 && tid < avail;
      cand = start && L >= 1 && L < M && nxt >= 0;
      start_mask = __ballot(start);
      cand_mask = __ballot(cand);
      if (lane == 0) sh.count[w] = (uint32_t)__popcll(start_mask) | ((uint32_t)__popcll(cand_mask) << 16);
      if (room <= 0) break;
      // ---- 3. proposals -------------------------------------------------------------------------------
      uint32_t* set = sh.set[it & (SETS - 1)];
      if (SETS == 1) {
        if (it > 0) __syncthreads();                             // (emptied at the end of the previous iteration)
      } else {
        if (own >= 0) sh.set[(it + 1) & 1][own] = kRoundEmpty;   // the previous iteration's
      }
      own = -1;
      if (cand) {
        own = Set::insert(set, sh.key, h, round_key(code, nxt), tid);
        if (own == -2) {                                         // later positions cannot see this edge
          atomicMin(&sh.spill_pos, tid + 1);
          sh.cut_asked = 1;
        }
      }
      __syncthreads();
      // ---- 4. matches with the entries of the round ------------------------------------------------------
      if (tid == 0) sh.changed[(it + 1) & 1] = 0;
      int L2 = L0;
      int32_t code2 = c0, nxt2 = nxt0;
      uint32_t h2 = h0;
      bool more = L0 >= 1 && L0 < M && nxt0 >= 0;
      while (__ballot(more) != 0) {
        if (more) {
          const int q = Set::find(set, sh.key, h2, round_key(code2, nxt2), tid);
          more = q >= 0;
          if (more) {
            code2 = kRoundEntry | q;
            ++L2;
            nxt2 = tk(L2);
            h2 = edge_hash(code2, nxt2);
            more = L2 < M && nxt2 >= 0;
          }
        }
      }
      // (which edges found no slot depends on timing; positions from the first of them on are cut off this window)
      const bool ch = start && (L2 != L || code2 != code) && tid < sh.spill_pos;
      L = L2;
      code = code2;
      nxt = nxt2;
      h = h2;
      if (__ballot(ch) != 0 && lane == 0) sh.changed[it & 1] = 1;
      skip_functions();
      __syncthreads();
      const bool settled = sh.changed[it & 1] == 0;
      if (own >= 0 && (SETS == 1 || settled)) set[own] = kRoundEmpty;
      if (settled) {
        break;
      }
    }

    // ---- 5. limits of the window ------------------------------------------------------------------------
    if (room <= 0) __syncthreads();             // (the counts; after an iteration with proposals they are there)
    uint32_t counts = row_scan_add(lane < NW ? sh.count[lane] : 0u);
    const uint32_t below = w == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)counts, w == 0 ? 0 : w - 1);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)counts, NW - 1);
    const u64 lanes_below = (1ull << lane) - 1;
    const int prank = (int)(below & 0xFFFFu) + __popcll(start_mask & lanes_below);   // phrases before this one
    const int rank = (int)(below >> 16) + __popcll(cand_mask & lanes_below);         // proposals before this one
    int n_start = (int)(total & 0xFFFFu), n_cand = (int)(total >> 16);
    int limit = avail;
    bool valid = start;
    u64 valid_mask = start_mask;
    u64 waves = __ballot(lane < NW && (sh.count[lane & (kMaxWaves - 1)] & 0xFFFFu) != 0);   // waves with a start
    const bool whole = !(sh.cut_asked || n_out + n_start > a.out_stride || (room > 0 && n_cand > room));   // uniform
    if (!whole) {
      const u64 bad_mask = __ballot(start && tok0 == -2);
      const u64 ovf_mask = __ballot(start && n_out + prank >= a.out_stride);
      const u64 full_mask = __ballot(room > 0 && cand && rank >= room);
      if (lane == 0) {
        if (bad_mask) atomicMin(&sh.bad_pos, w * kWave + (int)__builtin_ctzll(bad_mask));
        if (ovf_mask) atomicMin(&sh.ovf_pos, w * kWave + (int)__builtin_ctzll(ovf_mask));
        if (full_mask) atomicMin(&sh.full_pos, w * kWave + (int)__builtin_ctzll(full_mask));
      }
      __syncthreads();
      const int bad_pos = sh.bad_pos, ovf_pos = sh.ovf_pos;
      limit = min(min(avail, min(sh.full_pos, sh.spill_pos)), min(bad_pos, ovf_pos));
      if (bad_pos < W && limit == bad_pos) {
        status |= Z2Z_ST_BAD_TOKEN;             // the sequence ends just before this token
        stop = true;
      } else if (ovf_pos < W && limit == ovf_pos) {
        status |= Z2Z_ST_OVERFLOW;
        stop = true;
      }
      valid = start && tid < limit;
      valid_mask = __ballot(valid);
      const u64 ins_mask = __ballot(cand && tid < limit);
      if (lane == 0) sh.count_valid[w] = (uint32_t)__popcll(valid_mask) | ((uint32_t)__popcll(ins_mask) << 16);
      __syncthreads();
      const uint32_t mine = lane < NW ? sh.count_valid[lane] : 0u;
      waves = __ballot((mine & 0xFFFFu) != 0);
      const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)row_scan_add(mine), NW - 1);
      n_start = (int)(all & 0xFFFFu);
      n_cand = (int)(all >> 16);
    }

    // ---- 6. publish ------------------------------------------------------------------------------------
    int32_t T[M4 ? 4 : Z2Z_MAX_M];              // the tokens of the entry this position makes
    const bool ins = room > 0 && valid && cand;
    if (room > 0) {
      if (cand) sh.rank[tid] = (uint16_t)rank;
#pragma unroll
      for (int k = 0; k < (M4 ? 4 : Z2Z_MAX_M); ++k) T[k] = ins && k < M && k <= L ? tk(k) : -1;
      __syncthreads();
      if (valid && (code & kRoundEntry) != 0) code = V + C + (int)sh.rank[code & (kRoundEntry - 1)];
    }
    // a window published whole ends at pos + W + overrun; the ring takes the next tokens in place of those behind it
    auto refill = [&](int32_t next_pos) {
      const int cnt = min(W, next_pos + kRing - fill);
      const int p = fill + tid;
      if (tid < cnt) sh.tok[p & (kRing - 1)] = p < n ? classify(ahead) : -1;
      fill += cnt;
      ahead = fill + tid < n ? in[fill + tid] : 0;
    };
    const bool early = whole && avail == W;
    if (early && fill < n) refill(pos + W + overrun);
    if (valid) out[n_out + prank] = code;
    if (ins) {
      const int idx = C + rank;
      t.insert_lane(code, nxt, idx);
      int32_t* row = ent_tokens + (size_t)idx * M;
#pragma unroll
      for (int k = 0; k < (M4 ? 4 : Z2Z_MAX_M); ++k)
        if (k < M) row[k] = T[k];
      ent_len[idx] = L + 1;
    }
    if (waves != 0 && w == 63 - (int)__builtin_clzll(waves) && lane == 63 - (int)__builtin_clzll(valid_mask)) {
      sh.last_code = code;
      sh.last_len = L;
      sh.last_end = pos + tid + L;
    }
    __syncthreads();                            // insertions, last phrase, staged tokens
    if (room > 0) C += n_cand;
    n_out += n_start;
    if (waves != 0) {
      prev = sh.last_code;
      prev_len = sh.last_len;
      pos = sh.last_end;
    } else {
      stop = true;                              // a limit of 0: bad token or no room at the first start
    }
    // after a cut window, or when the last phrases of many windows have used up the slack
    while (fill < n && (!early || fill < pos + W + 32)) {
      refill(pos);
      __syncthreads();
      if (fill >= pos + W + 32) break;
    }
  }

  table_close_all<WHERE, W>(tid, t);
  if (reset) {                                  // rows of the codebook that was there before
    for (int i = C + tid; i < size0; i += W) ent_len[i] = 0;
    for (int i = C * M + tid; i < size0 * M; i += W) ent_tokens[i] = -1;
  }
  if (tid == 0) {
    st.size[b] = C;
    st.prev_code[b] = prev;
    st.prev_len[b] = prev_len;
    st.rounds[b] = n_rounds;
    a.out_n[b] = n_out;
    a.status[b] = status;
  }
}

// A short appended call touches a handful of slots: probing the table where it lives, in global memory,
// is cheaper than staging all of it in LDS and writing it back (the length is known only on the device,
// so the LDS kernels take this decision per sequence; for the tags the line lies at kTagAppendTokens).
template <int NW, int WHERE, int SETS = 2, int PER = 4>
__global__ void __launch_bounds__(NW * kWave, SETS == 1 ? 8 : 1) lzw_encode_kernel(LzwArgs a) {
  __shared__ EncShared<NW, SETS, PER> sh;
  const int b = sequence_of_block<NW>(a, reinterpret_cast<BlockOrder&>(sh));
  bool short_append = a.flags != Z2Z_RESET && call_length(a, b) <= kShortAppend;
  if (WHERE == kTag && a.flags != Z2Z_RESET)
    short_append = min(call_length(a, b), 2 * (a.st.cap - a.st.size[b])) < kTagAppendTokens;
  if (WHERE == kTag && short_append && a.st.M <= 4) {
    lzw_encode_windows<NW, SETS, PER, kMem, true>(a, b, sh);
  } else if (WHERE != kMem && short_append) {
    lzw_encode_windows<NW, SETS, PER, kMem, false>(a, b, sh);
  } else if (a.st.M <= 4) {
    lzw_encode_windows<NW, SETS, PER, WHERE, true>(a, b, sh);
  } else {
    lzw_encode_windows<NW, SETS, PER, WHERE, false>(a, b, sh);
  }
}

// ------------------------------------------------------------------------------------------------
// decode
// ------------------------------------------------------------------------------------------------
// (length, first token) of an entry packed in 32 bits: length in the top 4 bits.
__device__ __forceinline__ uint32_t pack_ef(int len, int32_t first) { return ((uint32_t)len << 28) | (uint32_t)first; }

// One code at a time (the textbook loop, wave-uniform): used for short appended calls, where a
// round of the kernel below would be mostly empty.
// (a read past the vector L1 of data another wave of the workgroup wrote earlier in the launch)
__device__ __forceinline__ int32_t load_fresh_i32(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool LDS>
__device__ __forceinline__ void lzw_decode_serial_body(const LzwArgs& a, int b, int lane) {
  const LzwState& st = a.st;
  const int V = st.V, M = st.M, cap = st.cap;
  const bool reset = a.flags == Z2Z_RESET;
  const bool ef_lds = LDS && a.lds_ef;
  uint32_t* ef = reinterpret_cast<uint32_t*>(lds_slots + st.nslots);   // [cap], valid when ef_lds
  int32_t* ent_tokens = st.ent_tokens + (size_t)b * cap * M;
  int32_t* ent_len = st.ent_len + (size_t)b * cap;

  int C = reset ? 0 : __builtin_amdgcn_readfirstlane(st.size[b]);
  int prev = reset ? -1 : __builtin_amdgcn_readfirstlane(st.prev_code[b]);
  int prev_len = reset ? 0 : __builtin_amdgcn_readfirstlane(st.prev_len[b]);
  int prev_first = prev < 0 ? 0 : (prev < V ? prev : __builtin_amdgcn_readfirstlane(ent_tokens[(size_t)(prev - V) * M]));

  Table<LDS> t;
  if (ef_lds && !reset) {
    for (int i = lane; i < C; i += kWave) ef[i] = pack_ef(ent_len[i], ent_tokens[(size_t)i * M]);
  }
  table_open<LDS>(a, b, lane, reset, &t);

  const int n = a.in_len ? min(max(__builtin_amdgcn_readfirstlane(a.in_len[b]), 0), a.stride) : a.stride;
  const int32_t* in = a.in + (size_t)b * (a.in_step > 0 ? a.in_step : a.stride);
  int32_t* out = a.out ? a.out + (size_t)b * a.out_stride : nullptr;

  int status = 0;
  int n_out = 0;
  bool stop = false;

  for (int base = 0; base < n && !stop; base += kWave) {
    const int cnt = min(kWave, n - base);
    const int32_t code_reg = lane < cnt ? in[base + lane] : 0;
    // ---- serial part: (length, first token) of each code and the codebook update, all in LDS and
    //      scalar registers.  Lane j keeps what the parallel part needs for code j: where its tokens
    //      go, and the entry (if any) that code j caused.
    int my_off = 0, my_len = 0;
    int new_idx = -1, new_parent = 0, new_tok = 0, new_plen = 0;
    int done = 0;                     // codes of this chunk accepted
    for (int j = 0; j < cnt; ++j) {
      const int32_t k = __builtin_amdgcn_readlane(code_reg, j);
      int cur_len = 0;
      int32_t first = 0;
      int free_pos = -1;
      bool fresh = false;             // the code names the entry made in this very step
      if (k >= 0 && k < V) {
        cur_len = 1;
        first = k;
      } else if (k >= V && k - V < C) {
        uint32_t e;
        if (ef_lds)
          e = ef[k - V];
        else
          e = pack_ef(ent_len[k - V], ent_tokens[(size_t)(k - V) * M]);
        e = __builtin_amdgcn_readfirstlane(e);
        cur_len = (int)(e >> 28);
        first = (int32_t)(e & 0x0FFFFFFFu);
      } else if (k >= V && k - V == C && prev >= 0 && prev_len < M && C < cap) {
        // previous phrase + its own first token, which must not exist yet
        const int idx = t.find(prev, prev_first, &free_pos);
        if (idx >= 0 || free_pos < 0) {
          status |= Z2Z_ST_BAD_CODE;
          stop = true;
          break;
        }
        cur_len = prev_len + 1;
        first = prev_first;
        fresh = true;
      } else {
        status |= Z2Z_ST_BAD_CODE;
        stop = true;
        break;
      }
      if (out != nullptr && n_out + cur_len > a.out_stride) {
        status |= Z2Z_ST_OVERFLOW;
        stop = true;
        break;
      }
      if (prev >= 0 && prev_len < M && C < cap) {
        int idx = -1;
        if (!fresh) idx = t.find(prev, first, &free_pos);
        if (idx < 0 && free_pos >= 0) {
          if (lane == 0) {
            t.store((uint32_t)free_pos, edge_bits(prev, first) | (u64)(uint32_t)C);
            if (ef_lds) {
              ef[C] = pack_ef(prev_len + 1, prev_first);
            } else {
              // no LDS copy: a later code of this chunk may already name this entry, and its length
              // and first token are then read from memory before the rows are completed below
              ent_len[C] = prev_len + 1;
              ent_tokens[(size_t)C * M] = prev_first;
            }
          }
          if (lane == j) {
            new_idx = C;
            new_parent = prev;
            new_tok = first;
            new_plen = prev_len;
          }
          ++C;
        }
      }
      if (lane == j) {
        my_off = n_out;
        my_len = cur_len;
      }
      n_out += cur_len;
      prev = k;
      prev_len = cur_len;
      prev_first = first;
      ++done;
    }
    // ---- parallel part 1: write the flattened rows of the entries made in this chunk, shortest
    //      parents first (a parent made in this chunk is shorter than its child, so it is complete
    //      by the time the child copies it)
    for (int L = 1; L < M; ++L) {
      if (new_idx >= 0 && new_plen == L) {
        int32_t* row = ent_tokens + (size_t)new_idx * M;
        if (new_parent < V) {
          row[0] = new_parent;
        } else {
          const int32_t* prow = ent_tokens + (size_t)(new_parent - V) * M;
          for (int i = 0; i < L; ++i) row[i] = prow[i];
        }
        row[L] = new_tok;
        for (int i = L + 1; i < M; ++i) row[i] = -1;
        ent_len[new_idx] = L + 1;
      }
      wave_sync();                    // one wave: orders this level's stores before the next level's loads
    }
    // ---- parallel part 2: lane j writes the tokens of code j
    if (out != nullptr && lane < done) {
      const int32_t k = code_reg;
      if (k < V) {
        out[my_off] = k;
      } else {
        const int32_t* row = ent_tokens + (size_t)(k - V) * M;
        for (int i = 0; i < my_len; ++i) out[my_off + i] = row[i];
      }
    }
  }

  table_close<LDS>(a, lane, t);
  if (lane == 0) {
    st.size[b] = C;
    st.prev_code[b] = prev;
    st.prev_len[b] = prev_len;
    st.rounds[b] = n;                 // one code per step
    a.out_n[b] = n_out;
    a.status[b] = status;
  }
}

template <bool LDS>
__global__ void __launch_bounds__(kWave) lzw_decode_serial_kernel(LzwArgs a) {
  lzw_decode_serial_body<LDS>(a, blockIdx.x, threadIdx.x);
}

// One generation step's codebook side in one launch (section 2.3, steps 9-10; "Hyper-Embedding Cache"): wave 0
// of the workgroup applies the sequence's new code to its codebook (the one-code-at-a-time update above, table
// in global memory), then all waves pool the newest entry's constituent embeddings into its row of the cache --
// what an appended z2z_lzw_decode of one code followed by z2z_hyper_embed of the last entry do in two launches.
// The newest entry is pooled whether or not this step made it (the row comes out bit-identical).
constexpr int kStepWaves = 8;
template <bool BF16>
__global__ void __launch_bounds__(kStepWaves * kWave) lzw_step_update_kernel(LzwArgs a, z2z_embed::EmbedArgs ea) {
  const int b = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (w == 0) lzw_decode_serial_body<false>(a, b, lane);
  sync_after_global_stores();          // the entry's row and the size are in memory before the other waves read them
  const int C = min(__builtin_amdgcn_readfirstlane(load_fresh_i32(a.st.size + b)), a.st.cap);
  if (C <= 0) return;
  const size_t row = (size_t)b * a.st.cap + (C - 1);
  const int L = min(max(__builtin_amdgcn_readfirstlane(load_fresh_i32(a.st.ent_len + row)), 1), a.st.M);
  int32_t toks[Z2Z_MAX_M];
#pragma unroll
  for (int j = 0; j < Z2Z_MAX_M; ++j) toks[j] = j < L ? load_fresh_i32(a.st.ent_tokens + row * a.st.M + j) : 0;
  if (w < ea.split) z2z_embed::embed_row<BF16, false>(ea, toks, L, row, lane, w);
}

// ------------------------------------------------------------------------------------------------
// decode
//
// Rounds like the encoder's: thread g of a window holds code cpos + g - 1, thread 0 the code before the window.
// Code g makes the entry (code g-1, first token of code g) if code g-1 is shorter than M, the codebook has room and
// the edge is absent; (length, first token) of a code come from the codebook as it stood when the round began, or,
// for an entry of this round, from the code before its maker.  Again a recurrence over lower positions, solved by
// iteration:
//   1. codes that are base tokens or old entries have their (length, first token); edges between those are looked
//      up in the table at once.  Codes that name entries of this round start from a guess of their length.
//   2. who makes an entry follows from the lengths; the makers' ranks are a prefix count, maker[rank] = position.
//   3. a code that names entry `rank` of this round takes (length + 1, first token) from the position before its
//      maker, or is invalid if that entry is made after it.  When nothing changes the values are exact.
//   4. the makers' edges go into the table.  What 1-3 assume about edges that involve this round's entries -- that they are
//      new -- shows there: if an edge is in the table, or proposed twice in the window, the window's insertions are taken
//      back, the encoder's round set and late look-ups say where the first such position is, and the window is cut there;
//      the next round meets it as its first code, where everything is known.  Streams of a greedy parse have none.  Behind
//      such a window the next looks before it inserts, until one is whole: codes that no parse made would pay for both in
//      every window (8 sequences of 4096 tokens out of 300, cap 2048: 51 us, so 45; out of 40 264, 221; a
//      parse's codes, one in 80 of them replaced, cap 4096: 72, 66).
//   5. publish: token offsets are prefix sums of the lengths; a thread writes its code's tokens to the output and,
//      with the next code's first token behind them, to the row of the entry the next code makes.
// Three to five iterations are usual: who is as long as M, and so makes nothing, moves the ranks behind it.
//
// What bounds it: those iterations, two barriers each.  A thread owns what its code does as the FIRST half of an entry, so that
// an iteration needs no exchange of lengths with the neighbour; the insertion into the table is itself the check of 4.
// Before (three barriers, a set for the edges of every window), us: 8 sequences of 4096 tokens, M = 3, cap 4096 38 -> 32; 4 of 32768,
// M = 4, cap 8192 97 -> 84; 16 of 16384, M = 5, cap 16384 100 -> 75; 2048 of up to 4096, M = 3, cap 2048 125 -> 113.
// ------------------------------------------------------------------------------------------------
// Codes that the decoder leaves to the kernel behind it, which takes a launch (5 us) where a window of 1024 takes 2.6.
constexpr int kTailMin = 3072;

template <int NW>
struct DecShared {
  static constexpr int W = NW * kWave;
  static constexpr int kSet = 4 * W;
  uint32_t set[kSet];
  u64 key[W];
  int32_t ring[2 * W];                       // codes: code p at p & (2 W - 1)
  int32_t code[W];                           // of the window
  uint32_t info[W];                          // pack_ef(length, first token)
  uint32_t count[kMaxWaves];                 // entries made by each wave; above them whether its makers changed and need others
  uint32_t tokens[kMaxWaves];                // of each wave's codes
  int32_t clash;                             // an edge of the window was in the table or proposed twice
  int32_t bad_pos, ovf_pos, cut;             // where the window ends early
  int32_t last_code, last_len, last_tokens, last_made;
  uint16_t parent[W];                        // position of the code before the one that makes entry `rank` of the round
};
static_assert(sizeof(DecShared<kMaxWaves>) <= sizeof(EncShared<kMaxWaves, 2>), "one LDS budget for both directions");

template <int NW, int WHERE, bool M4>
__device__ __forceinline__ void lzw_decode_windows(const LzwArgs& a, int b, DecShared<NW>& sh) {
  constexpr int W = NW * kWave;
  constexpr int kSet = DecShared<NW>::kSet, kRing = 2 * W;
  constexpr int kTok = M4 ? 4 : Z2Z_MAX_M;
  constexpr int32_t kFirst = 0x0FFFFFFF;
  typedef RoundSet<kSet> Set;
  const LzwState& st = a.st;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int V = st.V, M = st.M, cap = st.cap;
  const bool reset = a.flags == Z2Z_RESET;
  const bool ef_lds = WHERE == kLds && a.lds_ef;
  uint32_t* ef = reinterpret_cast<uint32_t*>(lds_slots + st.nslots);   // [cap], valid when ef_lds

  const int size0 = __builtin_amdgcn_readfirstlane(st.size[b]);
  int C = reset ? 0 : size0;
  int prev = reset ? -1 : __builtin_amdgcn_readfirstlane(st.prev_code[b]);
  int prev_len = reset ? 0 : __builtin_amdgcn_readfirstlane(st.prev_len[b]);
  const int n = call_length(a, b);
  const int32_t* in = a.in + (size_t)b * a.stride;
  int32_t* out = a.out ? a.out + (size_t)b * a.out_stride : nullptr;
  int32_t* ent_tokens = st.ent_tokens + (size_t)b * cap * M;
  int32_t* ent_len = st.ent_len + (size_t)b * cap;

  Table<WHERE> t;
  table_open_all<WHERE, W>(a, b, tid, reset, &t, C < cap);
  if (ef_lds && !reset) {
    for (int i = tid; i < C; i += W) ef[i] = pack_ef(ent_len[i], ent_tokens[(size_t)i * M]);
  }
  for (int i = tid; i < kSet; i += W) sh.set[i] = kRoundEmpty;
  int fill = kRing;
  for (int i = tid; i < kRing; i += W) sh.ring[i] = i < n ? in[i] : -1;
  int32_t ahead = fill + tid < n ? in[fill + tid] : -1;
  sync_after_global_stores();        // (a table cleared in global memory is read past the L1)

  const u64 lanes_below = (1ull << lane) - 1;
  int status = 0;
  int n_out = 0;
  bool stop = false;
  int cpos = 0;                       // codes consumed
  int n_rounds = 0;
  bool suspect = false;               // the window before was cut at an edge that is no entry's first: step 4 looks before it inserts
  while (cpos < n && !stop) {
    // ---- 1. the codes of the window ---------------------------------------------------------------------
    const int ci = cpos + tid - 1;
    const bool present = tid == 0 ? prev >= 0 : ci < n;
    const int32_t k = tid == 0 ? prev : (ci < n ? sh.ring[ci & (kRing - 1)] : -1);
    const bool old_entry = present && k >= V && k - V < C;
    const bool new_entry = present && tid > 0 && k >= V + C;
    int len = 0;
    int32_t first = 0;
    int32_t T[kTok];                  // the tokens of a base token or an old entry
#pragma unroll
    for (int j = 0; j < kTok; ++j) T[j] = -1;
    if (present && k >= 0 && k < V) {
      len = 1;
      first = T[0] = k;
    } else if (old_entry) {
      const int32_t* row = ent_tokens + (size_t)(k - V) * M;
#pragma unroll
      for (int j = 0; j < kTok; ++j)
        if (j < M) T[j] = row[j];
      if (ef_lds) {
        const uint32_t e = ef[k - V];
        len = (int)(e >> 28);
        first = (int32_t)(e & kFirst);
      } else {
#pragma unroll
        for (int j = 0; j < kTok; ++j) len += T[j] >= 0 ? 1 : 0;
        first = T[0];
      }
    } else if (new_entry) {
      len = min(2, M);                // a guess
    }
    sh.code[tid] = k;
    sh.info[tid] = pack_ef(len, first);
    if (tid == 0) sh.bad_pos = sh.ovf_pos = sh.cut = W;
    __syncthreads();
    // this position's part in the entry that the code behind it makes: this code and the first token of that one
    const int next = tid + 1;
    const int32_t nk = next < W ? sh.code[next] : -1;
    const bool next_present = next < W && ci + 1 < n;
    const bool next_new = next_present && nk >= V + C;
    const int room = cap - C;
    const bool may_add = present && k >= 0 && next_present && room > 0;
    bool taken = false;               // the edge is an entry already
    // (the first code of the window may name the entry it makes itself: its first token is then the previous code's)
    if (may_add && !new_entry && (!next_new || next == 1) && len < M)
      taken = t.find_lane(k, next_new ? first : (int32_t)(sh.info[next] & kFirst)) >= 0;

    // ---- 2., 3. lengths and makers -----------------------------------------------------------------------
    bool makes = false;
    int rank = 0, n_made = 0;
    const bool has_new = __ballot(new_entry) != 0;
    bool stepped = true;              // a length of this wave changed in the iteration before
    for (int it = 0; it <= W; ++it) {           // (a position becomes final with every iteration: the bound is never met)
      ++n_rounds;
      makes = may_add && !taken && len < M;
      const u64 makes_mask = __ballot(makes);
      if (lane == kWave - 1)
        sh.count[w] = (uint32_t)__popcll(makes_mask) | (stepped ? 0x80000000u : 0u) | (has_new ? 0x40000000u : 0u);
      __syncthreads();
      const uint32_t word = lane < NW ? sh.count[lane] : 0u;
      if (__ballot((word & 0x80000000u) != 0) == 0) break;        // (rank and n_made stand)
      const uint32_t counts = row_scan_add(word & 0xFFFFu);
      rank = (w == 0 ? 0 : __builtin_amdgcn_readlane((int)counts, w == 0 ? 0 : w - 1)) + __popcll(makes_mask & lanes_below);
      n_made = min(__builtin_amdgcn_readlane((int)counts, NW - 1), room);
      if (__ballot((word & 0x40000000u) != 0) == 0) break;        // no code of the window depends on an entry of it
      if (makes && rank < room) sh.parent[rank] = (uint16_t)tid;
      __syncthreads();
      bool ch = false;
      if (new_entry) {
        const int e = k - V - C;
        const int p = e < n_made ? (int)sh.parent[e] : W;
        const uint32_t base = p < tid ? sh.info[p] : 0u;            // (of this iteration or the one before, as it comes)
        const int len2 = (base >> 28) != 0 ? min((int)(base >> 28) + 1, M) : 0;
        const int32_t first2 = (int32_t)(base & kFirst);
        ch = len2 != len || first2 != first;
        len = len2;
        first = first2;
        sh.info[tid] = pack_ef(len, first);
      }
      stepped = __ballot(ch) != 0;
    }

    // ---- 4. limits of the window --------------------------------------------------------------------------
    const bool makes_it = makes && rank < room;      // with the code at `next`
    const int mylen = tid > 0 ? len : 0;
    int incl = 0;                               // tokens of the codes up to this one
#pragma unroll
    for (int bit = 0; bit < 4; ++bit) {
      const u64 m = __ballot((mylen >> bit) & 1);
      incl += (__popcll(m & lanes_below) + ((mylen >> bit) & 1)) << bit;
    }
    if (lane == kWave - 1) sh.tokens[w] = (uint32_t)incl;
    const u64 bad_mask = __ballot(tid > 0 && present && len == 0);
    if (bad_mask != 0 && lane == 0) atomicMin(&sh.bad_pos, w * kWave + (int)__builtin_ctzll(bad_mask));
    if (tid == 0) sh.clash = 0;
    __syncthreads();
    const uint32_t tokens = row_scan_add(lane < NW ? sh.tokens[lane] : 0u);
    incl += w == 0 ? 0 : __builtin_amdgcn_readlane((int)tokens, w == 0 ? 0 : w - 1);
    const int n_tokens = __builtin_amdgcn_readlane((int)tokens, NW - 1);
    const int bad_pos = sh.bad_pos;
    int limit = min(min(W, n - cpos + 1), bad_pos);                 // codes 1 .. limit-1 of the window are taken
    int ovf_pos = W;
    if (out != nullptr && n_out + n_tokens > a.out_stride) {        // uniform
      const u64 ovf_mask = __ballot(tid > 0 && present && len > 0 && n_out + incl > a.out_stride);
      if (ovf_mask && lane == 0) atomicMin(&sh.ovf_pos, w * kWave + (int)__builtin_ctzll(ovf_mask));
      __syncthreads();
      ovf_pos = sh.ovf_pos;
      limit = min(limit, ovf_pos);
    }
    if (n_made > 0) {
      const int32_t tok = makes_it ? (int32_t)(sh.info[next] & kFirst) : 0;
      if (!suspect) {
        int slot = -2;
        const bool inserts = makes_it && next < limit;
        if (inserts) slot = t.insert_new(k, tok, C + rank);
        if (__ballot(inserts && slot < 0) != 0 && lane == 0) sh.clash = 1;
        __syncthreads();
        suspect = sh.clash != 0;
        if (suspect) {                          // (codes that no greedy parse made)
          if (slot >= 0) t.remove(slot);
          sync_after_global_stores();
        }
      }
      if (suspect) {
        const uint32_t h = edge_hash(k, tok);
        int own = -1;
        bool clash = false;
        if (makes_it) {
          own = Set::insert(sh.set, sh.key, h, round_key(k, tok), next);
          if (own == -2) atomicMin(&sh.cut, next + 1);            // later positions cannot see this edge
          if (next_new && next > 1 && !new_entry) clash = t.find_lane(k, tok, h) >= 0;
        }
        __syncthreads();
        if (makes_it && !clash) clash = Set::find(sh.set, sh.key, h, round_key(k, tok), next) >= 0;
        if (clash) atomicMin(&sh.cut, next);
        __syncthreads();
        if (own >= 0) sh.set[own] = kRoundEmpty;
        limit = min(limit, sh.cut);
        suspect = sh.cut < W;
        if (makes_it && next < limit) t.insert_lane(k, tok, C + rank);
      }
    }
    if (ovf_pos < W && limit == ovf_pos) {
      status |= Z2Z_ST_OVERFLOW;
      stop = true;
    } else if (bad_pos < W && limit == bad_pos) {
      status |= Z2Z_ST_BAD_CODE;
      stop = true;
    }

    // ---- 5. publish ---------------------------------------------------------------------------------------
    const bool next_makes = makes_it && next < limit;
    const bool writes = tid > 0 && tid < limit && out != nullptr;
    if (writes || next_makes) {
      int l = len;
      int32_t kk = k;
      while (kk >= V + C) {                     // entries of this round: last token first (at most M - 1 steps)
        const int p = sh.parent[kk - V - C];
        const int32_t tok = (int32_t)(sh.info[p + 1] & kFirst);
        --l;
#pragma unroll
        for (int j = 0; j < kTok; ++j) T[j] = j == l ? tok : T[j];
        kk = sh.code[p];
      }
      if (kk != k) {
        if (kk < V) {
          T[0] = kk;
        } else {
          const int32_t* src = ent_tokens + (size_t)(kk - V) * M;
#pragma unroll
          for (int j = 0; j < kTok; ++j)
            if (j < l) T[j] = src[j];
        }
      }
      if (writes) {
        int32_t* dst = out + n_out + incl - len;
#pragma unroll
        for (int j = 0; j < kTok; ++j)
          if (j < len) dst[j] = T[j];
      }
      if (next_makes) {
        const int32_t tok = (int32_t)(sh.info[next] & kFirst);
#pragma unroll
        for (int j = 0; j < kTok; ++j) T[j] = j < len ? T[j] : j == len ? tok : -1;
        int32_t* row = ent_tokens + (size_t)(C + rank) * M;
#pragma unroll
        for (int j = 0; j < kTok; ++j)
          if (j < M) row[j] = T[j];
        ent_len[C + rank] = len + 1;
        if (ef_lds) ef[C + rank] = pack_ef(len + 1, first);
      }
    }
    if (limit >= 2 && tid == limit - 1) {
      sh.last_code = k;
      sh.last_len = len;
      sh.last_tokens = incl;
      sh.last_made = min(rank, room);
    }
    if (fill < n) {                             // the ring takes the next codes in place of those behind the window
      const int cnt = min(W, cpos + limit - 1 + kRing - fill);
      const int p = fill + tid;
      if (tid < cnt) sh.ring[p & (kRing - 1)] = p < n ? ahead : -1;
      fill += cnt;
      ahead = fill + tid < n ? in[fill + tid] : -1;
    }
    __syncthreads();                            // rows, insertions, the ring
    if (limit >= 2) {
      prev = sh.last_code;
      prev_len = sh.last_len;
      n_out += sh.last_tokens;
      C += sh.last_made;
      cpos += limit - 1;
      if (C >= cap && n - cpos >= a.tail_min) break;
    } else {
      stop = true;
    }
  }

  table_close_all<WHERE, W>(tid, t);
  if (reset) {                                  // rows of the codebook that was there before
    for (int i = C + tid; i < size0; i += W) ent_len[i] = 0;
    for (int i = C * M + tid; i < size0 * M; i += W) ent_tokens[i] = -1;
  }
  if (tid == 0) {
    st.size[b] = C;
    st.prev_code[b] = prev;
    st.prev_len[b] = prev_len;
    st.rounds[b] = n_rounds;
    a.out_n[b] = n_out;
    a.status[b] = status;
    st.tail[3 * b] = stop ? n : cpos;
    st.tail[3 * b + 1] = n_out;
    st.tail[3 * b + 2] = n;
  }
}

template <int NW, int WHERE>
__global__ void __launch_bounds__(NW * kWave) lzw_decode_kernel(LzwArgs a) {
  __shared__ DecShared<NW> sh;
  const int b = sequence_of_block<NW>(a, reinterpret_cast<BlockOrder&>(sh));
  bool short_append = a.flags != Z2Z_RESET && call_length(a, b) <= kShortAppend;
  if (WHERE == kTag && a.flags != Z2Z_RESET) {
    const int room = a.st.cap - a.st.size[b];                 // (full: nothing is looked up, the tags are not made)
    short_append = room > 0 && min(call_length(a, b), room) < kTagAppendCodes;
  }
  if (WHERE == kTag && short_append && a.st.M <= 4) {
    lzw_decode_windows<NW, kMem, true>(a, b, sh);
  } else if (WHERE != kMem && short_append) {
    lzw_decode_windows<NW, kMem, false>(a, b, sh);
  } else if (a.st.M <= 4) {
    lzw_decode_windows<NW, WHERE, true>(a, b, sh);
  } else {
    lzw_decode_windows<NW, WHERE, false>(a, b, sh);
  }
}

// The codes behind a full codebook: nothing is made any more, so lengths are a table look-up, offsets a prefix sum, and
// all CUs can take part.  grid = (parts, B); a part of a sequence adds up the lengths of the codes before its own by
// itself (a chain of parts, each waiting for the one before, would be as long as the window kernel's).
//
// What bounds it: the launch, two dependent trips to L2 per 1024 codes before the part.  4 sequences of 22300 codes, of which
// 13700 lie behind the 8192 entries of a full codebook: 35 us in the window kernel, 10 here; 27400 behind 1024: 84 -> 33 in all.
__global__ void __launch_bounds__(1024) lzw_decode_tail_kernel(LzwArgs a) {
  constexpr int W = 1024, NW = W / kWave;
  struct Shared {
    uint32_t count[NW];
    int32_t bad;                               // a code before this part that names nothing
    int32_t end;                               // first element of a turn that is not taken
  };
  __shared__ Shared sh;
  const LzwState& st = a.st;
  const int b = blockIdx.y;
  // (the length as well: where the caller has counts and lengths in one buffer, in_len holds token counts by now)
  const int from = __builtin_amdgcn_readfirstlane(st.tail[3 * b]), n = __builtin_amdgcn_readfirstlane(st.tail[3 * b + 2]);
  const int share = (n - from + (int)gridDim.x - 1) / (int)gridDim.x;
  const int span = (share + W - 1) / W * W;
  const int lo = from + (int)blockIdx.x * span;
  if (from >= n || lo >= n) return;
  const int hi = min(n, lo + span);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int V = st.V, M = st.M, cap = st.cap;
  const int C = min(max(__builtin_amdgcn_readfirstlane(st.size[b]), 0), cap);
  const int32_t* in = a.in + (size_t)b * a.stride;
  int32_t* out = a.out ? a.out + (size_t)b * a.out_stride : nullptr;
  const int32_t* ent_tokens = st.ent_tokens + (size_t)b * cap * M;
  const int32_t* ent_len = st.ent_len + (size_t)b * cap;
  auto length = [&](int32_t k) -> int {        // 0: names nothing
    if (k < 0) return 0;
    if (k < V) return 1;
    return k - V < C ? ent_len[k - V] : 0;
  };

  if (tid == 0) sh.bad = 0;
  __syncthreads();
  int sum = 0;
  bool bad = false;
#pragma unroll 4
  for (int i = from + tid; i < lo; i += W) {
    const int len = length(in[i]);
    bad |= len == 0;
    sum += len;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) sh.count[w] = (uint32_t)sum;
  if (__ballot(bad) != 0 && lane == 0) sh.bad = 1;
  __syncthreads();
  int base = st.tail[3 * b + 1];               // tokens of the codes before
  for (int j = 0; j < NW; ++j) base += (int)sh.count[j];
  // the sequence ended in an earlier part
  if (sh.bad || (out != nullptr && base > a.out_stride)) return;

  const u64 lanes_below = (1ull << lane) - 1;
  for (int pos = lo; pos < hi; pos += W) {
    const int i = pos + tid;
    const bool present = i < hi;
    const int32_t k = present ? in[i] : -1;
    const int len = present ? length(k) : 0;
    int incl = 0;                              // tokens of the codes of this turn up to this one
#pragma unroll
    for (int bit = 0; bit < 4; ++bit) {
      const u64 m = __ballot((len >> bit) & 1);
      incl += (__popcll(m & lanes_below) + ((len >> bit) & 1)) << bit;
    }
    __syncthreads();                           // (the previous turn's counts have been read)
    if (tid == 0) sh.end = W;
    if (lane == kWave - 1) sh.count[w] = (uint32_t)incl;
    __syncthreads();
    const uint32_t counts = row_scan_add(lane < NW ? sh.count[lane] : 0u);
    incl += w == 0 ? 0 : __builtin_amdgcn_readlane((int)counts, w == 0 ? 0 : w - 1);
    const int total = __builtin_amdgcn_readlane((int)counts, NW - 1);
    const u64 ends = __ballot(present && (len == 0 || (out != nullptr && base + incl > a.out_stride)));
    if (ends != 0 && lane == 0) atomicMin(&sh.end, w * kWave + (int)__builtin_ctzll(ends));
    __syncthreads();
    const int end = sh.end;
    if (present && tid < end && out != nullptr) {
      int32_t* dst = out + base + incl - len;
      if (k < V) {
        dst[0] = k;
      } else {
        const int32_t* row = ent_tokens + (size_t)(k - V) * M;
        int32_t T[Z2Z_MAX_M];
#pragma unroll
        for (int j = 0; j < Z2Z_MAX_M; ++j) T[j] = j < M ? row[j] : -1;
#pragma unroll
        for (int j = 0; j < Z2Z_MAX_M; ++j)
          if (j < len) dst[j] = T[j];
      }
    }
    if (end < W) {                             // uniform
      if (tid == end) {
        a.status[b] = len == 0 ? Z2Z_ST_BAD_CODE : Z2Z_ST_OVERFLOW;
        a.out_n[b] = base + incl - len;
        if (i > from) {
          st.prev_code[b] = in[i - 1];
          st.prev_len[b] = length(in[i - 1]);
        }
      }
      return;
    }
    if (i == n - 1) {
      a.out_n[b] = base + incl;
      st.prev_code[b] = k;
      st.prev_len[b] = len;
    }
    base += total;
  }
}

// Empty every codebook.  grid = B, block = 256.
__global__ void lzw_reset_kernel(LzwState st) {
  const int b = blockIdx.x;
  for (int i = threadIdx.x; i < st.nslots; i += blockDim.x) st.slots[(size_t)b * st.nslots + i] = kEmpty;
  for (int i = threadIdx.x; i < st.cap; i += blockDim.x) st.ent_len[(size_t)b * st.cap + i] = 0;
  for (size_t i = threadIdx.x; i < (size_t)st.cap * st.M; i += blockDim.x)
    st.ent_tokens[(size_t)b * st.cap * st.M + i] = -1;
  if (threadIdx.x == 0) {
    st.size[b] = 0;
    st.prev_code[b] = -1;
    st.prev_len[b] = 0;
  }
}

// Clear the entry rows of a sequence that a RESET encode/decode is about to refill, so that rows at
// and beyond the new size read as unused.  grid = B, block = 256.
__global__ void lzw_clear_entries_kernel(LzwState st) {
  const int b = blockIdx.x;
  const int C = st.size[b];
  for (int i = threadIdx.x; i < C; i += blockDim.x) st.ent_len[(size_t)b * st.cap + i] = 0;
  for (size_t i = threadIdx.x; i < (size_t)C * st.M; i += blockDim.x)
    st.ent_tokens[(size_t)b * st.cap * st.M + i] = -1;
}

// How a call is launched: table in LDS or in memory, waves per sequence, dynamic LDS.
//   - A short appended call (a decode step) touches a handful of slots: one wave, the table where it is.
//   - While every sequence has a CU to itself, the widest window is the fastest (4096 tokens, 8 sequences: 44 us
//     with 16 waves, 54 with 8); up to 512 elements a call is a single window of 8 waves.
//   - With more sequences than CUs, workgroups of a CU hide each other's latencies: 8 waves each where two fit its LDS
//     (2048 sequences of 4096 tokens, cap 2048: 260 us; 16 waves 576), else for the decoder 4 (without its (length, first
//     token) copy), else one of 8.  Up to four fit (z2z_lzw_prepare); the encoder's iterations then share one RoundSet
//     where two would keep one workgroup from fitting (2048 documents of 1024 to 4096 tokens, cap 2048: two workgroups 200
//     us, three 162); where they would not, two sets are faster, by a barrier an iteration (500 sequences: 73, one set 82).
//     With tables in memory the fourth workgroup's 64 registers are not enough: two sets -> one, cap 12000, 2048 of 1024
//     tokens 243 -> 259, of 4096 595 -> 607 (1024 of 4096 319 -> 303).
//   - While every sequence has a CU, the encoder's sets have eight slots per position where the table leaves the LDS for it: a
//     wave inserts with as many compare-and-swaps as its unluckiest lane needs (8 sequences of 4096 tokens, four slots -> eight,
//     cap 2048: 46 -> 42 us; cap 4096: 51 -> 47; 8 of 8192, cap 2900: 67 -> 57; 200 of 2000: 38 -> 34; 1 of 512: 12.1 -> 11.5).
struct ParsePlan {
  bool lds, tags;
  int nw;
  int sets;                // encoder: RoundSets that the iterations of a window use in turn ...
  int per;                 // ... and their slots per position
  size_t smem;
};
// Lengths that a call overwrites (one buffer for lengths and counts): every workgroup reads its own before it writes, but in
// order of length the late ones would look at the counts of those that have ended.
bool writes_lengths(const LzwArgs& a, size_t B) {
  const uintptr_t lo = reinterpret_cast<uintptr_t>(a.in_len), hi = lo + B * sizeof(int32_t);
  auto meets = [&](const int32_t* p, size_t n) {
    const uintptr_t at = reinterpret_cast<uintptr_t>(p);
    return p != nullptr && at < hi && lo < at + n * sizeof(int32_t);
  };
  return meets(a.out_n, B) || meets(a.status, B) || meets(a.out, B * (size_t)a.out_stride);
}
ParsePlan plan(const z2z_ctx* c, int32_t stride, int32_t flags, bool decode, LzwArgs* a) {
  ParsePlan p;
  const bool tiny_append = !(flags & Z2Z_RESET) && stride <= kShortAppend;
  p.lds = c->st.slots_fit_lds && !tiny_append && c->opt_lzw_kernel != 2;
  p.nw = tiny_append || c->opt_lzw_kernel == 4 ? 1 : stride <= 512 ? 8 : 16;
  p.smem = p.lds ? (size_t)c->st.nslots * sizeof(u64) : 0;
  p.tags = c->st.tags_fit_lds && p.nw == 16 && c->opt_lzw_kernel != 2 &&
           ((flags & Z2Z_RESET) || stride >= (decode ? kTagAppendCodes : kTagAppendTokens));
  if (p.tags) p.smem = (size_t)c->st.nslots * sizeof(uint16_t);
  const size_t all = (size_t)c->lds_limit, fixed8 = sizeof(DecShared<8>), fixed4 = sizeof(DecShared<4>);
  size_t ef = decode && p.lds ? (size_t)c->st.cap * sizeof(uint32_t) : 0;
  if (p.smem + ef + kParseStaticLds > all) ef = 0;
  if (c->cfg.B > c->num_cu && p.nw > 1) {
    p.nw = 8;
    if (decode && p.lds && 2 * (p.smem + ef + fixed8) > all && 2 * (p.smem + fixed4) <= all) {
      p.nw = 4;
      if (2 * (p.smem + ef + fixed4) > all) ef = 0;
    }
  }
  a->lds_ef = ef != 0;
  p.sets = 2;
  p.per = 4;
  if (!decode && c->cfg.B <= c->num_cu && p.lds && p.nw >= 8 && p.smem + (p.nw == 16 ? kWideSets16 : kWideSets8) <= all) p.per = 8;
  if (!decode && c->cfg.B > c->num_cu && p.nw > 1 && p.lds) {
    // workgroups that a CU holds, by its LDS and by 32 (two sets: 28) waves of registers, no more than there are
    auto held = [&](size_t fixed, int waves) {
      return std::min({all / (p.smem + fixed), (size_t)(waves / p.nw), (size_t)((c->cfg.B + c->num_cu - 1) / c->num_cu)});
    };
    if (held(sizeof(EncShared<8, 1>), 32) > held(sizeof(EncShared<8, 2>), 28)) p.sets = 1;
  }
  const int most = std::min(16 * c->num_cu, (decode ? 4 : 8) * c->num_cu + stride / 2);
  a->by_length = a->in_len != nullptr && c->cfg.B > 2 * c->num_cu && c->cfg.B <= most && p.nw >= 4 && stride >= (decode ? 2048 : 640) &&
                 !writes_lengths(*a, (size_t)c->cfg.B);
  p.smem += ef;
  return p;
}
// A launch asks for no more dynamic LDS than z2z_lzw_prepare has declared for its kernel.
bool fits(const z2z_ctx* c, const ParsePlan& p) {
  const int own = p.per == 8 ? (p.nw == 16 ? kWideSets16 : kWideSets8) : kParseStaticLds;
  return p.smem + own <= (size_t)c->lds_limit;
}

// How often each entry is named by a code stream: usage[b][e] += number of codes equal to V + e (codes of base
// tokens and codes that name no entry are skipped).  One workgroup per sequence.
__global__ void __launch_bounds__(256) lzw_usage_kernel(LzwState st, const int32_t* codes, const int32_t* n_codes,
                                                        int stride, int32_t* usage) {
  const int b = blockIdx.x;
  const int n = n_codes ? min(max(n_codes[b], 0), stride) : stride;
  const int C = min(max(st.size[b], 0), st.cap);
  for (int i = threadIdx.x; i < n; i += 256) {
    const int e = codes[(size_t)b * stride + i] - st.V;
    if (e >= 0 && e < C) atomicAdd(&usage[(size_t)b * st.cap + e], 1);
  }
}

// Pruning / selective retention (zip2zip paper, discussion, "Codebook Management Strategy", item 1): entry e
// stays iff keep[e] != 0 and its prefix without the last token is a base token or an entry that stays; the
// survivors keep their order and are renumbered.  One wave per sequence, wave-uniform, in two sweeps over the
// entries in creation order (a prefix is always older than its extensions): the first walks the trie as it
// is to find every entry's prefix and decides who stays (new_id: new index or -1; prefix: scratch); the
// second empties the table, moves the survivors' rows down and inserts their edges under the new numbers.
__global__ void __launch_bounds__(kWave) lzw_prune_kernel(LzwArgs a, const int32_t* keep, int32_t* new_id, int32_t* prefix) {
  const LzwState& st = a.st;
  const int b = blockIdx.x;
  const int lane = threadIdx.x;
  const int V = st.V, M = st.M, cap = st.cap;
  const int C = min(max(__builtin_amdgcn_readfirstlane(st.size[b]), 0), cap);
  int32_t* ent_tokens = st.ent_tokens + (size_t)b * cap * M;
  int32_t* ent_len = st.ent_len + (size_t)b * cap;
  const int32_t* kp = keep + (size_t)b * cap;
  int32_t* nid = new_id + (size_t)b * cap;
  int32_t* pre = prefix + (size_t)b * cap;
  Table<false> t;
  table_open<false>(a, b, lane, false, &t);
  int kept = 0;
  for (int e = 0; e < C; ++e) {
    const int L = min(max(__builtin_amdgcn_readfirstlane(ent_len[e]), 2), M);
    const int32_t tok = lane < L ? ent_tokens[(size_t)e * M + lane] : 0;
    int32_t code = __builtin_amdgcn_readlane(tok, 0);
    for (int j = 1; j < L - 1; ++j) {
      int fp;
      code = V + t.find(code, __builtin_amdgcn_readlane(tok, j), &fp);     // exists: the codebook is prefix-closed
    }
    const int p = L == 2 ? -1 : code - V;
    // (read past the vector L1: the line may have been cached before lane 0 wrote this element)
    const int pn = p < 0 ? 0 : __builtin_amdgcn_readfirstlane(__hip_atomic_load(&nid[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const bool stays = __builtin_amdgcn_readfirstlane(kp[e]) != 0 && pn >= 0;
    if (lane == 0) {
      nid[e] = stays ? kept : -1;
      pre[e] = p;
    }
    kept += stays ? 1 : 0;
    __syncthreads();                                 // nid[e] is read by the entries that extend e
  }
  for (int i = lane; i < st.nslots; i += kWave) t.g[i] = kEmpty;
  sync_after_global_stores();                        // the re-insert sweep probes the cleared table past the L1
  for (int e = 0; e < C; ++e) {
    const int n = __builtin_amdgcn_readfirstlane(__hip_atomic_load(&nid[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (n < 0) continue;
    const int L = min(max(__builtin_amdgcn_readfirstlane(ent_len[e]), 2), M);
    const int32_t tok = lane < M ? ent_tokens[(size_t)e * M + lane] : -1;
    const int p = __builtin_amdgcn_readfirstlane(__hip_atomic_load(&pre[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const int32_t parent = p < 0 ? __builtin_amdgcn_readlane(tok, 0)
                                 : V + __builtin_amdgcn_readfirstlane(__hip_atomic_load(&nid[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    int free_pos = -1;
    t.find(parent, __builtin_amdgcn_readlane(tok, L - 1), &free_pos);
    __syncthreads();                                 // row e is read before row n <= e is overwritten
    if (lane == 0) {
      t.store((uint32_t)free_pos, edge_bits(parent, __builtin_amdgcn_readlane(tok, L - 1)) | (u64)(uint32_t)n);
      ent_len[n] = L;
    }
    if (lane < M) ent_tokens[(size_t)n * M + lane] = tok;
    __syncthreads();
  }
  for (int e = kept + lane; e < C; e += kWave) ent_len[e] = 0;            // the rows above the survivors are unused again
  for (int i = kept * M + lane; i < C * M; i += kWave) ent_tokens[i] = -1;
  if (lane == 0) {
    st.size[b] = kept;
    st.prev_code[b] = -1;
    st.prev_len[b] = 0;
    a.out_n[b] = kept;
  }
}

// Codebook prefilling: the given phrases become entries, in order, before any input is parsed (zip2zip
// paper, discussion, "Codebook Management Strategy", item 2).  A phrase is taken if it keeps the codebook what
// the parse kernels rely on: 2..M tokens, all in [0, V), its prefix without the last token a base token or an
// entry already, itself not an entry yet, and the codebook not full; the first phrase that is not ends the
// sequence's prefill with a status bit.  One wave per sequence, wave-uniform scalar walk of the trie in the
// global table.  a.in = phrases [B, stride, M], a.in_len = [B] counts or nullptr, a.out = phrase lengths
// [B, stride], a.out_n = [B] entries added.
__global__ void __launch_bounds__(kWave) lzw_prefill_kernel(LzwArgs a) {
  const LzwState& st = a.st;
  const int b = blockIdx.x;
  const int lane = threadIdx.x;
  const int V = st.V, M = st.M, cap = st.cap;
  const bool reset = a.flags == Z2Z_RESET;
  int C = reset ? 0 : __builtin_amdgcn_readfirstlane(st.size[b]);
  Table<false> t;
  table_open<false>(a, b, lane, reset, &t);
  const int n = call_length(a, b);
  const int32_t* phrases = a.in + (size_t)b * a.stride * M;
  const int32_t* lens = a.out + (size_t)b * a.stride;
  int status = 0, added = 0;
  for (int i = 0; i < n; ++i) {
    const int L = __builtin_amdgcn_readfirstlane(lens[i]);
    if (L < 2 || L > M) {
      status |= Z2Z_ST_BAD_TOKEN;
      break;
    }
    const int32_t tok = lane < L ? phrases[(size_t)i * M + lane] : 0;      // lane j = token j
    if (__any(lane < L && (tok < 0 || tok >= V))) {
      status |= Z2Z_ST_BAD_TOKEN;
      break;
    }
    int32_t code = __builtin_amdgcn_readlane(tok, 0);
    bool known = true;
    for (int j = 1; j < L - 1 && known; ++j) {
      int fp;
      const int idx = t.find(code, __builtin_amdgcn_readlane(tok, j), &fp);
      known = idx >= 0;
      code = V + idx;
    }
    int free_pos = -1;
    const int32_t last = __builtin_amdgcn_readlane(tok, L - 1);
    if (!known || t.find(code, last, &free_pos) >= 0 || free_pos < 0) {
      status |= Z2Z_ST_BAD_CODE;                     // prefix unknown, or the phrase is an entry already
      break;
    }
    if (C >= cap) {
      status |= Z2Z_ST_OVERFLOW;
      break;
    }
    table_insert<false>(a, b, lane, t, free_pos, C, code, last, tok, L - 1);
    ++C;
    ++added;
    __syncthreads();                                 // the slot is visible to the next phrase's walk
  }
  if (lane == 0) {
    st.size[b] = C;
    st.prev_code[b] = -1;                            // the parse starts afresh: no pending phrase
    st.prev_len[b] = 0;
    a.out_n[b] = added;
    a.status[b] = status;
  }
}

}  // namespace

int z2z_launch_lzw_reset(z2z_ctx* c, hipStream_t s) {
  c->enc_kept = false;   // the rows a keeping encoder pass left behind belong to the codebook as it was
  hipLaunchKernelGGL(lzw_reset_kernel, dim3(c->cfg.B), dim3(256), 0, s, c->st);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

int z2z_launch_codebook_usage(z2z_ctx* c, const int32_t* codes, const int32_t* n_codes, int32_t stride, int32_t* usage,
                              hipStream_t s) {
  hipLaunchKernelGGL(lzw_usage_kernel, dim3(c->cfg.B), dim3(256), 0, s, c->st, codes, n_codes, stride, usage);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

int z2z_launch_codebook_prune(z2z_ctx* c, const int32_t* keep, int32_t* new_id, int32_t* n_kept, hipStream_t s) {
  c->enc_kept = false;   // the rows a keeping encoder pass left behind belong to the codebook as it was
  if (!c->prune_prefix && c->cfg.cap > 0) return Z2Z_EHIP;       // (allocated by z2z_create)
  LzwArgs a;
  memset(&a, 0, sizeof(a));
  a.st = c->st;
  a.out_n = n_kept;
  hipLaunchKernelGGL(lzw_prune_kernel, dim3(c->cfg.B), dim3(kWave), 0, s, a, keep, new_id,
                     reinterpret_cast<int32_t*>(c->prune_prefix));
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

int z2z_launch_codebook_prefill(z2z_ctx* c, const int32_t* phrases, const int32_t* phrase_len, const int32_t* counts,
                                int32_t n_max, int32_t flags, int32_t* n_added, int32_t* status, hipStream_t s) {
  c->enc_kept = false;   // the rows a keeping encoder pass left behind belong to the codebook as it was
  LzwArgs a;
  memset(&a, 0, sizeof(a));
  a.st = c->st;
  a.in = phrases;
  a.in_len = counts;
  a.stride = n_max;
  a.flags = flags;
  a.out = const_cast<int32_t*>(phrase_len);          // read only
  a.out_n = n_added;
  a.out_stride = n_max;
  a.status = status;
  a.lds_ef = 0;
  if (flags & Z2Z_RESET) hipLaunchKernelGGL(lzw_clear_entries_kernel, dim3(c->cfg.B), dim3(256), 0, s, c->st);
  hipLaunchKernelGGL(lzw_prefill_kernel, dim3(c->cfg.B), dim3(kWave), 0, s, a);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

template <int WHERE>
static void launch_encode(const LzwArgs& a, int B, int nw, int sets, size_t smem, hipStream_t s) {
  if constexpr (WHERE == kLds) {
    if (sets == 1 && nw == 8) {
      hipLaunchKernelGGL((lzw_encode_kernel<8, WHERE, 1>), dim3(B), dim3(512), smem, s, a);
      return;
    }
  }
  switch (nw) {
    case 1: hipLaunchKernelGGL((lzw_encode_kernel<1, WHERE>), dim3(B), dim3(64), smem, s, a); break;
    case 8: hipLaunchKernelGGL((lzw_encode_kernel<8, WHERE>), dim3(B), dim3(512), smem, s, a); break;
    default: hipLaunchKernelGGL((lzw_encode_kernel<16, WHERE>), dim3(B), dim3(1024), smem, s, a); break;
  }
}
template <int WHERE>
static void launch_decode(const LzwArgs& a, int B, int nw, size_t smem, hipStream_t s) {
  if constexpr (WHERE == kLds) {
    if (nw == 4) {
      hipLaunchKernelGGL((lzw_decode_kernel<4, WHERE>), dim3(B), dim3(256), smem, s, a);
      return;
    }
  }
  switch (nw) {
    case 1: hipLaunchKernelGGL((lzw_decode_kernel<1, WHERE>), dim3(B), dim3(64), smem, s, a); break;
    case 8: hipLaunchKernelGGL((lzw_decode_kernel<8, WHERE>), dim3(B), dim3(512), smem, s, a); break;
    default: hipLaunchKernelGGL((lzw_decode_kernel<16, WHERE>), dim3(B), dim3(1024), smem, s, a); break;
  }
}

int z2z_launch_lzw_encode(z2z_ctx* c, const int32_t* tokens, const int32_t* lens, int32_t stride, int32_t flags,
                          int32_t* codes, int32_t* n_codes, int32_t out_stride, int32_t* status, hipStream_t s) {
  c->enc_kept = false;   // the rows a keeping encoder pass left behind belong to the codebook as it was
  LzwArgs a;
  memset(&a, 0, sizeof(a));
  a.st = c->st;
  a.in = tokens;
  a.in_len = lens;
  a.stride = stride;
  a.flags = flags;
  a.out = codes;
  a.out_n = n_codes;
  a.out_stride = out_stride;
  a.status = status;
  const ParsePlan p = plan(c, stride, flags, false, &a);
  if (!fits(c, p)) return Z2Z_EUNSUPPORTED;
  if (p.tags)
    hipLaunchKernelGGL((lzw_encode_kernel<16, kTag>), dim3(c->cfg.B), dim3(1024), p.smem, s, a);
  else if (p.per == 8 && p.nw == 16)
    hipLaunchKernelGGL((lzw_encode_kernel<16, kLds, 2, 8>), dim3(c->cfg.B), dim3(1024), p.smem, s, a);
  else if (p.per == 8)
    hipLaunchKernelGGL((lzw_encode_kernel<8, kLds, 2, 8>), dim3(c->cfg.B), dim3(512), p.smem, s, a);
  else if (p.lds)
    launch_encode<kLds>(a, c->cfg.B, p.nw, p.sets, p.smem, s);
  else
    launch_encode<kMem>(a, c->cfg.B, p.nw, p.sets, 0, s);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

int z2z_launch_lzw_decode(z2z_ctx* c, const int32_t* codes, const int32_t* n_codes, int32_t stride, int32_t flags,
                          int32_t* tokens, int32_t* n_tokens, int32_t out_stride, int32_t* status, hipStream_t s) {
  c->enc_kept = false;   // the rows a keeping encoder pass left behind belong to the codebook as it was
  LzwArgs a;
  memset(&a, 0, sizeof(a));
  a.st = c->st;
  a.in = codes;
  a.in_len = n_codes;
  a.stride = stride;
  a.flags = flags;
  a.out = tokens;
  a.out_n = n_tokens;
  a.out_stride = out_stride;
  a.status = status;
  const ParsePlan p = plan(c, stride, flags, true, &a);
  if (!fits(c, p)) return Z2Z_EUNSUPPORTED;
  const bool serial = stride <= 8 || c->opt_lzw_kernel == 3;
  // Long rows of few sequences: a second launch over all CUs takes the codes behind a full codebook.  A codebook that starts
  // empty is full after cap codes at the earliest; how many follow only the device knows, and the first launch goes on
  // by itself when they are fewer than kTailMin.  (16 sequences of 9700 codes, 8192 entries, nothing
  // left for it: 95 -> 98 us.)
  const bool tail = !serial && p.nw > 1 && 2 * c->cfg.B <= c->num_cu &&
                    stride >= ((flags & Z2Z_RESET) ? (int64_t)c->cfg.cap : 0) + 2 * kTailMin;
  a.tail_min = tail ? kTailMin : INT32_MAX;
  // (the window kernels clear the rows behind the new codebook themselves)
  if (serial && (flags & Z2Z_RESET)) hipLaunchKernelGGL(lzw_clear_entries_kernel, dim3(c->cfg.B), dim3(256), 0, s, c->st);
  if (serial && p.lds)
    hipLaunchKernelGGL(lzw_decode_serial_kernel<true>, dim3(c->cfg.B), dim3(kWave), p.smem, s, a);
  else if (serial)
    hipLaunchKernelGGL(lzw_decode_serial_kernel<false>, dim3(c->cfg.B), dim3(kWave), 0, s, a);
  else if (p.tags)
    hipLaunchKernelGGL((lzw_decode_kernel<16, kTag>), dim3(c->cfg.B), dim3(1024), p.smem, s, a);
  else if (p.lds)
    launch_decode<kLds>(a, c->cfg.B, p.nw, p.smem, s);
  else
    launch_decode<kMem>(a, c->cfg.B, p.nw, 0, s);
  if (tail) {
    const int parts = std::min(64, c->num_cu / c->cfg.B);
    hipLaunchKernelGGL(lzw_decode_tail_kernel, dim3(parts, c->cfg.B), dim3(1024), 0, s, a);
  }
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

int z2z_launch_step_update(z2z_ctx* c, const int32_t* codes, int32_t stride, const void* E, void* W_hyper,
                           int32_t* n_tokens, int32_t* status, hipStream_t s) {
  c->enc_kept = false;
  LzwArgs a;
  memset(&a, 0, sizeof(a));
  a.st = c->st;
  a.in = codes;
  a.in_len = nullptr;
  a.stride = 1;                         // one code per sequence; `stride` is the distance between them
  a.flags = Z2Z_APPEND;
  a.out = nullptr;
  a.out_n = n_tokens;
  a.out_stride = 0;
  a.status = status;
  a.lds_ef = 0;
  a.in_step = stride;
  z2z_embed::EmbedArgs ea;
  z2z_embed::fill_embed_args(c, E, W_hyper, &ea);
  const int chunks = c->cfg.d / (c->cfg.dtype == Z2Z_BF16 ? 8 : 4);
  int split = 1;
  while (split < kStepWaves && chunks >= 128 * split) split *= 2;    // a wave takes at least 64 chunks of the row
  ea.split = split;
  if (c->cfg.dtype == Z2Z_BF16)
    hipLaunchKernelGGL(lzw_step_update_kernel<true>, dim3(c->cfg.B), dim3(kStepWaves * kWave), 0, s, a, ea);
  else
    hipLaunchKernelGGL(lzw_step_update_kernel<false>, dim3(c->cfg.B), dim3(kStepWaves * kWave), 0, s, a, ea);
  Z2Z_HIP_TRY(hipGetLastError());
  return Z2Z_OK;
}

// Size the hash table for the device's LDS and raise the dynamic-LDS ceiling of the parse kernels.
// Load factor at a full codebook is at most 0.8 (at least 1.25 slots per entry; 2 or 4 when LDS allows).
int z2z_lzw_prepare(z2z_ctx* c) {
  LzwState& st = c->st;
  const int cap = st.cap;
  const int want4 = 4 * cap < 64 ? 64 : 4 * cap;
  const int want = 2 * cap < 64 ? 64 : 2 * cap;
  const int floor125 = cap + cap / 4 + 1;
  const int lds_slots = (c->lds_limit - kParseStaticLds) / (int)sizeof(u64);   // the encoder's own LDS comes first
  // With fewer sequences than CUs a workgroup has its CU to itself and the roomier table (shorter probe
  // sequences) is free; with many, LDS decides how many sequences a CU works on at once.
  const bool roomy = c->cfg.B < 256;
  // ... but not where it keeps the encoder from sets of eight slots per position, which gain more than the probes it shortens.
  const int beside_large_sets = (c->lds_limit - kWideSets16) / (int)sizeof(u64);
  // A CU holds up to four workgroups of 8 waves (32 waves of 64 registers; the decoder's, with 67, three): as many as there are
  // sequences for it, the tables as large as that leaves room for.  Another workgroup hides more than the longer probes cost: 2048 documents of
  // 1024 to 4096 tokens, encode (decode), cap 2048: 4096 slots, three per CU 162 us (152), 2906 slots, four 149 (125); cap
  // 3000: 6000 slots, two 237 (177), 4440 slots, three 171 (163).  More than there are sequences for only costs: 600 of 4096
  // tokens, cap 2048: 4096 slots 67 us, 2561 slots 81 (four workgroups on one CU, fewer on another).  That holds down to 1.25
  // slots per entry (2048 documents, encode (decode): cap 2150 170 us (145) -> 156 (119), cap 3500 210 (207) -> 172 (151)).  What
  // it costs are short calls on the tables where they are, nearly full ones above all: 1024 sequences, cap 2048, 97 % full, 4096
  // -> 2906 slots: an appended token 9.6 -> 10.8 us, a step update 11.8 -> 12.6, 16 appended codes 11.9 -> 14.  (Two steps of a probe at
  // once there gave back half of it, but its registers took a workgroup off the CU: decode of 768 of 400 codes 15.8 -> 20.2.)
  int shared = 0;
  if (c->cfg.B > c->num_cu) {
    for (int k = std::min(4, (c->cfg.B + c->num_cu - 1) / c->num_cu); k >= 2 && shared == 0; --k) {
      const int share = c->lds_limit / k & ~2047;      // (LDS is handed out in pieces of 1280 bytes)
      const int slots = std::min(want, (share - (int)sizeof(EncShared<8, 1>)) / (int)sizeof(u64));
      if (slots >= std::max(floor125, 64)) shared = slots;
    }
  }
  if (shared > 0) {
    st.nslots = shared;
    st.slots_fit_lds = 1;
  } else if (roomy && want4 + cap / 2 <= lds_slots) {        // room left for the decoder's entry info
    st.nslots = want <= beside_large_sets ? std::min(want4, beside_large_sets) : want4;
    st.slots_fit_lds = 1;
  } else if (want <= lds_slots) {
    st.nslots = want;
    st.slots_fit_lds = 1;
  } else if (floor125 <= lds_slots) {
    st.nslots = lds_slots;
    st.slots_fit_lds = 1;
  } else {
    // A table in memory: its tags in LDS, while a sequence has a CU to itself (several on a CU hide the latency of tables in
    // memory, and the tags would keep them from it).
    st.tags_fit_lds = c->cfg.B <= c->num_cu && want <= (c->lds_limit - kParseStaticLds) / (int)sizeof(uint16_t);
    st.nslots = want;
    st.slots_fit_lds = 0;
  }
  st.nslots &= ~1;                                     // whole buckets
  const void* parse[] = {reinterpret_cast<const void*>(lzw_encode_kernel<1, kLds>),
                         reinterpret_cast<const void*>(lzw_encode_kernel<8, kLds, 1>),
                         reinterpret_cast<const void*>(lzw_encode_kernel<8, kLds>),
                         reinterpret_cast<const void*>(lzw_encode_kernel<16, kLds>),
                         reinterpret_cast<const void*>(lzw_decode_kernel<1, kLds>),
                         reinterpret_cast<const void*>(lzw_decode_kernel<4, kLds>),
                         reinterpret_cast<const void*>(lzw_decode_kernel<8, kLds>),
                         reinterpret_cast<const void*>(lzw_decode_kernel<16, kLds>),
                         reinterpret_cast<const void*>(lzw_encode_kernel<16, kTag>),
                         reinterpret_cast<const void*>(lzw_decode_kernel<16, kTag>),
                         reinterpret_cast<const void*>(lzw_decode_serial_kernel<true>)};
  for (const void* f : parse)
    Z2Z_HIP_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, c->lds_limit - kParseStaticLds));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(lzw_encode_kernel<16, kLds, 2, 8>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, c->lds_limit - kWideSets16));
  Z2Z_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(lzw_encode_kernel<8, kLds, 2, 8>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, c->lds_limit - kWideSets8));
  return Z2Z_OK;
}

// Device-side helpers shared by the attention kernels (gfx950 / CDNA4 only): types, lane exchanges, LDS addresses,
// waits, the order of workgroups, the cut of a launch, and the kernels' arguments.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace s1f {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

#define S1F_DEV __device__ __forceinline__
#define S1F_LDS(ptr_type, p) ((__attribute__((address_space(3))) ptr_type *)(p))

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMaxFloat = 3.402823466e38f;

template <typename T> struct Elem;
template <> struct Elem<float> { static constexpr int CE = 4; };    // elements per 16-byte chunk
template <> struct Elem<bf16_t> { static constexpr int CE = 8; };

S1F_DEV float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }   // v_exp_f32; exp2(-inf) = 0
// The lane's own value and the value held by its partner lane (lane ^ 32), in unspecified order.
// v_permlane32_swap exchanges the upper half of its first operand with the lower half of its second, so
// with both operands equal to x the register pair ends up as (own, partner) in the lower half-wave and
// (partner, own) in the upper one.  Written as assembly: with two identical operands the compiler's
// builtin hands back its first result for both.  The leading s_nop covers the wait states the
// instruction needs after a vector write of its operands.
S1F_DEV void own_and_partner(float x, float &a, float &b) {
  a = x;
  b = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
S1F_DEV float max_xor32(float x) {
  float a, b;
  own_and_partner(x, a, b);
  return fmaxf(a, b);
}
S1F_DEV float sum_xor32(float x) {
  float a, b;
  own_and_partner(x, a, b);
  return a + b;
}

constexpr int pow2_at_least(int x) { int p = 1; while (p < x) p *= 2; return p; }

// LDS addresses are handled as 32-bit byte offsets (lds_addr) so that address arithmetic stays in the LDS address space.
typedef unsigned lds_addr;
S1F_DEV lds_addr to_lds_addr(const void *p) { return (lds_addr)(uintptr_t)S1F_LDS(const char, p); }
template <typename V> S1F_DEV V lds_load(lds_addr a) {
  return *reinterpret_cast<const __attribute__((address_space(3))) V *>((uintptr_t)a);
}
// Marks a value loaded from memory as used here.  The compiler then waits for the load at this point
// instead of at the first real use; kernels call it on operands fetched before their main loop, whose
// first use inside the loop would otherwise put a vmcnt wait there that also waits (on every iteration)
// for the asynchronous tile copies in flight.
template <typename V> S1F_DEV void settle(V &v) { asm volatile("" : "+v"(v)); }

// Wait until every asynchronous tile copy issued by this wave has landed (vmcnt(0), other counters untouched).
S1F_DEV void wait_async_tiles() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// The same, except that the wave's N most recent copy instructions may still be in flight (loads complete in order).
template <int N> S1F_DEV void wait_async_tiles_but_last() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }

// Store 4 consecutive head_dim elements of one row.
template <typename T> S1F_DEV void store4(T *p, float a, float b, float c, float d);
template <> S1F_DEV void store4<float>(float *p, float a, float b, float c, float d) {
  *reinterpret_cast<f32x4 *>(p) = f32x4{a, b, c, d};
}
template <> S1F_DEV void store4<bf16_t>(bf16_t *p, float a, float b, float c, float d) {
  bf16x4 r = {(bf16_t)a, (bf16_t)b, (bf16_t)c, (bf16_t)d};
  *reinterpret_cast<bf16x4 *>(p) = r;
}

// Division by a number that the host knows: n / d = n * mul >> (31 + shift) for 0 <= n < 2^31 (with 2^shift >= d and mul =
// floor(2^(31 + shift) / d) + 1 the product exceeds n * 2^(31 + shift) / d by less than 2^(31 + shift) / d).  Workgroups decode their
// number with half a dozen of them before their first load; divisions, of some 30 scalar and vector instructions each, took longer: forward
// of 4 heads, 256 rows behind 768 keys, bf16, D 64 6.4 -> 6.1 us, 63 backwards of up to 30 us 2 % on average.
struct Divisor {
  uint32_t mul, shift;
  int32_t d;
  static Divisor of(int64_t d) {
    uint32_t s = 0;
    while ((int64_t(1) << s) < d) ++s;
    return Divisor{(uint32_t)(((uint64_t)1 << (31 + s)) / (uint64_t)d + 1), s, (int32_t)d};
  }
};
S1F_DEV int div(int n, const Divisor &by) { return (int)(((uint64_t)(uint32_t)n * by.mul) >> (31 + by.shift)); }
S1F_DEV void div_mod(int n, const Divisor &by, int &quotient, int &rest) {
  quotient = div(n, by);
  rest = n - quotient * by.d;
}

// Workgroup id -> (tile, batch*head).  The hardware hands consecutive workgroup ids to the 8 XCDs in turn,
// and each XCD has its own L2.  All tiles of one (batch, head) stream the same K/V prefix (or the same
// Q/dO segment), so they are given ids that land on one XCD: the shared operand is then fetched from HBM once
// per XCD instead of once per workgroup.  An XCD takes n_bh / 8 CONSECUTIVE (batch, head) pairs, so that query
// heads sharing a K/V head share an XCD as well.  Within an XCD the ids run head by head (`tile_major` = 0: best
// when the tiles of a launch take about the same time, i.e. behind a long prefix) or tile by tile over the XCD's
// heads (`tile_major` = 1: the light tiles of every head come last, which shortens the end of a launch whose
// tiles differ a lot, i.e. the first segments; and heads that share K/V rows walk them together).  Falls back to
// the plain order when the number of (batch, head) pairs is not a multiple of 8.
// tiles: per (batch, head) pair; per_xcd: an eighth of the pairs, where that is a whole number
S1F_DEV void decode_workgroup(int id, const Divisor &tiles, int n_bh, const Divisor &per_xcd, int tile_major, int &tile, int &bh) {
  if ((n_bh & 7) == 0) {
    const int slot = id >> 3;
    if (tile_major) div_mod(slot, per_xcd, tile, bh);
    else div_mod(slot, tiles, bh, tile);
    bh += (id & 7) * per_xcd.d;
  } else {
    div_mod(id, tiles, bh, tile);
  }
}

// Cut launches.  The workgroups of a launch are handed to the chip's workgroup slots in id order; when the last
// round of units fills only part of the slots, the launch ends with most of the chip idle for the length of one
// unit (forward and dQ: a row tile against its whole prefix; dK/dV: a key tile against the rows that see it).  The host may
// therefore cut each of the LAST units of a launch into n_split chunks, along the keys or (dK/dV) along the query rows,
// which then run side by side; a chunk leaves a partial result in a workspace (the first chunk of a dK/dV unit adds to the
// accumulators itself) and a small second kernel merges them.  Row tiles deal out evenly the keys that every row of the
// unit sees in full (`full`, counted in pieces of the kernel's step; see chunk_range); the last chunk also takes the pieces
// on the diagonal.
// In: workgroup id.  Out: unit id, the chunk's number and its index in the workspace (-1: whole).
constexpr int kMaxChunks = 16;   // most chunks a unit is ever cut into
struct UnitChunk {
  int unit, chunk, n_chunks, slot;
};
// Chunk-major order: the ids past n_whole first run through one chunk of every split unit, then through the next
// chunk, so that the workgroups that start one after the other walk the SAME keys of neighbouring row tiles and
// share them in the L2 (in unit-major order, a unit's chunks side by side, the workgroups of one key range start
// too far apart for that: 1.5 to 1.7 times the reads from memory over a 32K-token step).  The chunk that holds the diagonal goes first: it is
// the longest.  A chunk keeps its unit's XCD (workgroup ids go to the XCDs in turn, and decode_workgroup ties a unit
// to the XCD of its id) whenever n_whole and the number of split units are multiples of 8, which they are when the
// heads are pinned to XCDs.
S1F_DEV UnitChunk split_unit(int id, int n_whole, int n_split, int n_split_units, const Divisor &split_units) {
  if (id < n_whole) return UnitChunk{id, 0, 1, -1};
  int pass, idx;
  div_mod(id - n_whole, split_units, pass, idx);
  const int chunk = n_split - 1 - pass;
  return UnitChunk{n_whole + idx, chunk, n_split, chunk * n_split_units + idx};
}
// Workspace index of chunk 0 of split unit number `unit_idx` (counted from n_whole), and the index step to its next chunk.
S1F_DEV void chunk_slots(int unit_idx, int n_split_units, int &first, int &step) {
  first = unit_idx;
  step = n_split_units;
}
// (at most 16 chunks of 2^25 pieces)
S1F_DEV void chunk_range(const UnitChunk &u, const Divisor &split, int full, int total, int &begin, int &end) {
  begin = u.chunk == 0 ? 0 : div(u.chunk * full, split);
  end = u.chunk + 1 < u.n_chunks ? div((u.chunk + 1) * full, split) : total;
}

// Arguments common to the three kernels (all strides in elements of the tensor they index).
struct AttnArgs {
  const void *q, *k, *v, *out, *dout;   // out: written by fwd, read by bwd
  void *out_w, *dq;
  float *lse;                            // [batch, Hq, seg_len]
  float *delta;                          // workspace (bwd): two planes [batch, Hq, seg_len], ws_plane floats apart:
                                         // -lse/scale, then -delta = -rowsum(dO * O)
  int64_t ws_plane;
  float *dk_acc, *dv_acc;
  int64_t q_sb, q_sh, q_ss;
  int64_t kv_sb, kv_sh, kv_ss;
  int32_t seg_off, seg_len;
  int32_t n_q_heads, group;              // group = Hq / Hkv
  int32_t n_tiles, n_bh;                 // launch shape: tiles per (batch, head) and number of (batch, head) pairs
  int32_t tile_major;                    // order of the workgroups within an XCD (see decode_workgroup)
  float scale;                           // 1/sqrt(head_dim)
  // The cut of the last units of a launch (see split_unit): workgroup ids below n_whole are whole units; the
  // n_split_units units after them are cut into n_split chunks each.
  int32_t n_whole, n_split, n_split_units;
  int32_t bm;                            // forward and dQ: rows per unit
  int32_t first_id;                      // forward: > 0 in a second launch, over the rows of the units from n_whole = first_id on
  Divisor by_heads, by_kv_heads, by_group;   // what a workgroup's number is decoded with: query and K/V heads, group,
  Divisor by_tiles, by_xcd;                  // n_tiles, n_bh / 8 (see decode_workgroup),
  Divisor by_split, by_split_units;          // n_split, n_split_units,
  Divisor by_rag;                            // second launch of a forward: its tiles per (batch, head) behind the n_tiles whole units,
  Divisor by_groups;                         // workgroups per unit of a merge, or per (batch, head) of the row statistics
  float *part;                           // partial results of the chunks: [chunk][cut unit][rows per unit][head_dim]
  float *part_ml;                        // forward only: running maximum (log2 units) and row sum, [..][rows per unit][2]
};

}  // namespace s1f

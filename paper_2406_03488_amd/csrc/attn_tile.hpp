// Matrix building blocks of the attention kernels (gfx950): 16x16 matrix instructions, 32-row operand tiles in LDS.
//
// Vocabulary:
//   lane      16*j + n with j in 0..3, n in 0..15
//   block     a 16x16 fp32 result held as 4 registers per lane: register v of lane (n, j) is element (row 4*j + v,
//             column n).  Kernels work on 32x32 scores as 2x2 blocks [rb][cb].
//   operand   what one lane feeds to one matrix instruction: A row n or B column n, and of the contraction index
//             bf16 (16x16x32): the 8 elements 8*j .. 8*j+7;   fp32 (16x16x4, four in a row): the 4 elements 4*j .. +3
//   slab      the 32 rows of a block pair [0..1][cb] as contraction index, so that scores are fed back as an operand
//             without any movement between lanes: slot (j, e) is row 16*(e/4) + 4*j + e%4, which lane (n, j) holds.
//             The other operand is read from LDS in the same row order.
//
// Why 16x16: a register-resident loop of v_mfma_f32_16x16x32_bf16 on N(0,1) operands sustains 1880-1920 TFLOP/s here,
// one of v_mfma_f32_32x32x16_bf16 1680 (the chip is power-limited; a 32x32 result passes twice the accumulator data per
// FLOP).  The operand traffic is the same when every A operand is used for two column blocks.
#pragma once
#include "attn_device.hpp"

namespace s1f {

S1F_DEV f32x4 mma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
S1F_DEV f32x4 mma16(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// Reductions over the four lanes that hold the rows of one column (lane ^ 16, lane ^ 32).  v_permlane16_swap exchanges
// the odd 16-lane rows of its first operand with the even ones of its second; see own_and_partner.
S1F_DEV void rows16_pair(float x, float &a, float &b) {
  a = x;
  b = x;
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
S1F_DEV float max_over_rows(float x) {
  float a, b;
  rows16_pair(x, a, b);
  return max_xor32(fmaxf(a, b));
}
S1F_DEV float sum_over_rows(float x) {
  float a, b;
  rows16_pair(x, a, b);
  return sum_xor32(a + b);
}

// The lane's number, computed anew where it is rarely needed instead of kept in a register across the main loops.
S1F_DEV int lane_id() {
  int x = -1;
  asm volatile("" : "+s"(x));
  return __builtin_amdgcn_mbcnt_hi(x, __builtin_amdgcn_mbcnt_lo(x, 0));
}
S1F_DEV float uniform(float x) { return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x))); }

// A [32 x D] tile in LDS, in pieces of 1 KiB: piece (rh, kq) = rows 16*rh .. +15, bytes 64*kq .. +63 of the rows, i.e.
// exactly the A operand of rows 16*rh for contraction step kq.  Inside a piece chunk c (16 bytes) of row r lies in slot
// 4*(r ^ rot) + (c ^ f(r)), f(r) = -(r / 4) mod 4; rot = kq & 3 in fp32, else 0.  Neither access pattern below has
// bank conflicts (the 16 lanes that a 128-bit read serves together, 0-3 with 12-15, 20-23 and 24-27 and so on, and the
// 32 of a 64-bit one cover all 64 banks), and the piece enters every
// address as a constant: one address register per pattern, where rows stored whole and swizzled took a vector
// instruction per operand.  Four consecutive slots hold 64 consecutive bytes of a row, which keeps the copies coalesced.
template <typename T, int D> struct Tile32 {
  static constexpr int CE = Elem<T>::CE;
  static constexpr int CPR = D / CE;                 // 16-byte chunks per row
  static constexpr int NP = (CPR + 3) / 4;           // pieces per row half
  static constexpr int BYTES = 2 * NP * 1024;
  static_assert(D % CE == 0, "head_dim must be a whole number of 16-byte chunks");
  S1F_DEV static int f(int r) { return -(r >> 2) & 3; }
  S1F_DEV static int rot(int kq) { return sizeof(T) == 4 ? kq & 3 : 0; }
};

// An LDS address as the compiler shall keep it: without this it folds the constant offsets of the operands into as many
// registers of their own (hoisted out of the loop, and spilled) instead of into the read instructions.
S1F_DEV lds_addr opaque(lds_addr x) {
  asm("" : "+v"(x));
  return x;
}

// Operands out of (and results behind) a Tile32.
//   nat   contraction along D.  Operand i = (row half i/NK, step i%NK), NN of them: row n of the half.
//   tr    contraction along the tile's 32 rows in slab order, NT of them: rows of A are head_dim.
//   RowOp the other operand of a nat product: one row per lane (row n of a 16-row block), held in registers
//   Slab  the other operand of a tr product
//   acc   [D/16] blocks of a tr product; quad q of them is four consecutive head_dim elements from quad_d0(q, j)
template <typename T, int D> struct Mat;

template <int D> struct Mat<bf16_t, D> {
  typedef Tile32<bf16_t, D> TL;
  typedef bf16x8 Frag;
  typedef bf16x8 Slab;
  static constexpr int NKS = TL::CPR / 4;            // whole steps of 32; head_dim 80 ends with half a one
  static constexpr int NK = TL::NP, NN = 2 * NK, NT = D / 16, DB = D / 16;
  static_assert(TL::CPR % 4 == 0 || TL::CPR % 4 == 2, "a last step of 16");
  struct RowOp {
    Frag f[NK];
  };
  unsigned nat_, tail_, tr_[2];
  S1F_DEV void init(int lane) {
    const int n = lane & 15, j = lane >> 4;
    nat_ = 64 * n + 16 * (j ^ TL::f(n));
    tail_ = 64 * n + 16 * ((j >> 1) ^ TL::f(n)) + 8 * (j & 1);
    // ds_read_b64_tr_b16: within 16 lanes, lane i supplies the address of 4 consecutive elements (row i/4 of a 4x16
    // matrix, columns 4*(i%4)..+3) and lane n receives column n of that matrix
    const int r = 4 * j + (n >> 2);
#pragma unroll
    for (int o = 0; o < 2; ++o) tr_[o] = 64 * r + 16 * ((2 * o + ((n & 3) >> 1)) ^ TL::f(r)) + 8 * (n & 1);
  }
  // The last 16 elements of head_dim 80 go through the same instruction as the others, four of them per lane and four
  // zeros: v_mfma_f32_16x16x16_bf16 takes as long, and right behind a 16x16x32 on the same accumulator (one column block
  // per wave) it returned wrong sums, the compiler seeing no wait states to insert between the two.
  S1F_DEV static Frag padded(s16x4 x) {
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x4 zero = {0, 0, 0, 0};
    s16x8 r = __builtin_shufflevector(x, zero, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(Frag, r);
  }
  // The lane's addresses in one tile: everything else about an operand is a constant offset.
  struct Nat {
    lds_addr a, tail;
  };
  struct Tr {
    lds_addr a[2];
  };
  S1F_DEV Nat nat_at(lds_addr tile) const { return Nat{opaque(tile + nat_), NK > NKS ? opaque(tile + tail_) : 0u}; }
  S1F_DEV Tr tr_at(lds_addr tile) const { return Tr{{opaque(tile + tr_[0]), opaque(tile + tr_[1])}}; }
  S1F_DEV static Frag nat(const Nat &x, int i, unsigned delta = 0) {
    const unsigned piece = i * 1024 + delta;
    if (i % NK < NKS) return lds_load<Frag>(x.a + piece);
    return padded(lds_load<s16x4>(x.tail + piece));
  }
  S1F_DEV static Frag tr(const Tr &x, int t, unsigned delta = 0) {
    const lds_addr p = x.a[t & 1] + (unsigned)(t >> 1) * 1024 + delta;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        reinterpret_cast<__attribute__((address_space(3))) s16x4 *>((uintptr_t)p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        reinterpret_cast<__attribute__((address_space(3))) s16x4 *>((uintptr_t)(p + TL::NP * 1024)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    s16x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(Frag, r);
  }
  // row pointer -> the lane's share of the row
  S1F_DEV static void load_row(RowOp &o, const bf16_t *row, int j) {
#pragma unroll
    for (int k = 0; k < NK; ++k)
      o.f[k] = k < NKS ? *reinterpret_cast<const Frag *>(row + 32 * k + 8 * j)
                       : padded(*reinterpret_cast<const s16x4 *>(row + 32 * k + 4 * j));
  }
  S1F_DEV static float dot(const RowOp &x, const RowOp &y) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
      for (int e = 0; e < (k < NKS ? 8 : 4); ++e) s += (float)x.f[k][e] * (float)y.f[k][e];
    return s;
  }
  S1F_DEV static f32x4 mma_nat(int i, Frag a, const RowOp &o, f32x4 c) {
    return mma16(a, o.f[i % NK], c);
  }
  // step k of a product along D whose other operand comes from LDS as well
  S1F_DEV static f32x4 mma_op(int, Frag a, Frag b, f32x4 c) { return mma16(a, b, c); }
  S1F_DEV static Slab slab(f32x4 x, f32x4 y) {
    Slab r;
#pragma unroll
    for (int e = 0; e < 4; ++e) { r[e] = (bf16_t)x[e]; r[4 + e] = (bf16_t)y[e]; }
    return r;
  }
  S1F_DEV static void settle_slab(Slab &s) { settle(s); }
  S1F_DEV static void mma_tr(int t, Frag a, const Slab &s, f32x4 (&acc)[DB]) { acc[t] = mma16(a, s, acc[t]); }
  S1F_DEV static int quad_d0(int q, int j) { return 16 * q + 4 * j; }
  S1F_DEV static f32x4 quad(const f32x4 (&acc)[DB], int q) { return acc[q]; }
};

// fp32: one 128-bit read feeds four matrix instructions.  In a nat product they contract elements 4*j+e of the step,
// e = 0..3.  In a tr product a lane reads four consecutive elements 4*n..+3 of a 64-wide group of head_dim, which are
// row n of four blocks: block 4*G+e holds d = 64*G + 4*row + e.  A last group of 16 (head_dim 80) is read one by one.
template <int D> struct Mat<float, D> {
  typedef Tile32<float, D> TL;
  typedef f32x4 Frag;
  struct Slab {
    f32x4 r[2];
  };
  static constexpr int NK = D / 16, NN = 2 * NK, NG = D / 64, DB = D / 16;
  static constexpr bool TAIL = D % 64 != 0;
  static constexpr int NT = 8 * NG + (TAIL ? 8 : 0);
  static_assert(D % 64 == 0 || D % 64 == 16, "whole groups of 64 and at most one of 16");
  struct RowOp {
    Frag f[NK];
  };
  unsigned nat_, tr_, tail_;
  S1F_DEV void init(int lane) {
    const int n = lane & 15, j = lane >> 4;
    nat_ = 64 * n + 16 * (j ^ TL::f(n));                                              // step k: ^ 64 * (k & 3)
    tr_ = 1024 * (n >> 2) + 64 * (4 * j + (n >> 2)) + 16 * ((n & 3) ^ TL::f(4 * j));  // row 4*j + v: ^ 64 * v
    tail_ = 64 * 4 * j + 16 * ((n >> 2) ^ TL::f(4 * j)) + 4 * (n & 3);
  }
  struct Nat {
    lds_addr a[4];
  };
  struct Tr {
    lds_addr a[4], tail;
  };
  S1F_DEV Nat nat_at(lds_addr tile) const {
    return Nat{{opaque(tile + nat_), opaque(tile + (nat_ ^ 64u)), opaque(tile + (nat_ ^ 128u)), opaque(tile + (nat_ ^ 192u))}};
  }
  S1F_DEV Tr tr_at(lds_addr tile) const {
    return Tr{{opaque(tile + tr_), opaque(tile + (tr_ ^ 64u)), opaque(tile + (tr_ ^ 128u)), opaque(tile + (tr_ ^ 192u))},
              TAIL ? opaque(tile + tail_) : 0u};
  }
  S1F_DEV static Frag nat(const Nat &x, int i, unsigned delta = 0) {
    return lds_load<Frag>(x.a[(i % NK) & 3] + (unsigned)(i * 1024 + delta));
  }
  S1F_DEV static Frag tr(const Tr &x, int t, unsigned delta = 0) {
    if (t < 8 * NG) {
      const int rv = t / NG, g = t % NG;
      return lds_load<Frag>(x.a[rv & 3] + (unsigned)(((rv >> 2) * TL::NP + 4 * g) * 1024 + delta));
    }
    const int rv = t - 8 * NG;
    const float y = lds_load<float>(x.tail + (unsigned)(((rv >> 2) * TL::NP + 4 * NG) * 1024 + 64 * (rv & 3) + delta));
    return Frag{y, y, y, y};
  }
  S1F_DEV static void load_row(RowOp &o, const float *row, int j) {
#pragma unroll
    for (int k = 0; k < NK; ++k) o.f[k] = *reinterpret_cast<const Frag *>(row + 16 * k + 4 * j);
  }
  S1F_DEV static float dot(const RowOp &x, const RowOp &y) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) s += x.f[k][e] * y.f[k][e];
    return s;
  }
  S1F_DEV static f32x4 mma_nat(int i, Frag a, const RowOp &o, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = mma16(a[e], o.f[i % NK][e], c);
    return c;
  }
  S1F_DEV static f32x4 mma_op(int, Frag a, Frag b, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = mma16(a[e], b[e], c);
    return c;
  }
  S1F_DEV static Slab slab(f32x4 x, f32x4 y) { return Slab{{x, y}}; }
  S1F_DEV static void settle_slab(Slab &) {}
  S1F_DEV static void mma_tr(int t, Frag a, const Slab &s, f32x4 (&acc)[DB]) {
    if (t < 8 * NG) {
      const int rv = t / NG, g = t % NG;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[4 * g + e] = mma16(a[e], s.r[rv >> 2][rv & 3], acc[4 * g + e]);
    } else if constexpr (TAIL) {
      const int rv = t - 8 * NG;
      acc[4 * NG] = mma16(a[0], s.r[rv >> 2][rv & 3], acc[4 * NG]);
    }
  }
  S1F_DEV static int quad_d0(int q, int j) { return q < 4 * NG ? 64 * (q >> 2) + 16 * j + 4 * (q & 3) : 64 * NG + 4 * j; }
  S1F_DEV static f32x4 quad(const f32x4 (&acc)[DB], int q) {
    if constexpr (TAIL)
      if (q >= 4 * NG) return acc[4 * NG];
    const int g = 4 * (q >> 2), v = q & 3;
    return f32x4{acc[g][v], acc[g + 1][v], acc[g + 2][v], acc[g + 3][v]};
  }
};

// Asynchronous copy of two Tile32s (the second right behind the first) from global memory by the four waves of a
// workgroup: wave w copies rows 16*(w & 1).. of tile w / 2.  One global_load_lds_dwordx4 moves 16 bytes per lane into
// 1 KiB of consecutive LDS, i.e. fills one piece: lane l lands at M0 + immediate offset + 16*l, and the immediate offset
// is added to the global address as well.  Up to four of a wave's NP pieces share one value of M0 (rewriting M0 between
// copies makes them complete one after the other instead of overlapping).  Written as assembly so that the compiler's
// wait-count pass does not tie LDS reads of OTHER ring stages to these copies; callers order the copies against their
// readers with wait_async_tiles() + a workgroup barrier.
// The address is (scalar base of the piece) + (32-bit lane offset fixed at init).  The pieces of a row half differ by
// 64 bytes in the scalar base and share the lane offset, except that fp32 has one per row rotation and that the last
// piece of head_dim 80 in bf16, half of it past the row's end, has its own (those slots re-read a valid chunk and are
// never used).  Rows past the last valid one re-read it (callers mask them).
template <typename T, int D> struct TilePairCopy {
  typedef Tile32<T, D> TL;
  static constexpr int NP = TL::NP;
  static constexpr bool PARTIAL = TL::CPR % 4 != 0;
  static constexpr int NV = sizeof(T) == 4 ? 4 : PARTIAL ? 2 : 1;
  unsigned voff[NV];

  S1F_DEV static constexpr int vclass(int kq) { return sizeof(T) == 4 ? kq & 3 : (PARTIAL && kq == NP - 1) ? 1 : 0; }
  S1F_DEV static int slot_row(int wave, int v, int lane) { return 16 * (wave & 1) + ((lane >> 2) ^ (sizeof(T) == 4 ? v : 0)); }
  S1F_DEV void init(int wave, int lane, int64_t row_stride) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int r = slot_row(wave, v, lane);
      int c = (lane & 3) ^ TL::f(r & 15);   // chunk within the piece
      if (sizeof(T) == 2 && v == 1 && c >= TL::CPR % 4) c -= 2;
      voff[v] = (unsigned)((r * row_stride + c * TL::CE) * (int64_t)sizeof(T));
    }
  }
  // pieces kq .. kq+N-1; tb: first byte of the tile's first row, advanced to piece kq
  template <int N> S1F_DEV static void issue_group(unsigned dst, const char *tb, unsigned o0, unsigned o1, unsigned o2, unsigned o3) {
    if (N == 1)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(o0), "s"(tb) : "m0");
    else if (N == 2)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\t"
                   "global_load_lds_dwordx4 %2, %4 offset:1024"
                   : : "s"(dst), "v"(o0), "v"(o1), "s"(tb), "s"(tb - 960) : "m0");
    else if (N == 3)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %4\n\t"
                   "global_load_lds_dwordx4 %2, %5 offset:1024\n\t"
                   "global_load_lds_dwordx4 %3, %6 offset:2048"
                   : : "s"(dst), "v"(o0), "v"(o1), "v"(o2), "s"(tb), "s"(tb - 960), "s"(tb - 1920) : "m0");
    else
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %5\n\t"
                   "global_load_lds_dwordx4 %2, %6 offset:1024\n\t"
                   "global_load_lds_dwordx4 %3, %7 offset:2048\n\t"
                   "global_load_lds_dwordx4 %4, %8 offset:3072"
                   : : "s"(dst), "v"(o0), "v"(o1), "v"(o2), "v"(o3), "s"(tb), "s"(tb - 960), "s"(tb - 1920), "s"(tb - 2880)
                   : "m0");
  }
  // row0/row1: the tiles' first rows in the two tensors (wave-uniform); left0/left1: valid rows from there on (WHOLE: at
  // least 32); stage: LDS address of the first tile
  template <bool WHOLE = false>
  S1F_DEV void issue(const T *row0, const T *row1, int64_t row_stride, int left0, int left1, lds_addr stage, int wave) const {
    // both are wave-uniform by construction; say so where the compiler cannot prove it
    const unsigned dst = __builtin_amdgcn_readfirstlane(stage + (unsigned)(wave * NP * 1024));
    const uint64_t tbits = reinterpret_cast<uint64_t>(wave >= 2 ? row1 : row0);
    const char *tb = reinterpret_cast<const char *>(
        ((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(tbits >> 32)) << 32) |
        (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)tbits));
    unsigned off[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) off[v] = voff[v];
    const int rows_left = wave >= 2 ? left1 : left0;
    if (!WHOLE && rows_left < 32) {   // the sequence ends inside this tile
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int over = slot_row(wave, v, lane_id()) - (rows_left - 1);
        if (over > 0) off[v] -= (unsigned)(over * row_stride * (int64_t)sizeof(T));
      }
    }
    constexpr int G = NP < 4 ? NP : 4;
#pragma unroll
    for (int i = 0; i + G <= NP; i += G)
      issue_group<G>(dst + i * 1024, tb + i * 64, off[vclass(i)], off[vclass(i + (G > 1 ? 1 : 0))],
                     off[vclass(i + (G > 2 ? 2 : 0))], off[vclass(i + (G > 3 ? 3 : 0))]);
#pragma unroll
    for (int i = NP / G * G; i < NP; ++i) issue_group<1>(dst + i * 1024, tb + i * 64, off[vclass(i)], 0, 0, 0);
  }
};

// Ring of five stages of one K and one V tile each, shared by the forward and the dQ kernel.  Step k computes on tiles
// k and k+1 and reads the first operands of tile k+2; tile k+4 is copied into the stage of tile k-1 meanwhile.  A copy
// therefore has two steps to land: a launch that leaves one workgroup per compute unit spends 0.4-0.5 us on a step, less
// than memory takes to answer.  With one step, 64 heads of 256 rows behind 16384 keys (forward, head_dim 128, 64-row
// units) took 359 us, with two 237.
template <typename T, int D> struct TileRing {
  static constexpr int STAGE_BYTES = 2 * Tile32<T, D>::BYTES;   // K tile then V tile
  static constexpr int LDS_BYTES = 5 * STAGE_BYTES;
  typedef TilePairCopy<T, D> Copy;
  Copy ld;
  const T *k_next, *v_next;      // first rows of the tile that the next copy fills
  int64_t row_stride;
  int to_issue, rows_left;       // tiles not copied yet; rows of the prefix from k_next on
  lds_addr st[5];                // stages of tiles k .. k+4 (the last is also that of tile k-1)
  int wave;
  S1F_DEV void init(const T *k, const T *v, int64_t row_stride_, int tiles, int rows, lds_addr lds, int wave_, int lane) {
    ld.init(wave_, lane, row_stride_);
    k_next = k; v_next = v;
    row_stride = row_stride_;
    to_issue = tiles; rows_left = rows;
#pragma unroll
    for (int i = 0; i < 5; ++i) st[i] = lds + (unsigned)(i * STAGE_BYTES);
    wave = wave_;
  }
  // WHOLE: there is a tile left and it is not the last of the sequence
  template <bool WHOLE = false> S1F_DEV void issue(int i) {
    if (!WHOLE && to_issue <= 0) return;
    ld.template issue<WHOLE>(k_next, v_next, row_stride, rows_left, rows_left, st[i], wave);
    --to_issue;
    rows_left -= 32;
    k_next += 32 * row_stride;
    v_next += 32 * row_stride;
  }
  // Start of the step whose current tile is k: tile k+2 has landed for every wave, and every wave has finished reading
  // tile k-1.  `left`: tiles after the current one.
  template <bool WHOLE> S1F_DEV void begin_step(int left) {
    if (WHOLE || left >= 3) wait_async_tiles_but_last<Copy::NP>();   // tile k+3 may still be in flight
    else wait_async_tiles();
    __syncthreads();
    issue<WHOLE>(4);
  }
  S1F_DEV void end_step() {
    const lds_addr s0 = st[0];
#pragma unroll
    for (int i = 0; i < 4; ++i) st[i] = st[i + 1];
    st[4] = s0;
  }
};

// How far a wave of the forward and dQ kernels walks: to the last tile that one of its rows sees, and in that tile only
// the column blocks (16 rows) that see it take part in the second product.  The tiles of a workgroup reach further for its
// other waves; walked all the same, with probabilities of zero, they would cost products, and an infinity or NaN in a key
// that the rows do not see would reach them as 0 * inf.  So a row is touched by the keys of the tile in which its block
// ends and by none behind it.
// rows [row0, row_end) of the segment, row r seeing the keys up to seg_off + r, counted like the n_kt tiles at hand
template <int BN> S1F_DEV int own_tiles(int seg_off, int row0, int row_end, int n_kt) {
  const int n = row_end > row0 ? (seg_off + row_end - 1) / BN + 1 : n_kt;
  return n < n_kt ? n : n_kt;
}
// column blocks, from the first on, that tile n_own - 1 is wholly hidden from; first: last key that the wave's first row sees
template <int BN> S1F_DEV int hidden_blocks(int first, int n_own) {
  const int past = BN * (n_own - 1) - first;
  return past > 0 ? past / 16 : 0;
}

}  // namespace s1f

// Matrix building blocks of the attention kernels (gfx950): 16x16 matrix instructions, 32-row operand tiles in LDS.
//
// Vocabulary:
//   lane      16*j + n with j in 0..3, n in 0..15
//   block     a 16x16 fp32 result held as 4 registers per lane: register v of lane (n, j) is element (row 4*j + v,
//             column n).  Kernels work on 32x32 scores as 2x2 blocks [rb][cb].
//   operand   what one lane feeds to one matrix instruction: A row n or B column n, and of the contraction index
//             the 8 elements 8*j .. 8*j+7 (fp32: of three planes, see split3)
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

// A [32 x D] tile of bf16 in LDS, in pieces of 1 KiB: piece (rh, kq) = rows 16*rh .. +15, bytes 64*kq .. +63 of the rows, i.e.
// exactly the A operand of rows 16*rh for contraction step kq.  Inside a piece chunk c (16 bytes) of row r lies in slot
// 4*r + (c ^ f(r)), f(r) = -(r / 4) mod 4.  Neither access pattern below has bank conflicts (the 16 lanes that a 128-bit read
// serves together, 0-3 with 12-15, 20-23 and 24-27 and so on, and the 32 of a 64-bit one cover all 64 banks), and the
// piece enters every address as a constant: one address register per pattern, where rows stored whole and swizzled took a
// vector instruction per operand.  Four consecutive slots hold 64 consecutive bytes of a row, which keeps the copies coalesced.
// An fp32 tile is three of them one behind the other, the planes of split3.
template <typename T, int D> struct Tile32 {
  static constexpr int CPR = D / 8;                  // 16-byte chunks per row
  static constexpr int NP = (CPR + 3) / 4;           // pieces per row half
  static constexpr int PLANE = 2 * NP * 1024;
  static constexpr int BYTES = (sizeof(T) == 4 ? 3 : 1) * PLANE;
  static_assert(D % 8 == 0, "head_dim must be a whole number of 16-byte chunks");
  S1F_DEV static int f(int r) { return -(r >> 2) & 3; }
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
  static constexpr int PRODUCTS = 1;   // matrix instructions per product of two operands
  static constexpr float UP = 1.f;     // what operands are multiplied by (fp32: kUp)
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
  // the lane's share of the dot product of two rows, the first of which it has loaded
  S1F_DEV static float row_dot(const RowOp &x, const bf16_t *, const bf16_t *y_row, int j) {
    RowOp y;
    load_row(y, y_row, j);
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
  S1F_DEV static Slab slab_up(f32x4 x, f32x4 y) { return slab(x, y); }
  S1F_DEV static void settle_slab(Slab &s) { settle(s); }
  S1F_DEV static void mma_tr(int t, Frag a, const Slab &s, f32x4 (&acc)[DB]) { acc[t] = mma16(a, s, acc[t]); }
  S1F_DEV static int quad_d0(int q, int j) { return 16 * q + 4 * j; }
  S1F_DEV static f32x4 quad(const f32x4 (&acc)[DB], int q) { return acc[q]; }
};

// fp32 operands as three bf16 planes: x = p[0] + p[1] + p[2] exactly (from 2^-110 on; see kUp), each what remains, rounded to nearest.  The
// planes of a value that is not finite, or that rounds up past the largest float, have a NaN or an infinity among them, which
// every product with them turns into: attn_plain.hpp computes what has become of such rows.
// Why: the fp32 matrix instructions run at a sixteenth of the bf16 ones' rate (153 against 1353 TFLOP/s in large matrix
// products here); six bf16 products for each take less than half as long, and accumulate fewer times.  Six, because the
// first plane leaves at most 2^-8 |x| and the second at most 2^-17 |x|: what the three products left out contribute is at most
// 2^-24 (1 + 2^-9) of |a| |b|, the rounding of one fp32 product, and of either sign.  (With a first plane cut off instead of rounded it
// is 2^-22, and of one sign where operands fill their bits: scores of operands just below 1 + 2^-7 were 1.9e-7 off on average.)  Relative error against 64 bits, 8/2 heads, 500 rows behind 3000 keys, head_dim 128
// (fp32 instructions / this): out 6.5e-7 / 4.3e-7, lse 5.60e-8 / 5.57e-8, dq 9.4e-7 / 8.3e-7, dk and dv 2.3e-6 / 2.0e-6; with
// queries 30 times as large 3.4e-6 / 2.5e-6, 1.7e-7 / 1.3e-7, 1.2e-5 / 0.9e-5, 2.8e-5 / 2.4e-5.  32 heads, 2048 rows behind 8000
// keys, us: head_dim 128 forward 2449 -> 1422, dQ 3500 -> 1909, dK/dV 4967 -> 2638; 80 1622 -> 1030, 2329 -> 1401, 3233 -> 1977; 64
// 1289 -> 700, 1885 -> 968, 2253 -> 1260: bound, like bf16, by the matrix pipe under the power limit (56-64 % busy at
// 2.0-2.2 GHz: 1230, 1360 and 1280 TFLOP/s executed, six products for each, at head_dim 128, 1320, 1440 and 1450 at 64).
struct Planes {
  bf16x8 p[3];
};
// Operands are split 2^16 times as large as they are (score gradients, which come out of a product of two such operands, as they
// come: 2^32 times), and accumulators divided in the end.  The last plane of a value below 2^-110 would lie under the smallest
// bf16 number: values of 2^-120 alone gave results 3.5e-5 off, of 2^-125 1e-3.  Nothing changes for the others, up to what then no
// longer has planes (operands and outputs from 2^112 on, scores and dV from 2^96, dQ and dK from 2^80: see attn_plain.hpp).  Not the
// forward's probabilities, of which a row has one of at least 1: the bits of 2^-134 that those below 2^-110 lose are nothing beside
// it.  Costs up to one vector instruction per operand element, 2 % of the forward at head_dim 64 and less elsewhere.
constexpr float kUp = 65536.f;
// two rounded values as one register; what is left of them
S1F_DEV uint32_t round_pair(float &x, float &y) {
  uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x, y}), bf16x2));
  asm("" : "+v"(w));   // (one conversion for both, which the compiler does anew for each to subtract it: f32 step of 8/2 heads 1078 -> 1043 us)
  x -= __builtin_bit_cast(float, w << 16);
  y -= __builtin_bit_cast(float, w & 0xffff0000u);
  return w;
}
S1F_DEV Planes split3(f32x4 lo, f32x4 hi) {
  u32x4 v[3];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float x = e < 2 ? lo[2 * e] : hi[2 * e - 4], y = e < 2 ? lo[2 * e + 1] : hi[2 * e - 3];
#pragma unroll
    for (int p = 0; p < 3; ++p) v[p][e] = round_pair(x, y);
  }
  return Planes{{__builtin_bit_cast(bf16x8, v[0]), __builtin_bit_cast(bf16x8, v[1]), __builtin_bit_cast(bf16x8, v[2])}};
}
S1F_DEV void settle(Planes &x) { asm volatile("" : "+v"(x.p[0]), "+v"(x.p[1]), "+v"(x.p[2])); }
// Product of two fp32 operands: the six products of planes that fp32 resolves (see Planes), smallest first.
S1F_DEV f32x4 mma16(const Planes &a, const Planes &b, f32x4 c) {
  c = mma16(a.p[2], b.p[0], c);
  c = mma16(a.p[0], b.p[2], c);
  c = mma16(a.p[1], b.p[1], c);
  c = mma16(a.p[1], b.p[0], c);
  c = mma16(a.p[0], b.p[1], c);
  return mma16(a.p[0], b.p[0], c);
}

// End of a scheduling slot of M's products: nothing moves across it.  In fp32 a slot holds the six matrix instructions of each of
// its products; they are spread over its vector instructions (a wave issues in order: one behind the other, each waits for
// the one before it and nothing runs beside them).
template <typename M> S1F_DEV void end_slot() {
  if constexpr (M::PRODUCTS > 1) {
#pragma unroll
    for (int i = 0; i < M::PRODUCTS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);   // a matrix instruction
      __builtin_amdgcn_sched_group_barrier(0x2, 6, 0);   // vector ones
    }
  }
  __builtin_amdgcn_sched_barrier(0);
}

template <int D> struct Mat<float, D> {
  static constexpr int PRODUCTS = 6;
  static constexpr float UP = kUp;
  typedef Mat<bf16_t, D> B;
  typedef Tile32<float, D> TL;
  typedef Planes Frag;
  typedef Planes Slab;
  typedef typename B::Nat Nat;
  typedef typename B::Tr Tr;
  static constexpr int NK = B::NK, NKS = B::NKS, NN = B::NN, NT = B::NT, DB = B::DB;
  struct RowOp {
    Frag f[NK];
  };
  B b;
  S1F_DEV void init(int lane) { b.init(lane); }
  S1F_DEV Nat nat_at(lds_addr tile) const { return b.nat_at(tile); }
  S1F_DEV Tr tr_at(lds_addr tile) const { return b.tr_at(tile); }
  S1F_DEV static Frag nat(const Nat &x, int i, unsigned delta = 0) {
    return Frag{{B::nat(x, i, delta), B::nat(x, i, delta + TL::PLANE), B::nat(x, i, delta + 2 * TL::PLANE)}};
  }
  S1F_DEV static Frag tr(const Tr &x, int t, unsigned delta = 0) {
    return Frag{{B::tr(x, t, delta), B::tr(x, t, delta + TL::PLANE), B::tr(x, t, delta + 2 * TL::PLANE)}};
  }
  S1F_DEV static void load_row(RowOp &o, const float *row, int j) {
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const f32x4 *at = reinterpret_cast<const f32x4 *>(row + 32 * k + (k < NKS ? 8 : 4) * j);
      o.f[k] = split3(at[0] * kUp, k < NKS ? at[1] * kUp : f32x4{0.f, 0.f, 0.f, 0.f});
    }
  }
  // (from the values themselves: those that have no planes count as well)
  S1F_DEV static float row_dot(const RowOp &, const float *x_row, const float *y_row, int j) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
      for (int h = 0; h < (k < NKS ? 2 : 1); ++h) {
        const int at = 32 * k + (k < NKS ? 8 : 4) * j + 4 * h;
        const f32x4 x = *reinterpret_cast<const f32x4 *>(x_row + at), y = *reinterpret_cast<const f32x4 *>(y_row + at);
#pragma unroll
        for (int e = 0; e < 4; ++e) s += x[e] * y[e];
      }
    return s;
  }
  S1F_DEV static f32x4 mma_nat(int i, const Frag &a, const RowOp &o, f32x4 c) { return mma16(a, o.f[i % NK], c); }
  S1F_DEV static f32x4 mma_op(int, const Frag &a, const Frag &b, f32x4 c) { return mma16(a, b, c); }
  S1F_DEV static Slab slab(f32x4 x, f32x4 y) { return split3(x, y); }
  S1F_DEV static Slab slab_up(f32x4 x, f32x4 y) { return split3(x * kUp, y * kUp); }
  S1F_DEV static void settle_slab(Slab &s) { settle(s); }
  S1F_DEV static void mma_tr(int t, const Frag &a, const Slab &s, f32x4 (&acc)[DB]) { acc[t] = mma16(a, s, acc[t]); }
  S1F_DEV static int quad_d0(int q, int j) { return B::quad_d0(q, j); }
  S1F_DEV static f32x4 quad(const f32x4 (&acc)[DB], int q) { return acc[q]; }
};

// Asynchronous copy of two Tile32s (the second right behind the first) from global memory by the four waves of a
// workgroup: wave w copies rows 16*(w & 1).. of tile w / 2.  One global_load_lds_dwordx4 moves 16 bytes per lane into
// 1 KiB of consecutive LDS, i.e. fills one piece: lane l lands at M0 + immediate offset + 16*l, and the immediate offset
// is added to the global address as well.  Up to four of a wave's NP pieces share one value of M0 (rewriting M0 between
// copies makes them complete one after the other instead of overlapping).  Written as assembly so that the compiler's
// wait-count pass does not tie LDS reads of OTHER ring stages to these copies; callers order the copies against their
// readers with wait_async_tiles() + a workgroup barrier.
// The address is (scalar base of the piece) + (32-bit lane offset fixed at init).  The pieces of a row half differ by
// 64 bytes in the scalar base and share the lane offset, except that the last piece of head_dim 80, half of it past the
// row's end, has its own (those slots re-read a valid chunk and are never used).  Rows past the last valid one re-read it
// (callers mask them).
template <typename T, int D> struct TilePairCopy {
  static_assert(sizeof(T) == 2, "fp32 tiles: SplitPairCopy");
  typedef Tile32<T, D> TL;
  static constexpr int NP = TL::NP;
  static constexpr bool PARTIAL = TL::CPR % 4 != 0;
  static constexpr int NV = PARTIAL ? 2 : 1;
  unsigned voff[NV];

  S1F_DEV static constexpr int vclass(int kq) { return (PARTIAL && kq == NP - 1) ? 1 : 0; }
  S1F_DEV static int slot_row(int wave, int lane) { return 16 * (wave & 1) + (lane >> 2); }
  S1F_DEV void init(int wave, int lane, int64_t row_stride) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int r = slot_row(wave, lane);
      int c = (lane & 3) ^ TL::f(r & 15);   // chunk within the piece
      if (v == 1 && c >= TL::CPR % 4) c -= 2;
      voff[v] = (unsigned)((r * row_stride + c * 8) * (int64_t)sizeof(T));
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
        const int over = slot_row(wave, lane_id()) - (rows_left - 1);
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

// The same for fp32 tensors, through registers (split once per workgroup, not by every wave that reads the operand): a lane loads the 8 elements of its slot in every piece, splits them and writes a
// chunk of each plane.  Between load() and write() the values travel in registers, so that a load has as long as the caller
// leaves it.
// WAVES: waves that share the work, 4 or 8 (then waves w and w + 4 take every other piece).
template <int D, int WAVES> struct SplitPairCopy {
  typedef Tile32<float, D> TL;
  static constexpr int STEP = WAVES / 4, NP = TL::NP, NI = (NP + STEP - 1) / STEP;
  static constexpr bool PARTIAL = TL::CPR % 4 != 0;
  f32x4 held[NI][2];
  unsigned dst;   // within the pair of tiles
  int row, chunk, first;
  S1F_DEV void init(int wave8, int lane, int64_t) {
    const int wave = wave8 & 3;
    first = wave8 >> 2;
    row = 16 * (wave & 1) + (lane >> 2);
    chunk = (lane & 3) ^ TL::f(row & 15);
    dst = (unsigned)((wave >> 1) * TL::BYTES + (wave & 1) * NP * 1024 + 16 * lane);
  }
  S1F_DEV int piece(int i) const { return STEP == 1 ? i : STEP * i + first; }
  // where the lane's row lies
  S1F_DEV const float *at(const float *row0, const float *row1, int64_t row_stride, int left0, int left1, int wave8) const {
    const int wave = wave8 & 3, left = wave >= 2 ? left1 : left0, r = row < left ? row : left - 1;
    return (wave >= 2 ? row1 : row0) + r * row_stride;
  }
  S1F_DEV void load(const float *lane_row, int i) {
    const int kq = piece(i);
    if (STEP * i + STEP > NP && kq >= NP) return;
    const int c = PARTIAL && kq == NP - 1 ? chunk & 1 : chunk;   // (of the last piece of head_dim 80 only half is ever read)
    held[i][0] = *reinterpret_cast<const f32x4 *>(lane_row + 32 * kq + 8 * c);
    held[i][1] = *reinterpret_cast<const f32x4 *>(lane_row + 32 * kq + 8 * c + 4);
  }
  S1F_DEV void load(const float *row0, const float *row1, int64_t row_stride, int left0, int left1, int wave8) {
    const float *lane_row = at(row0, row1, row_stride, left0, left1, wave8);
#pragma unroll
    for (int i = 0; i < NI; ++i) load(lane_row, i);
  }
  S1F_DEV void write(int i, lds_addr stage) const {
    write_half(i, 0, stage);
    write_half(i, 1, stage);
  }
  // half h of piece i: four of the eight elements
  S1F_DEV void write_half(int i, int h, lds_addr stage) const {
    const int kq = piece(i);
    if (STEP * i + STEP > NP && kq >= NP) return;
    const f32x4 none = {0.f, 0.f, 0.f, 0.f};
    const Planes x = split3(held[i][h] * kUp, none);
    const lds_addr at = opaque(stage + dst + (unsigned)(kq * 1024 + 8 * h));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const u32x4 v = __builtin_bit_cast(u32x4, x.p[p]);
      *reinterpret_cast<__attribute__((address_space(3))) u32x2 *>((uintptr_t)(at + (unsigned)(p * TL::PLANE))) = u32x2{v[0], v[1]};
    }
  }
};

// Ring of five stages of one K and one V tile each, shared by the forward and the dQ kernel.  Step k computes on tiles
// k and k+1 and reads the first operands of tile k+2; tile k+4 is copied into the stage of tile k-1 meanwhile.  A copy
// therefore has two steps to land: a launch that leaves one workgroup per compute unit spends 0.4-0.5 us on a step, less
// than memory takes to answer.  With one step, 64 heads of 256 rows behind 16384 keys (forward, head_dim 128, 64-row
// units) took 359 us, with two 237.
template <typename T, int D, int WAVES = 4> struct TileRing {
  static_assert(WAVES == 4, "four waves copy a pair of tiles");
  static constexpr bool AHEAD = true;   // a step may read the first operands of the next one
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
  template <bool WHOLE> S1F_DEV void work(int, int) {}
  S1F_DEV void end_step() {
    const lds_addr s0 = st[0];
#pragma unroll
    for (int i = 0; i < 4; ++i) st[i] = st[i + 1];
    st[4] = s0;
  }
};

// The ring of fp32 tiles: three stages, all that LDS holds of three planes at head_dim 128.  Step k computes on tiles k and k+1; meanwhile
// tile k+2, loaded during step k-1, is split and written into the stage of tile k-1, and tile k+3 is loaded.
template <int D, int WAVES> struct TileRing<float, D, WAVES> {
  static constexpr bool AHEAD = false;
  static constexpr int STAGE_BYTES = 2 * Tile32<float, D>::BYTES;
  static constexpr int LDS_BYTES = 3 * STAGE_BYTES;
  typedef SplitPairCopy<D, WAVES> Copy;
  Copy ld;
  const float *k_next, *v_next;
  int64_t row_stride;
  int to_load, rows_left;
  bool held;                     // a tile is in registers
  lds_addr st[3];                // stages of tiles k, k+1 and k+2 (= k-1)
  int wave;
  S1F_DEV void init(const float *k, const float *v, int64_t row_stride_, int tiles, int rows, lds_addr lds, int wave_, int lane) {
    ld.init(wave_, lane, row_stride_);
    k_next = k; v_next = v;
    row_stride = row_stride_;
    to_load = tiles; rows_left = rows;
#pragma unroll
    for (int i = 0; i < 3; ++i) st[i] = lds + (unsigned)(i * STAGE_BYTES);
    wave = wave_;
    held = false;
  }
  S1F_DEV void load() {
    held = to_load > 0;
    if (!held) return;
    ld.load(k_next, v_next, row_stride, rows_left, rows_left, wave);
    --to_load;
    rows_left -= 32;
    k_next += 32 * row_stride;
    v_next += 32 * row_stride;
  }
  S1F_DEV void write(int i) {
    if (!held) return;
#pragma unroll
    for (int x = 0; x < Copy::NI; ++x) ld.write(x, st[i]);
  }
  // Before the first step: tiles 0 and 1 into their stages, tile 2 into registers.  Tiles 0 and 1 are both loaded before either
  // is written, and the caller loads its own rows in between: one wait for memory instead of three (8/8 heads, head_dim 80, 947 rows
  // behind 4053 keys, backward 232 -> 228 us; 32/8 heads, 64, 1675 behind 6325 1477 -> 1436, forward 488 -> 479; the
  // same in the dK/dV kernel is part of that).  Four waves above head_dim 64 have no registers for two tiles next to their rows (backward of
  // 8/2 heads, 128, 941 behind 2300: 253 -> 261).
  static constexpr bool TWO = WAVES == 8 || D == 64;
  Copy ld0;
  S1F_DEV void issue(int i) {
    if (i > 2) return;
    if constexpr (TWO) {
      if (i == 2) {
#pragma unroll
        for (int x = 0; x < Copy::NI; ++x) ld0.write(x, st[0]);   // (there always is a first tile)
        write(1);
      }
      load();
      if (i == 0) ld0 = ld;
    } else {
      load();
      if (i < 2) write(i);
    }
  }
  // WHOLE: a whole tile is in registers and another is left to load; both then happen piece by piece in work()
  template <bool WHOLE> S1F_DEV void begin_step(int) {
    __syncthreads();
    if constexpr (WHOLE) {
      lane_row = ld.at(k_next, v_next, row_stride, 32, 32, wave);
      --to_load;
      rows_left -= 32;
      k_next += 32 * row_stride;
      v_next += 32 * row_stride;
    } else {
      write(2);
      load();
    }
  }
  const float *lane_row;
  // Share `slot` of `slots` of a step's splitting, under the matrix instructions of one operand
  static constexpr int HALVES = 2 * Copy::NI;
  template <bool WHOLE> S1F_DEV void work(int slot, int slots) {
    if constexpr (WHOLE) {
#pragma unroll
      for (int x = HALVES * slot / slots; x < HALVES * (slot + 1) / slots; ++x) {
        ld.write_half(x >> 1, x & 1, st[2]);
        if (x & 1) ld.load(lane_row, x >> 1);
      }
    }
  }
  S1F_DEV void end_step() {
    const lds_addr s0 = st[0];
    st[0] = st[1];
    st[1] = st[2];
    st[2] = s0;
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

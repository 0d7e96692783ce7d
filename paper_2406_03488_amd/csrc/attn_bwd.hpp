// Backward of one segment (derivative of Section 3.1, Eq. 3; accumulation per Section 3.2):
//   p_ij = exp(s_ij - lse_i),  delta_i = dO_i . O_i,  dp_ij = dO_i . v_j,  ds_ij = p_ij (dp_ij - delta_i)
//   dq_i = scale * sum_j ds_ij k_j      dk_j += scale * sum_i ds_ij q_i      dv_j += sum_i p_ij dO_i
//
// Two bodies, neither uses atomics:
//   bwd_dq_body    owns query rows (same decomposition as the forward), loops over key tiles, and, by itself, first computes
//                  the row statistics of the other;
//   bwd_dkdv_body  owns key rows, loops over the query heads of its K/V group and over the
//                  segment's query tiles, and adds its result into the fp32 prefix accumulators
//                  (each accumulator element is touched by exactly one lane of one workgroup).
// The probabilities are recomputed in both (7 matrix products in total instead of 5) in exchange for
// deterministic sums and no dQ workspace.  seg_attn_bwd_dq_kernel and
// seg_attn_bwd_dkdv_kernel run one of them; seg_attn_bwd_kernel runs the units of both in one launch, behind
// seg_attn_bwd_stats_kernel, which then computes the row statistics.
#pragma once
#include <type_traits>

#include "attn_plain.hpp"

namespace s1f {

// Row statistics of 16 rows, one per lane in row order: lane (n, j) returns -lse and -delta = -rowsum(dO * O) of row n and,
// with `write`, leaves -lse/scale and -delta in the two planes of the workspace.  dor: the rows of dO
template <typename T, int D>
S1F_DEV void bwd_row_stats(const AttnArgs &a, const typename Mat<T, D>::RowOp &dor, int64_t off, int64_t at, bool write, int j, float &nlse,
                           float &nd) {
  nd = -sum_over_rows(Mat<T, D>::row_dot(dor, reinterpret_cast<const T *>(a.dout) + off, reinterpret_cast<const T *>(a.out) + off, j));
  const float lse = a.lse[at];
  nlse = -lse;
  if (write && j == 0) {
    a.delta[at] = -lse / a.scale;
    a.delta[a.ws_plane + at] = nd;
  }
}
// ... of all rows, for halves of the backward that run in one launch: a wave per 16 rows of one (batch, head).  The same sums as
// in the dQ kernel's own prologue.  Bound by its launch (4 to 5 us of small calls) or by memory (67 MB of out and dout: 15 us).
template <typename T, int D> __global__ void __launch_bounds__(256) seg_attn_bwd_stats_kernel(const AttnArgs a) {
  typedef Mat<T, D> M;
  int bh, group64;
  div_mod(blockIdx.x, a.by_groups, bh, group64);
  const int lane = threadIdx.x & 63, j = lane >> 4;
  const int r = group64 * 64 + ((int)threadIdx.x >> 6) * 16 + (lane & 15), rc = r < a.seg_len ? r : a.seg_len - 1;
  int b, h;
  div_mod(bh, a.by_heads, b, h);
  const int64_t off = b * a.q_sb + h * a.q_sh + (int64_t)rc * a.q_ss;
  typename M::RowOp dor;
  M::load_row(dor, reinterpret_cast<const T *>(a.dout) + off, j);
  float nlse, nd;
  bwd_row_stats<T, D>(a, dor, off, (int64_t)bh * a.seg_len + rc, r < a.seg_len, j, nlse, nd);
}

// One workgroup (4 waves) owns 64*NC query rows of one head, a wave NC column blocks of 16; lane = one query per column
// block, keys run over registers.
//   S^T[key][q]  = K Q^T      A = K (LDS),            B = Q (registers)
//   dP^T[key][q] = V dO^T     A = V (LDS),            B = dO (registers)
//   dQ^T[d][q]  += K^T dS^T   A = K read transposed,  B = dS^T slab (registers)
// The accumulators of dP start from -delta (the same in every register of a lane), so that dS = p * dp.
// K/V tiles of 32 keys travel through a ring as in the forward, with one barrier per tile.  The loop is
// software-pipelined so that every phase has matrix instructions that do not wait for its vector work:
//   A  S(k+1)                ||  dS(k) = p(k) * dP(k), packed
//   B  dQ += K(k)^T dS(k)    ||  p(k+1) = exp2(c * S(k+1) - lse)
//   C  dP(k+1)
// The order is pinned matrix instruction by matrix instruction; LDS operands are read kDqRing operands ahead.
// Bound by the matrix pipe at the clock the power limit leaves (head_dim 128: 71-77 % busy at 1.73-1.78 GHz), with 64 registers
// of accumulators and 64 of Q and dO per lane at NC = 2.  32 heads, 4096 rows behind 28672 keys: head_dim 128
// 2.52 -> 2.29 ms (three products executed: 1230 -> 1350 TFLOP/s), 80 1.89 -> 1.57 ms and 64 1.54 -> 1.26 ms (NC = 3).
// One wave per SIMD with 64 rows (half the LDS reads) ran 15 % slower: half of its registers are accumulator
// registers, which the vector phases reach by copies only.
template <typename T, int D> constexpr int kDqRing = sizeof(T) == 2 ? 4 : D == 64 ? 2 : 3;   // (fp32: three registers for one)

// id: number of the workgroup among those of this half; smem: TileRing::LDS_BYTES
// STATS: computes the row statistics and leaves them for the dK/dV half, instead of reading them
// PAIR: a workgroup has one of the two tiles of a chunk of a unit of a.bm = 2 * BM rows: the same sums as in one tile of a.bm
template <typename T, int D, int NC, int WAVES, bool STATS, bool PAIR = false> S1F_DEV void bwd_dq_body(const AttnArgs &a, int id, char *smem) {
  typedef Mat<T, D> M;
  typedef typename M::Frag Frag;
  typedef TileRing<T, D, WAVES> Ring;
  constexpr int DB = M::DB, BM = 16 * NC * WAVES, BN = 32, NN = M::NN, NK = M::NK, NT = M::NT, PR = kDqRing<T, D>;
  constexpr int TOTAL = NN + NT + NN;
  static_assert(NN >= PR && NT >= PR, "operand ring deeper than a product");

  const int tid = threadIdx.x, lane = tid & 63, j = lane >> 4, n = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  UnitChunk uc = split_unit(id, a.n_whole, PAIR ? 2 * a.n_split : a.n_split, a.n_split_units, a.by_split_units);
  int second = 0;
  if (PAIR) {   // (no unit is whole)
    second = uc.chunk & 1;
    uc = UnitChunk{uc.unit, uc.chunk >> 1, a.n_split, (uc.chunk >> 1) * a.n_split_units + uc.unit};
  }
  int qt, bh;
  decode_workgroup(uc.unit, a.by_tiles, a.n_bh, a.by_xcd, a.tile_major, qt, bh);
  qt = a.n_tiles - 1 - qt;   // later (heavier) row tiles are scheduled first
  int b, h;
  div_mod(bh, a.by_heads, b, h);
  const int hk = div(h, a.by_group);
  const int seg_len = a.seg_len;
  const int unit_row0 = qt * (PAIR ? 2 * BM : BM), row0 = unit_row0 + second * BM, wrow0 = row0 + wave * 16 * NC;
  if (PAIR && row0 >= seg_len) return;
  const int last_row = (row0 + BM < seg_len ? row0 + BM : seg_len) - 1;
  // This workgroup's key tiles: all that hold keys 0 .. seg_off+last_row, or one chunk of them.  From here on keys
  // are counted from the chunk's first key: seg_off and kv_len are relative to it.
  int kt0, kt1;
  chunk_range(uc, a.by_split, (a.seg_off + unit_row0) / BN, (a.seg_off + last_row) / BN + 1, kt0, kt1);
  const int seg_off = a.seg_off - BN * kt0, kv_len = seg_off + seg_len;
  const int n_kt = kt1 - kt0;
  const int64_t part_at = ((int64_t)uc.slot * (PAIR ? 2 : 1) + second) * (BM * D);   // of a chunk's tile

  const int64_t qoff = b * a.q_sb + h * a.q_sh;
  const int64_t kv_first = b * a.kv_sb + hk * a.kv_sh + (int64_t)(BN * kt0) * a.kv_ss;
  Ring ring;
  ring.init(reinterpret_cast<const T *>(a.k) + kv_first, reinterpret_cast<const T *>(a.v) + kv_first, a.kv_ss, n_kt, kv_len,
            to_lds_addr(smem), wave, lane);
  ring.issue(0);
  ring.issue(1);

  auto row_stats = [&](const typename M::RowOp &dor, int64_t off, int64_t at, bool write, int j, float &nlse, float &d) {
    if constexpr (STATS) {
      bwd_row_stats<T, D>(a, dor, off, at, write, j, nlse, d);
    } else {
      nlse = -a.lse[at];
      d = a.delta[a.ws_plane + at];
    }
  };
  typename M::RowOp q[NC], dor[NC];
  float nl[NC];    // -lse in log2 units
  f32x4 nd[NC];    // -delta
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    const int r = wrow0 + 16 * cb + n, rc = r < seg_len ? r : seg_len - 1;
    const int64_t off = qoff + (int64_t)rc * a.q_ss;
    M::load_row(q[cb], reinterpret_cast<const T *>(a.q) + off, j);
    M::load_row(dor[cb], reinterpret_cast<const T *>(a.dout) + off, j);
    const int64_t at = ((int64_t)b * a.n_q_heads + h) * seg_len + rc;
    float nlse, d;
    row_stats(dor[cb], off, at, r < seg_len && uc.chunk == 0, j, nlse, d);
    d *= M::UP * M::UP;
    nd[cb] = f32x4{d, d, d, d};
    nl[cb] = nlse * kLog2e;
  }
  f32x4 dq[NC][DB];
#pragma unroll
  for (int cb = 0; cb < NC; ++cb)
#pragma unroll
    for (int db = 0; db < DB; ++db) dq[cb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c = uniform(a.scale * kLog2e / (M::UP * M::UP));
  M rd;
  rd.init(lane);
#pragma unroll
  for (int cb = 0; cb < NC; ++cb)
#pragma unroll
    for (int i = 0; i < M::NK; ++i) { settle(q[cb].f[i]); settle(dor[cb].f[i]); }

  if (n_kt <= 0) {   // more chunks than this unit has whole tiles: nothing to add
    float *pd = a.part + part_at;
    for (int i = tid; i < BM * D; i += 64 * WAVES) pd[i] = 0.f;
    return;
  }
  wait_async_tiles();
  ring.issue(2);
  ring.issue(3);
  __syncthreads();
  int k = 0;   // current tile
  if (wrow0 >= seg_len) {   // no rows of its own: the wave only copies its share of the tiles
    for (; k + 1 < n_kt; ++k, ring.end_step()) ring.template begin_step<false>(n_kt - 1 - k);
    return;
  }
  const int wfirst = seg_off + wrow0;   // last key that the wave's first row sees
  // Hidden scores of a tile on the diagonal get probability zero (whatever the exponential made of them).
  auto hide = [&](f32x4 (&p)[2][NC], int key0) {
    const int ln = lane_id(), lim = wfirst - key0 + (ln & 15) - 4 * (ln >> 4);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int cb = 0; cb < NC; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (16 * rb + v > lim + 16 * cb) p[rb][cb][v] = 0.f;
  };

  // Tile 0: S, p and dP by themselves.
  f32x4 p[2][NC], dp[2][NC];
  {
    const typename M::Nat ka = rd.nat_at(ring.st[0]);
#pragma unroll
    for (int i = 0; i < NN; ++i) {
      const Frag kf = M::nat(ka, i), vf = M::nat(ka, i, Tile32<T, D>::BYTES);
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        p[i / NK][cb] = M::mma_nat(i, kf, q[cb], i % NK ? p[i / NK][cb] : zero);
        dp[i / NK][cb] = M::mma_nat(i, vf, dor[cb], i % NK ? dp[i / NK][cb] : nd[cb]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int cb = 0; cb < NC; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v) p[rb][cb][v] = exp2_fast(fmaf(p[rb][cb][v], c, nl[cb]));
    if (BN - 1 > wfirst) hide(p, 0);
  }
  Frag fr[PR];   // operand ring: operand x of a step sits in fr[x % PR]
  auto first_operands = [&]() {
    const typename M::Nat ka = rd.nat_at(ring.st[1]);
#pragma unroll
    for (int i = 0; i < PR; ++i) fr[i] = M::nat(ka, i);
  };
  if (Ring::AHEAD) first_operands();
  typename M::Slab ds[NC];
  auto make_ds = [&](int cb) {
    ds[cb] = M::slab(p[0][cb] * dp[0][cb], p[1][cb] * dp[1][cb]);
    M::settle_slab(ds[cb]);
  };
  auto step = [&](auto mask, auto whole) {
    constexpr bool MASK = decltype(mask)::value, WHOLE = decltype(whole)::value;
    ring.template begin_step<WHOLE>(n_kt - 1 - k);
    if (!Ring::AHEAD) first_operands();
    const typename M::Nat kn = rd.nat_at(ring.st[1]), ka = rd.nat_at(ring.st[2]);
    const typename M::Tr kt = rd.tr_at(ring.st[0]);
    auto next_operand = [&](int x) {   // operand x has been used up: the one that takes its place
      const int y = x + PR;
      if (y < NN) fr[x % PR] = M::nat(kn, y);
      else if (y < NN + NT) fr[x % PR] = M::tr(kt, y - NN);
      else if (y < TOTAL) fr[x % PR] = M::nat(kn, y - NN - NT, Tile32<T, D>::BYTES);
      else if (Ring::AHEAD) fr[x % PR] = M::nat(ka, x % PR);   // the next step's first ones
    };
    if (D != 80) __builtin_amdgcn_s_setprio(1);   // phase A first: of two ready waves the one with little else to issue
    f32x4 sn[2][NC];
#pragma unroll
    for (int i = 0; i < NN; ++i)
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        sn[i / NK][cb] = M::mma_nat(i, fr[i % PR], q[cb], i % NK ? sn[i / NK][cb] : zero);
        if (cb + 1 == NC) next_operand(i);
        if (i == 1) make_ds(cb);
        ring.template work<WHOLE>(i * NC + cb, TOTAL * NC);
        end_slot<M>();
      }
    if (D != 80) __builtin_amdgcn_s_setprio(0);
    // probability x of 8 * NC: column block by column block, so that half of them do not wait for the last scores
    auto probs = [&](int x0, int x1) {
#pragma unroll
      for (int x = x0; x < x1; ++x) {
        const int rb = x / (4 * NC), cb = (x >> 2) % NC, v = x & 3;
        float y = exp2_fast(fmaf(sn[rb][cb][v], c, nl[cb]));
        settle(y);
        p[rb][cb][v] = y;
      }
    };
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        M::mma_tr(i, fr[(NN + i) % PR], ds[cb], dq[cb]);
        if (cb + 1 == NC) next_operand(NN + i);
        const int w = i * NC + cb, W = NT * NC;
        probs(8 * NC * w / W, 8 * NC * (w + 1) / W);
        ring.template work<WHOLE>(NN * NC + w, TOTAL * NC);
        end_slot<M>();
      }
#pragma unroll
    for (int i = 0; i < NN; ++i)
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        dp[i / NK][cb] = M::mma_nat(i, fr[(NN + NT + i) % PR], dor[cb], i % NK ? dp[i / NK][cb] : nd[cb]);
        if (cb + 1 == NC) next_operand(NN + NT + i);
        if (MASK && i == 0 && cb + 1 == NC) hide(p, BN * (k + 1));
        ring.template work<WHOLE>((NN + NT + i) * NC + cb, TOTAL * NC);
        end_slot<M>();
      }
    ++k;
    ring.end_step();
  };
  const int n_own = own_tiles<BN>(seg_off, wrow0, wrow0 + 16 * NC < seg_len ? wrow0 + 16 * NC : seg_len, n_kt);
  int n_full = (wfirst + 1) / BN;   // tiles that every row of the wave sees in full
  n_full = n_full < n_kt - 1 ? n_full : n_kt - 1;
  const std::integral_constant<bool, true> yes;
  const std::integral_constant<bool, false> no;
  const int n_fast = n_full < n_kt - 4 ? n_full : n_kt - 4;   // ... while there is a whole tile to copy
  while (k + 1 < n_fast) step(no, yes);
  while (k + 1 < n_full) step(no, no);
  while (k + 1 < n_own) step(yes, no);
  // The wave's last tile: dS and dQ.  Waves that have more tiles to walk are let into their next step first.
  if (k + 1 < n_kt) ring.template begin_step<false>(n_kt - 1 - k);
  {
    const int hidden = hidden_blocks<BN>(wfirst, n_own);
    const typename M::Tr kt = rd.tr_at(ring.st[0]);
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) make_ds(cb);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const Frag kf = M::tr(kt, i);
#pragma unroll
      for (int cb = 0; cb < NC; ++cb)
        if (cb + 1 == NC || cb >= hidden) M::mma_tr(i, kf, ds[cb], dq[cb]);   // (the last block is never hidden)
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (k + 1 < n_kt) {   // its share of the others' tiles
    ring.end_step();
    for (++k; k + 1 < n_kt; ++k, ring.end_step()) ring.template begin_step<false>(n_kt - 1 - k);
  }

  if constexpr (sizeof(T) == 4) {
    float bad = 0.f;
#pragma unroll
    for (int cb = 0; cb < NC; ++cb)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        bad = add_if_not_finite(dq[cb][db], bad);
        dq[cb][db] *= 1.f / (M::UP * M::UP * M::UP);
      }
    if (__builtin_expect(any_not_finite(bad), 0)) {
      const T *k0 = reinterpret_cast<const T *>(a.k) + kv_first, *v0 = reinterpret_cast<const T *>(a.v) + kv_first;
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        const int r_last = wrow0 + 16 * cb + 15, last = seg_off + (r_last < seg_len ? r_last : seg_len - 1);
        const int pl = lane_id(), r = wrow0 + 16 * cb + (pl & 15), rc = r < seg_len ? r : seg_len - 1;
        const int64_t off = qoff + (int64_t)rc * a.q_ss;
        float nlse, d;   // (anew: not kept in registers across the loop)
        row_stats(dor[cb], off, ((int64_t)b * a.n_q_heads + h) * seg_len + rc, false, pl >> 4, nlse, d);
        dq_plain<D>(reinterpret_cast<const T *>(a.q) + off, reinterpret_cast<const T *>(a.dout) + off, k0, v0, a.kv_ss, seg_off + rc,
                    last < BN * n_kt ? last + 1 : BN * n_kt, c * (M::UP * M::UP), nlse * kLog2e, d, pl >> 4, dq[cb]);
      }
    }
  }
  if (uc.slot >= 0) {   // a chunk: its unscaled share of the unit's dQ rows goes to the workspace
    float *pd = a.part + part_at;
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      const int rl = wave * 16 * NC + 16 * cb + n;   // row within the tile
#pragma unroll
      for (int x = 0; x < DB; ++x) *reinterpret_cast<f32x4 *>(pd + rl * D + M::quad_d0(x, j)) = M::quad(dq[cb], x);
    }
    return;
  }
  T *dqb = reinterpret_cast<T *>(a.dq) + qoff;
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    const int r = wrow0 + 16 * cb + n;
    if (r < seg_len) {
      T *row = dqb + (int64_t)r * a.q_ss;
#pragma unroll
      for (int x = 0; x < DB; ++x) {
        const f32x4 y = M::quad(dq[cb], x) * a.scale;
        store4<T>(row + M::quad_d0(x, j), y[0], y[1], y[2], y[3]);
      }
    }
  }
}

// Sums the chunks of the units that were cut along the keys: dq = scale * sum_c part_c.
// Thread and grid layout as in seg_attn_fwd_merge_kernel.
template <typename T, int D, int MC> S1F_DEV void bwd_dq_merge_body(const AttnArgs &a, int id) {
  constexpr int C4 = D / 4, RG = 256 / C4;
  const int BM = a.bm;
  int unit, rg;
  div_mod(id, a.by_groups, unit, rg);
  const int rl = rg * RG + (int)threadIdx.x / C4, c4 = (int)threadIdx.x % C4;
  int qt, bh;
  decode_workgroup(a.n_whole + unit, a.by_tiles, a.n_bh, a.by_xcd, a.tile_major, qt, bh);
  qt = a.n_tiles - 1 - qt;
  int b, h;
  div_mod(bh, a.by_heads, b, h);
  const int r = qt * BM + rl, S = a.n_split;
  if ((int)threadIdx.x >= RG * C4 || rl >= BM || r >= a.seg_len) return;
  int slot0, slot_step;
  chunk_slots(unit, a.n_split_units, slot0, slot_step);
  const float *pd = a.part + (int64_t)slot0 * (BM * D) + rl * D + 4 * c4;
  f32x4 pc[MC];
#pragma unroll
  for (int c = 0; c < MC; ++c)   // past the last chunk: that one again, not added
    pc[c] = *reinterpret_cast<const f32x4 *>(pd + (int64_t)(c < S ? c : S - 1) * slot_step * (BM * D));
  f32x4 acc = pc[0];
#pragma unroll
  for (int c = 1; c < MC; ++c)
    if (c < S) acc += pc[c];
  T *dqb = reinterpret_cast<T *>(a.dq) + b * a.q_sb + h * a.q_sh;
  store4<T>(dqb + (int64_t)r * a.q_ss + 4 * c4, acc[0] * a.scale, acc[1] * a.scale, acc[2] * a.scale, acc[3] * a.scale);
}

template <typename T, int D> struct BwdDkdvCfg {
  static constexpr int BQ = 32;                        // rows per Q/dO tile
  static constexpr int BNW = 128;                      // keys per workgroup: 4 waves of 32, in fp32 above head_dim 64 8 waves of 16
  static constexpr int WAVES = sizeof(T) == 4 && D > 64 ? 8 : 4;
  static constexpr int CB = 8 / WAVES;                 // column blocks of 16 keys per wave
  typedef Tile32<T, D> TL;
  static constexpr int STAGES = sizeof(T) == 4 ? 1 : 2;   // (fp32: three planes of V and one stage are what LDS holds)
  static constexpr int STAGE_BYTES = 2 * TL::BYTES;    // Q tile, dO tile right behind it
  static constexpr int STAT_BYTES = 2 * BQ * 4;        // -lse/scale and -delta of the tile's rows
  static constexpr int V_BYTES = 4 * TL::BYTES;        // the workgroup's V rows
  static constexpr int LOOP_BYTES = STAGES * STAGE_BYTES + V_BYTES + 2 * STAT_BYTES;   // stages, V, statistics
  static constexpr int EPI_ROW = pow2_at_least(D * 4); // bytes per row of the epilogue's staging regions
  static constexpr int EPI_BYTES = BNW * EPI_ROW;
  static constexpr int LDS_BYTES = LOOP_BYTES > EPI_BYTES ? LOOP_BYTES : EPI_BYTES;
};

// dK/dV kernel.  A workgroup owns 128 keys of one K/V head, a wave 32 of them in two column blocks of 16; lane = one key
// per column block; queries run over registers.  Q/dO tiles of 32 rows and their row statistics travel through a
// two-stage LDS ring, copied HBM -> LDS asynchronously.  (fp32: one stage of planes, the next tile waiting in registers; above
// head_dim 64 eight waves of one column block each, two to a SIMD: 32 heads, 2048 rows behind 8000 keys, head_dim 128 3235 ->
// 2676 us, 80 2364 -> 1995; at 64, where two workgroups of four waves share a compute unit, 1359 -> 1511, hence four there.)
//   S[q][key]  = Q K^T         A = Q (LDS),              B = K (registers)
//   dP[q][key] = dO V^T        A = dO (LDS),             B = V (LDS)
//   dV^T[d][key] += dO^T P     A = dO read transposed,   B = P slab (registers)
//   dK^T[d][key] += Q^T dS     A = Q read transposed,    B = dS slab (registers)
// The wave's K rows, its dK and dV accumulators and the tile's S and dP fill the register budget of two waves per SIMD;
// its V rows are therefore read from LDS (copied there once).
// The accumulators of S and dP start from the row statistics instead of zero, so that s = q.k - lse/scale and
// dp = dO.v - delta come out of the matrix pipe ready for p = exp2(c*s) and dS = p*dp.
// Vector work runs under the matrix instructions of the next product: the exponentials under dP, dS under dV; the order
// is pinned matrix instruction by matrix instruction, LDS operands are read kDkdvRing operands ahead.  Two workgroups
// share a compute unit, with barriers of their own: one's prologue, epilogue and waits overlap the other's products.
// Bound by the matrix pipe at the clock the power limit leaves (head_dim 128: 62-68 % busy at 1.85-1.89 GHz).  32 heads, 4096
// rows behind 28672 keys: head_dim 128 3.70 -> 3.41 ms (1114 -> 1210 TFLOP/s), 80 2.80 -> 2.54 ms; head_dim 64 with
// three workgroups per compute unit 1.94 -> 1.74 ms (two: 1.89).  A ring of 6 operands measures the same, one of 8
// 12 % slower.
template <typename T> constexpr int kDkdvRing = sizeof(T) == 4 ? 3 : 4;   // (fp32: three registers for one)

// id: number of the workgroup among those of this half; smem: BwdDkdvCfg::LDS_BYTES
template <typename T, int D> S1F_DEV void bwd_dkdv_body(const AttnArgs &a, int id, char *smem) {
  typedef BwdDkdvCfg<T, D> Cfg;
  typedef Mat<T, D> M;
  typedef typename M::Frag Frag;
  typedef typename TileRing<T, D, Cfg::WAVES>::Copy Copy;
  constexpr bool ASYNC = Cfg::STAGES == 2;   // tiles are copied past the registers
  constexpr int DB = M::DB, BQ = Cfg::BQ, NN = M::NN, NK = M::NK, NT = M::NT, PR = kDkdvRing<T>, CB = Cfg::CB;
  constexpr int TB = Tile32<T, D>::BYTES, X1 = NN, X2 = X1 + (2 + CB) * NK, X3 = X2 + NT, TOTAL = X3 + NT;

  const int tid = threadIdx.x, lane = tid & 63, j = lane >> 4, n = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const UnitChunk uc = split_unit(id, a.n_whole, a.n_split, a.n_split_units, a.by_split_units);
  int kt, bh;
  decode_workgroup(uc.unit, a.by_tiles, a.n_bh, a.by_xcd, a.tile_major, kt, bh);   // early key tiles see every query row: heaviest first
  int b, hk;
  div_mod(bh, a.by_kv_heads, b, hk);
  const int seg_off = a.seg_off, seg_len = a.seg_len, kv_len = seg_off + seg_len;
  const int j0 = kt * Cfg::BNW;                    // first key of the workgroup
  const int wkey0 = j0 + wave * 16 * CB;                // first key of the wave

  const int64_t kvoff = b * a.kv_sb + hk * a.kv_sh;
  const T *kbase = reinterpret_cast<const T *>(a.k) + kvoff;
  const T *vbase = reinterpret_cast<const T *>(a.v) + kvoff;

  // First query row that can see any key of this workgroup, and the tile holding it.  Iteration `it` covers
  // tile qt_first + it % per_head of query head hk * group + it / per_head.
  const int r_first = j0 > seg_off ? j0 - seg_off : 0;
  const int qt_first = r_first / BQ;
  const int n_qt = (seg_len + BQ - 1) / BQ;
  const int per_head = n_qt - qt_first;            // >= 1 because j0 < kv_len
  // All iterations, or one chunk of them.
  const int all = per_head * a.group;
  int it_begin = 0, it_end = all;
  if (uc.n_chunks > 1) {   // (at most 16 chunks of 2^28 / 32 + 65535 iterations: batch * heads * rows are at most 2^28)
    it_begin = div(uc.chunk * all, a.by_split);
    it_end = div((uc.chunk + 1) * all, a.by_split);
  }
  int head0 = 0, tile0 = it_begin;   // where iteration it_begin is
  if (it_begin > 0) {
    head0 = it_begin / per_head;
    tile0 = it_begin - head0 * per_head;
  }
  const float c = uniform(a.scale * kLog2e / (M::UP * M::UP));
  const bool w_active = wkey0 < kv_len;

  const lds_addr lds0 = to_lds_addr(smem);
  const lds_addr vtile = lds0 + Cfg::STAGES * Cfg::STAGE_BYTES;
  const lds_addr stats0 = vtile + Cfg::V_BYTES;
  M rd;
  rd.init(lane);
  // V rows of the workgroup's keys -> LDS (keys past the prefix: copies of its last row, products never stored).  fp32: through
  // registers, written when the first tile and the K rows are on their way as well
  Copy lv[ASYNC ? 1 : 2];
#pragma unroll
  for (int i = 0; i < 4; i += 2) {
    const int key0 = j0 + 32 * (i + ((wave >> 1) & 1)), at = key0 < kv_len ? key0 : kv_len - 1;
    const T *row = vbase + (int64_t)at * a.kv_ss;
    Copy &l = lv[ASYNC ? 0 : i / 2];
    if (!ASYNC || i == 0) l.init(wave, lane, a.kv_ss);
    if constexpr (ASYNC) l.issue(row, row, a.kv_ss, kv_len - at, kv_len - at, vtile + i * TB, wave);
    else l.load(row, row, a.kv_ss, kv_len - at, kv_len - at, wave);
  }
  // Tile cursors (row offset of the tile, its query head, its ring stage), advanced once per iteration.
  struct Cursor {
    int r0, hq, stage;
  };
  auto advance = [&](Cursor &t) {
    t.r0 += BQ;
    if (t.r0 >= n_qt * BQ) { t.r0 = qt_first * BQ; ++t.hq; }
    t.stage ^= 1;
  };
  Copy ld;
  ld.init(wave, lane, a.q_ss);
  auto issue = [&](const Cursor &t) {   // rows past the segment re-read its last row
    const int64_t qoff = b * a.q_sb + t.hq * a.q_sh + (int64_t)t.r0 * a.q_ss;
    const T *q = reinterpret_cast<const T *>(a.q) + qoff, *dout = reinterpret_cast<const T *>(a.dout) + qoff;
    const int left = seg_len - t.r0;
    if constexpr (ASYNC) ld.issue(q, dout, a.q_ss, left, left, lds0 + t.stage * Cfg::STAGE_BYTES, wave);
    else ld.load(q, dout, a.q_ss, left, left, wave);
    if (wave == 0) {   // lane l copies entry l of {-lse/scale [32], -delta [32]}
      const int l = lane_id(), rr = t.r0 + l % BQ;
      const unsigned plane = (unsigned)((l / BQ) * a.ws_plane);
      const float *sb = a.delta + ((int64_t)b * a.n_q_heads + t.hq) * seg_len;     // wave-uniform
      const unsigned so = (plane + (unsigned)(rr < seg_len ? rr : seg_len - 1)) * 4u;
      const unsigned dst = stats0 + (unsigned)(t.stage * Cfg::STAT_BYTES);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(dst), "v"(so), "s"(sb) : "m0");
    }
  };
  Cursor t_iss = {(qt_first + tile0) * BQ, hk * a.group + head0, 0};   // next tile to copy
  Cursor cur = t_iss;                                                  // tile of the current iteration
  if (it_begin < it_end) issue(t_iss);
  advance(t_iss);
  // K rows of the wave's keys stay in registers for the whole kernel.
  typename M::RowOp kr[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    int key = wkey0 + 16 * cb + n;
    key = key < kv_len ? key : kv_len - 1;     // keys past the prefix are computed on a copy and never stored
    M::load_row(kr[cb], kbase + (int64_t)key * a.kv_ss, j);
#pragma unroll
    for (int i = 0; i < M::NK; ++i) settle(kr[cb].f[i]);
  }
  f32x4 dk[CB][DB], dv[CB][DB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int db = 0; db < DB; ++db) dk[cb][db] = dv[cb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  // one stage: the tile whose rows are in registers
  auto write_tile = [&]() {
    if constexpr (!ASYNC) {
#pragma unroll
      for (int x = 0; x < Copy::NI; ++x) ld.write(x, lds0);
    }
  };
  if constexpr (!ASYNC) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int x = 0; x < Copy::NI; ++x) lv[i].write(x, vtile + 2 * i * TB);
    if (it_begin < it_end) write_tile();
  }
  wait_async_tiles();
  __syncthreads();

  for (int it = it_begin; it < it_end; ++it) {
    // (two stages) the stage this copy overwrites was last read before the barrier that ended the previous iteration
    if (it + 1 < it_end) issue(t_iss);
    advance(t_iss);
    if (w_active && wkey0 <= seg_off + cur.r0 + 31) {
      const lds_addr qt = lds0 + (ASYNC ? cur.stage * Cfg::STAGE_BYTES : 0);   // the dO tile lies TB behind it
      const lds_addr st = opaque(stats0 + (unsigned)(cur.stage * Cfg::STAT_BYTES + 16 * j));
      const typename M::Nat qn = rd.nat_at(qt), vn = rd.nat_at(CB == 2 ? vtile + wave * TB : vtile + (wave >> 1) * TB + (wave & 1) * NK * 1024);
      const typename M::Tr qx = rd.tr_at(qt);
      // Operand x of the iteration: Q [NN], then per step along D dO, V [CB], dO, then dO and Q transposed [NT each].
      auto operand = [&](int x) {
        if (x < X1) return M::nat(qn, x);
        if (x < X2) {
          const int ks = (x - X1) / (2 + CB), w = (x - X1) % (2 + CB);
          return w == 0 ? M::nat(qn, ks, TB) : w == 1 + CB ? M::nat(qn, NK + ks, TB) : M::nat(vn, (w - 1) * NK + ks);
        }
        return x < X3 ? M::tr(qx, x - X2, TB) : M::tr(qx, x - X3);
      };
      Frag fr[PR];
      auto used = [&](int x) {   // operand x has been used up: read the one that takes its place
        if (x + PR < TOTAL) fr[x % PR] = operand(x + PR);
      };
      f32x4 s[2][CB], dp[2][CB];
      f32x4 nl[2], nd[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) fr[x] = operand(x);
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) nl[rb] = lds_load<f32x4>(st + 64 * rb) * (M::UP * M::UP);
#pragma unroll
      for (int x = 2; x < PR; ++x) fr[x] = operand(x);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NN; ++i)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          s[i / NK][cb] = M::mma_nat(i, fr[i % PR], kr[cb], i % NK ? s[i / NK][cb] : nl[i / NK]);
          if (cb + 1 == CB) used(i);
          if (cb + 1 == CB && i + 2 >= NN) nd[i + 2 - NN] = lds_load<f32x4>(st + 4 * BQ + 64 * (i + 2 - NN)) * (M::UP * M::UP);
          __builtin_amdgcn_sched_barrier(0);
        }
      auto probs = [&](int x0, int x1) {   // probabilities x0 .. x1-1 of the lane's 8 * CB
#pragma unroll
        for (int x = x0; x < x1; ++x) {
          float y = exp2_fast(s[x / (4 * CB)][(x >> 2) % CB][x & 3] * c);
          settle(y);
          s[x / (4 * CB)][(x >> 2) % CB][x & 3] = y;
        }
      };
#pragma unroll
      for (int ks = 0; ks < NK; ++ks)
#pragma unroll
        for (int i = 0; i < 2 * CB; ++i) {
          const int rb = i / CB, cb = i % CB, x = X1 + (2 + CB) * ks;
          dp[rb][cb] = M::mma_op(ks, fr[(x + (rb ? 1 + CB : 0)) % PR], fr[(x + 1 + cb) % PR], ks ? dp[rb][cb] : nd[rb]);
          if (rb == 0 && cb + 1 == CB) used(x);   // the first row half's dO; then V as the second half uses it; its dO last
          if (rb == 1) used(x + 1 + cb);
          if (rb == 1 && cb + 1 == CB) used(x + 1 + CB);
          const int w = 2 * CB * ks + i, W = 2 * CB * NK;
          probs(8 * CB * w / W, 8 * CB * (w + 1) / W);
          __builtin_amdgcn_sched_barrier(0);
        }
      // Visible iff key <= seg_off + row and row < seg_len.  Tiles on the diagonal or at the end of the segment: entries
      // above the diagonal and rows past the segment are set to zero here, in a branch that holds nothing else (whatever
      // the exponential made of them, infinity included, is overwritten).
      if ((wkey0 + 16 * CB - 1 > seg_off + cur.r0) || (cur.r0 + 32 > seg_len)) {
        asm volatile("" ::: "memory");   // keeps this a branch
        const int fl = lane_id(), fj = fl >> 4;
        const int lo = wkey0 + (fl & 15) - seg_off - cur.r0 - 4 * fj;   // need 16*rb + v >= lo + 16*cb
        const int hi = seg_len - cur.r0 - 4 * fj;                       // and  16*rb + v <  hi
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 * rb + v < lo + 16 * cb || 16 * rb + v >= hi) {
                s[rb][cb][v] = 0.f;
                dp[rb][cb][v] = 0.f;
              }
      }
      typename M::Slab pf[CB], ds[CB];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        pf[cb] = M::slab_up(s[0][cb], s[1][cb]);
        M::settle_slab(pf[cb]);
      }
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          M::mma_tr(i, fr[(X2 + i) % PR], pf[cb], dv[cb]);
          if (cb + 1 == CB) used(X2 + i);
          if (i == 1) {
            ds[cb] = M::slab(s[0][cb] * dp[0][cb], s[1][cb] * dp[1][cb]);
            M::settle_slab(ds[cb]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          M::mma_tr(i, fr[(X3 + i) % PR], ds[cb], dk[cb]);
          if (cb + 1 == CB) used(X3 + i);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    advance(cur);
    wait_async_tiles();   // this wave's part of tile it+1 has landed
    __syncthreads();
    if constexpr (!ASYNC) {
      if (it + 1 < it_end) write_tile();
      __syncthreads();
    }
  }

  if constexpr (sizeof(T) == 4) {
    float bad = 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        bad = add_if_not_finite(dv[cb][db], add_if_not_finite(dk[cb][db], bad));
        dv[cb][db] *= 1.f / (M::UP * M::UP);
        dk[cb][db] *= 1.f / (M::UP * M::UP * M::UP);
      }
    if (__builtin_expect(any_not_finite(bad), 0)) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const int pl = lane_id(), pj = pl >> 4, key = wkey0 + 16 * cb + (pl & 15), kc = key < kv_len ? key : kv_len - 1;
        PlainRow<D> k_row, v_row;
        k_row.load(kbase + (int64_t)kc * a.kv_ss, pj);
        v_row.load(vbase + (int64_t)kc * a.kv_ss, pj);
#pragma unroll
        for (int db = 0; db < DB; ++db) dk[cb][db] = dv[cb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
        float met = 0.f;
#pragma unroll 1
        for (int it = it_begin; it < it_end && !all_nan(met); ++it) {
          const int hq = hk * a.group + it / per_head, r0 = (qt_first + it % per_head) * BQ, r1 = r0 + BQ < seg_len ? r0 + BQ : seg_len;
          const int64_t qoff = b * a.q_sb + hq * a.q_sh;
          dkdv_plain<D>(k_row, v_row, reinterpret_cast<const T *>(a.q) + qoff, reinterpret_cast<const T *>(a.dout) + qoff, a.q_ss,
                        a.delta + ((int64_t)b * a.n_q_heads + hq) * seg_len, a.ws_plane, r0, r1, kc - seg_off,
                        c * (M::UP * M::UP), pj, dk[cb], dv[cb], met);
        }
      }
    }
  }

  // Epilogue: acc[key][d] += result, each element touched by exactly one lane of the grid.  In the accumulators a
  // lane holds ONE key per column block and 4-element pieces of its row: read-modify-write straight from there would
  // touch 16 cache lines per 64 lanes.  Each wave therefore passes its 32 x D block through LDS (its own region; 16-byte
  // chunk c of row r at position c ^ (r & 15), so that the row-per-lane writes spread over all banks) and updates the
  // accumulators row by row, LPR lanes side by side on one row.
  const int el = lane_id(), en = el & 15, ej = el >> 4;   // (anew: not kept in registers across the loop)
  float *dkb = a.dk_acc + kvoff, *dvb = a.dv_acc + kvoff;
  constexpr int LPR = D / 4;                        // lanes per row (16 bytes each)
  constexpr int RPI = 64 / LPR;                     // rows per instruction
  constexpr int KW = 16 * CB;                       // keys of the wave
  constexpr int NI = (KW + RPI - 1) / RPI;          // instructions per block
  char *region = smem + wave * (KW * Cfg::EPI_ROW);
  const int row_in = el / LPR, col = el % LPR;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const float mul = which == 0 ? a.scale : 1.f;
    float *base = which == 0 ? dkb : dvb;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int x = 0; x < DB; ++x) {
        const int r = 16 * cb + en, ch = M::quad_d0(x, ej) >> 2;
        *reinterpret_cast<f32x4 *>(region + r * Cfg::EPI_ROW + 16 * (ch ^ en)) = M::quad(which == 0 ? dk[cb] : dv[cb], x) * mul;
      }
    if (uc.chunk > 0) {   // a chunk other than the first: its share goes to the workspace, [chunk - 1][dK, dV][key][head_dim]
      float *part = a.part + ((int64_t)(uc.slot - a.n_split_units) * 2 + which) * (Cfg::BNW * D) + (int64_t)(wave * KW) * D;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int r = i * RPI + row_in, rc = r < KW ? r : KW - 1;
        const f32x4 x = *reinterpret_cast<const f32x4 *>(region + rc * Cfg::EPI_ROW + 16 * (col ^ (rc & 15)));
        if (row_in < RPI && r < KW) *reinterpret_cast<f32x4 *>(part + (int64_t)r * D + 4 * col) = x;
      }
      continue;
    }
    f32x4 old[NI];   // rows that are not this lane's to update are read all the same, from a valid place
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int key = wkey0 + i * RPI + row_in;
      old[i] = *reinterpret_cast<const f32x4 *>(base + (int64_t)(key < kv_len ? key : kv_len - 1) * a.kv_ss + 4 * col);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = i * RPI + row_in, key = wkey0 + r, rc = r < KW ? r : KW - 1;
      const f32x4 sum = old[i] + *reinterpret_cast<const f32x4 *>(region + rc * Cfg::EPI_ROW + 16 * (col ^ (rc & 15)));
      if (row_in < RPI && r < KW && key < kv_len) *reinterpret_cast<f32x4 *>(base + (int64_t)key * a.kv_ss + 4 * col) = sum;
    }
  }
}

// Adds the chunks of the units that were cut along the queries into the accumulators, which chunk
// 0 has updated itself: acc += sum_c part_c, c = 1 .. n_split - 1, in the order of the chunks.  A thread handles 4
// consecutive head_dim elements of one key of one of the two accumulators (grid: split units x DkdvMerge<D>::GROUPS).
template <int D> struct DkdvMerge {
  static constexpr int PER = 128 * D / 4;                  // threads per unit and accumulator
  static constexpr int GROUPS = 2 * PER / 256;
  static_assert(PER % 256 == 0, "whole workgroups per accumulator");
};
template <typename T, int D, int MC> S1F_DEV void bwd_dkdv_merge_body(const AttnArgs &a, int id) {
  typedef DkdvMerge<D> DM;
  const int unit = id / DM::GROUPS, g = id % DM::GROUPS;
  const int which = g / (DM::GROUPS / 2), t = (g % (DM::GROUPS / 2)) * 256 + (int)threadIdx.x;
  int kt, bh;
  decode_workgroup(a.n_whole + unit, a.by_tiles, a.n_bh, a.by_xcd, a.tile_major, kt, bh);
  int b, hk;
  div_mod(bh, a.by_kv_heads, b, hk);
  const int key = kt * 128 + t / (D / 4), S = a.n_split - 1;   // partial results
  if (key >= a.seg_off + a.seg_len) return;
  int slot0, slot_step;
  chunk_slots(unit, a.n_split_units, slot0, slot_step);
  const float *part = a.part + ((int64_t)slot0 * 2 + which) * (128 * D) + 4 * t;
  f32x4 pc[MC];
#pragma unroll
  for (int c = 0; c < MC; ++c)   // past the last chunk: that one again, not added
    pc[c] = *reinterpret_cast<const f32x4 *>(part + (int64_t)(c < S ? c : S - 1) * slot_step * (2 * 128 * D));
  float *acc = (which ? a.dv_acc : a.dk_acc) + b * a.kv_sb + hk * a.kv_sh + (int64_t)key * a.kv_ss + 4 * (t % (D / 4));
  f32x4 sum = pc[0];
#pragma unroll
  for (int c = 1; c < MC; ++c)
    if (c < S) sum += pc[c];
  *reinterpret_cast<f32x4 *>(acc) = *reinterpret_cast<const f32x4 *>(acc) + sum;
}

// ---- the kernels: one half by itself, and both ----
template <typename T, int D, int NC, int OCC, int WAVES, bool PAIR = false>
__global__ void __launch_bounds__(64 * WAVES, OCC) seg_attn_bwd_dq_kernel(const AttnArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  bwd_dq_body<T, D, NC, WAVES, true, PAIR>(a, blockIdx.x, smem);
}
template <typename T, int D, int WGS>   // WGS: waves meant to share a SIMD
__global__ void __launch_bounds__((64 * BwdDkdvCfg<T, D>::WAVES), WGS) seg_attn_bwd_dkdv_kernel(const AttnArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  bwd_dkdv_body<T, D>(a, blockIdx.x, smem);
}
// Both halves in one launch, first `first` workgroups of the one with the longer units, then those of the other: small calls,
// chains of launches that each leave most of the chip idle, get shorter by one, and the last round of the first half
// is filled by units of the second.
template <typename T, int D, int NC, int OCC, int WAVES>
__global__ void __launch_bounds__(64 * WAVES, OCC) seg_attn_bwd_kernel(const AttnArgs aq, const AttnArgs ak, int first, int dq_first) {
  static_assert(WAVES == BwdDkdvCfg<T, D>::WAVES, "both halves run in workgroups of one size");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int id = blockIdx.x < first ? blockIdx.x : blockIdx.x - first;
  if ((blockIdx.x < first) == (dq_first != 0)) bwd_dq_body<T, D, NC, WAVES, false>(aq, id, smem);
  else bwd_dkdv_body<T, D>(ak, id, smem);
}
// The merges of either half or both: `q_groups` workgroups of the dQ half, then those of the dK/dV half.
template <typename T, int D, int MC>
__global__ void __launch_bounds__(256) seg_attn_bwd_merge_kernel(const AttnArgs aq, const AttnArgs ak, int q_groups) {
  if (blockIdx.x < q_groups) bwd_dq_merge_body<T, D, MC>(aq, blockIdx.x);
  else bwd_dkdv_merge_body<T, D, MC>(ak, blockIdx.x - q_groups);
}

}  // namespace s1f

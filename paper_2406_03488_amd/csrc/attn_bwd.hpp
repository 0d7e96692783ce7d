// Backward of one segment (derivative of Section 3.1, Eq. 3; accumulation per Section 3.2):
//   p_ij = exp(s_ij - lse_i),  delta_i = dO_i . O_i,  dp_ij = dO_i . v_j,  ds_ij = p_ij (dp_ij - delta_i)
//   dq_i = scale * sum_j ds_ij k_j      dk_j += scale * sum_i ds_ij q_i      dv_j += sum_i p_ij dO_i
//
// Two kernels, neither uses atomics:
//   seg_attn_bwd_dq_kernel    owns query rows (same decomposition as the forward), loops over key tiles,
//                             also writes delta for the second kernel;
//   seg_attn_bwd_dkdv_kernel  owns key rows, loops over the query heads of its K/V group and over the
//                             segment's query tiles, and adds its result into the fp32 prefix accumulators
//                             (each accumulator element is touched by exactly one lane of one workgroup).
// The probabilities are recomputed in both (7 matrix products in total instead of 5) in exchange for
// deterministic sums and no dQ workspace.
#pragma once
#include <type_traits>

#include "attn_tile.hpp"


namespace s1f {

template <typename T, int D, int NC> struct BwdDqCfg {
  static constexpr int BM = 64 * NC, BN = 32, THREADS = 256;
  static constexpr int LDS_BYTES = TileRing<T, D>::LDS_BYTES;
};

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
// Bound by the matrix pipe at the clock the power limit leaves (head_dim 128: 60 % busy at 1.85 GHz), with 64 registers
// of accumulators and 64 of Q and dO per lane at NC = 2.  32 heads, 4096 rows behind 28672 keys: head_dim 128
// 2.52 -> 2.29 ms (three products executed: 1230 -> 1350 TFLOP/s), 80 1.89 -> 1.57 ms and 64 1.54 -> 1.26 ms (NC = 3).
// One wave per SIMD with 64 rows (half the LDS reads) ran 15 % slower: half of its registers are accumulator
// registers, which the vector phases reach by copies only.
constexpr int kDqRing = 4;

template <typename T, int D, int NC, int OCC>
__global__ void __launch_bounds__(256, OCC) seg_attn_bwd_dq_kernel(const AttnArgs a) {
  typedef BwdDqCfg<T, D, NC> Cfg;
  typedef Mat<T, D> M;
  typedef typename M::Frag Frag;
  typedef TileRing<T, D> Ring;
  constexpr int DB = M::DB, BM = Cfg::BM, BN = Cfg::BN, NN = M::NN, NK = M::NK, NT = M::NT, PR = kDqRing;
  constexpr int TOTAL = NN + NT + NN;
  static_assert(NN >= PR && NT >= PR, "operand ring deeper than a product");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, j = lane >> 4, n = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const UnitChunk uc = split_unit(blockIdx.x, a.n_whole, a.n_split, a.n_split_units);
  int qt, bh;
  decode_workgroup(uc.unit, a.n_tiles, a.n_bh, a.tile_major, qt, bh);
  qt = a.n_tiles - 1 - qt;   // later (heavier) row tiles are scheduled first
  const int h = bh % a.n_q_heads, b = bh / a.n_q_heads, hk = h / a.group;
  const int seg_len = a.seg_len;
  const int row0 = qt * BM, wrow0 = row0 + wave * 16 * NC;
  const int last_row = (row0 + BM < seg_len ? row0 + BM : seg_len) - 1;
  // This workgroup's key tiles: all that hold keys 0 .. seg_off+last_row, or one chunk of them.  From here on keys
  // are counted from the chunk's first key: seg_off and kv_len are relative to it.
  int kt0, kt1;
  chunk_range(uc, (a.seg_off + row0) / BN, (a.seg_off + last_row) / BN + 1, kt0, kt1);
  const int seg_off = a.seg_off - BN * kt0, kv_len = seg_off + seg_len;
  const int n_kt = kt1 - kt0;

  const int64_t qoff = b * a.q_sb + h * a.q_sh;
  const int64_t kv_first = b * a.kv_sb + hk * a.kv_sh + (int64_t)(BN * kt0) * a.kv_ss;
  Ring ring;
  ring.init(reinterpret_cast<const T *>(a.k) + kv_first, reinterpret_cast<const T *>(a.v) + kv_first, a.kv_ss, n_kt, kv_len,
            to_lds_addr(smem), wave, lane);
  ring.issue(0);
  ring.issue(1);

  typename M::RowOp q[NC], dor[NC];
  float nl[NC];    // -lse in log2 units
  f32x4 nd[NC];    // -delta
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    const int r = wrow0 + 16 * cb + n, rc = r < seg_len ? r : seg_len - 1;
    const int64_t off = qoff + (int64_t)rc * a.q_ss;
    M::load_row(q[cb], reinterpret_cast<const T *>(a.q) + off, j);
    M::load_row(dor[cb], reinterpret_cast<const T *>(a.dout) + off, j);
    typename M::RowOp o;
    M::load_row(o, reinterpret_cast<const T *>(a.out) + off, j);
    const float d = -sum_over_rows(M::dot(dor[cb], o));
    nd[cb] = f32x4{d, d, d, d};
    const int64_t at = ((int64_t)b * a.n_q_heads + h) * seg_len + rc;
    const float lse = a.lse[at];
    nl[cb] = -lse * kLog2e;
    if (r < seg_len && j == 0 && uc.chunk == 0) {   // row statistics for the dK/dV kernel
      a.delta[at] = -lse / a.scale;
      a.delta[a.ws_plane + at] = d;
    }
  }
  f32x4 dq[NC][DB];
#pragma unroll
  for (int cb = 0; cb < NC; ++cb)
#pragma unroll
    for (int db = 0; db < DB; ++db) dq[cb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c = uniform(a.scale * kLog2e);
  M rd;
  rd.init(lane);
#pragma unroll
  for (int cb = 0; cb < NC; ++cb)
#pragma unroll
    for (int i = 0; i < M::NK; ++i) { settle(q[cb].f[i]); settle(dor[cb].f[i]); }

  if (n_kt <= 0) {   // more chunks than this unit has whole tiles: nothing to add
    float *pd = a.part + (int64_t)uc.slot * (BM * D);
    for (int i = tid; i < BM * D; i += 256) pd[i] = 0.f;
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
  {
    const typename M::Nat ka = rd.nat_at(ring.st[1]);
#pragma unroll
    for (int i = 0; i < PR; ++i) fr[i] = M::nat(ka, i);
  }
  typename M::Slab ds[NC];
  auto make_ds = [&](int cb) {
    ds[cb] = M::slab(p[0][cb] * dp[0][cb], p[1][cb] * dp[1][cb]);
    M::settle_slab(ds[cb]);
  };
  auto step = [&](auto mask, auto whole) {
    constexpr bool MASK = decltype(mask)::value, WHOLE = decltype(whole)::value;
    ring.template begin_step<WHOLE>(n_kt - 1 - k);
    const typename M::Nat kn = rd.nat_at(ring.st[1]), ka = rd.nat_at(ring.st[2]);
    const typename M::Tr kt = rd.tr_at(ring.st[0]);
    auto next_operand = [&](int x) {   // operand x has been used up: the one that takes its place
      const int y = x + PR;
      if (y < NN) fr[x % PR] = M::nat(kn, y);
      else if (y < NN + NT) fr[x % PR] = M::tr(kt, y - NN);
      else if (y < TOTAL) fr[x % PR] = M::nat(kn, y - NN - NT, Tile32<T, D>::BYTES);
      else fr[x % PR] = M::nat(ka, x % PR);   // the next step's first ones
    };
    f32x4 sn[2][NC];
#pragma unroll
    for (int i = 0; i < NN; ++i)
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        sn[i / NK][cb] = M::mma_nat(i, fr[i % PR], q[cb], i % NK ? sn[i / NK][cb] : zero);
        if (cb + 1 == NC) next_operand(i);
        if (i == 1) make_ds(cb);
        __builtin_amdgcn_sched_barrier(0);
      }
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
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
    for (int i = 0; i < NN; ++i)
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        dp[i / NK][cb] = M::mma_nat(i, fr[(NN + NT + i) % PR], dor[cb], i % NK ? dp[i / NK][cb] : nd[cb]);
        if (cb + 1 == NC) next_operand(NN + NT + i);
        if (MASK && i == 0 && cb + 1 == NC) hide(p, BN * (k + 1));
        __builtin_amdgcn_sched_barrier(0);
      }
    ++k;
    ring.end_step();
  };
  int n_full = (wfirst + 1) / BN;   // tiles that every row of the wave sees in full
  n_full = n_full < n_kt - 1 ? n_full : n_kt - 1;
  const std::integral_constant<bool, true> yes;
  const std::integral_constant<bool, false> no;
  const int n_fast = n_full < n_kt - 4 ? n_full : n_kt - 4;   // ... while there is a whole tile to copy
  while (k + 1 < n_fast) step(no, yes);
  while (k + 1 < n_full) step(no, no);
  while (k + 1 < n_kt) step(yes, no);
  {   // last tile: dS and dQ
    const typename M::Tr kt = rd.tr_at(ring.st[0]);
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) make_ds(cb);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const Frag kf = M::tr(kt, i);
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) M::mma_tr(i, kf, ds[cb], dq[cb]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  if (uc.slot >= 0) {   // a chunk: its unscaled share of the unit's dQ rows goes to the workspace
    float *pd = a.part + (int64_t)uc.slot * (BM * D);
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      const int rl = wave * 16 * NC + 16 * cb + n;   // row within the unit
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

// Sums the chunks of the units that seg_attn_bwd_dq_kernel split along the keys: dq = scale * sum_c part_c.
// Thread and grid layout as in seg_attn_fwd_merge_kernel.
template <typename T, int D>
__global__ void __launch_bounds__(256) seg_attn_bwd_dq_merge_kernel(const AttnArgs a) {
  constexpr int C4 = D / 4, RG = 256 / C4;
  const int BM = a.bm, GROUPS = (BM + RG - 1) / RG;
  const int unit = (int)blockIdx.x / GROUPS, rg = (int)blockIdx.x % GROUPS;
  const int rl = rg * RG + (int)threadIdx.x / C4, c4 = (int)threadIdx.x % C4;
  int qt, bh;
  decode_workgroup(a.n_whole + unit, a.n_tiles, a.n_bh, a.tile_major, qt, bh);
  qt = a.n_tiles - 1 - qt;
  const int h = bh % a.n_q_heads, b = bh / a.n_q_heads;
  const int r = qt * BM + rl, S = a.n_split;
  if ((int)threadIdx.x >= RG * C4 || rl >= BM || r >= a.seg_len) return;
  int slot0, slot_step;
  chunk_slots(unit, a.n_split_units, slot0, slot_step);
  const float *pd = a.part + (int64_t)slot0 * (BM * D) + rl * D + 4 * c4;
  f32x4 pc[kMaxChunks];
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c)
    pc[c] = c < S ? *reinterpret_cast<const f32x4 *>(pd + (int64_t)c * slot_step * (BM * D)) : f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 acc = pc[0];
#pragma unroll
  for (int c = 1; c < kMaxChunks; ++c) acc += pc[c];
  T *dqb = reinterpret_cast<T *>(a.dq) + b * a.q_sb + h * a.q_sh;
  store4<T>(dqb + (int64_t)r * a.q_ss + 4 * c4, acc[0] * a.scale, acc[1] * a.scale, acc[2] * a.scale, acc[3] * a.scale);
}

// dK/dV kernel.  NW waves of 32 keys each; Q/dO tiles of 32 rows travel through a ring of NST LDS stages.
// DIST: a tile's copy is issued DIST iterations before the iteration that consumes it.
// LAG:  with LAG = 1 the upper half of the waves runs one phase behind the lower half (see the kernel), which
// keeps each tile alive for one more iteration.
template <typename T, int D, int NW, int DIST, int LAG> struct BwdDkdvCfg {
  static constexpr int BQ = 32;                        // rows per Q/dO tile
  static constexpr int BNW = 32 * NW;                  // keys per workgroup
  static constexpr int THREADS = 64 * NW;
  static constexpr int NST = DIST + LAG + 1;           // ring stages
  typedef LdsTile<T, BQ, D> QT;
  static constexpr int STAGE_BYTES = 2 * QT::BYTES;    // Q tile, dO tile right behind it
  static constexpr int STAT_BYTES = 2 * BQ * 4;        // -lse/scale and -delta of the tile's rows
  typedef PaddedRows<T, BNW, D> VT;                    // the workgroup's V rows
  static constexpr int LDS_BYTES = NST * STAGE_BYTES + VT::BYTES + NST * STAT_BYTES;   // stages, V, statistics
  static_assert(STAGE_BYTES % 8192 == 0, "stages must keep the 8 KiB alignment of the fragment reader");
  static_assert(DIST >= 1 && LAG >= 0 && LAG <= 1 && NW % 4 == 0, "schedule");
};

// Lane = one key (column ln); queries run over registers.
//   S[q][key]  = Q K^T         A = Q (LDS),              B = K (registers)
//   dP[q][key] = dO V^T        A = dO (LDS),             B = V (LDS)
//   dV^T[d][key] += dO^T P     A = dO read transposed,   B = P slab (registers)
//   dK^T[d][key] += Q^T dS     A = Q read transposed,    B = dS slab (registers)
// The wave's K fragments, its dK and dV accumulators and the block's S and dP fill the register budget of
// two waves per SIMD; its V rows are therefore read from LDS (copied there once, in padded rows).
// Q/dO tiles and their row statistics are copied HBM -> LDS asynchronously (no staging registers).
//
// A wave's work on one tile has three phases: B (S and dP on the matrix pipe), C (exp and dS on the vector
// pipe), D (dV and dK on the matrix pipe).  Two waves share a SIMD, and one's vector phase should meet the other's
// matrix phases instead of both queueing for the same pipe.  Either the two belong to different workgroups (NW = 4,
// WGS = 2: two workgroups per compute unit with barriers of their own, which also overlaps one's prologue and
// epilogue with the other's loop; the shape the library launches for bf16), or to the two halves of one workgroup
// (NW = 8) whose upper half, with LAG = 1, runs the sequence one phase late (C and D of the previous tile, then B of
// the current one).
template <typename T, int D, int NW, int DIST, int LAG, int WGS = 1>   // WGS: workgroups meant to share a compute unit
__global__ void __launch_bounds__(64 * NW, WGS * NW / 4) seg_attn_bwd_dkdv_kernel(const AttnArgs a) {
  typedef Elem<T> E;
  typedef typename E::Frag Frag;
  typedef BwdDkdvCfg<T, D, NW, DIST, LAG> Cfg;
  typedef typename Cfg::QT QT;
  typedef FragReader<QT, T> RD;
  constexpr int EPL = E::EPL, KSTEP = 2 * EPL, NKS = D / KSTEP;
  constexpr int DB = QT::DPAD / 32, NSLAB = 16 / EPL, BQ = Cfg::BQ, NST = Cfg::NST;
  constexpr int PF = 2;              // steps by which operand fragments are read ahead in phase B ...
  constexpr int PFD = 2;             // ... and in phase D (deeper rings spill at two waves per SIMD and run slower)
  constexpr int NV = NSLAB * DB;     // (slab, d-block) steps of the second pair of products
  static_assert(NKS >= PF && NV >= PFD && PFD >= PF, "prefetch ring deeper than the products");

  extern __shared__ __attribute__((aligned(8192))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, ln = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int kt, bh;
  decode_workgroup(blockIdx.x, a.n_tiles, a.n_bh, a.tile_major, kt, bh);   // early key tiles see every query row: heaviest first
  const int n_kv_heads = a.n_q_heads / a.group;
  const int hk = bh % n_kv_heads, b = bh / n_kv_heads;
  const int seg_off = a.seg_off, seg_len = a.seg_len, kv_len = seg_off + seg_len;
  const int j0 = kt * Cfg::BNW;                    // first key of the workgroup
  const int wkey0 = j0 + wave * 32;                // first key of the wave

  const int64_t kvoff = b * a.kv_sb + hk * a.kv_sh;
  const T *kbase = reinterpret_cast<const T *>(a.k) + kvoff;
  const T *vbase = reinterpret_cast<const T *>(a.v) + kvoff;

  // First query row that can see any key of this workgroup, and the tile holding it.  Iteration `it` covers
  // tile qt_first + it % per_head of query head hk * group + it / per_head.
  const int r_first = j0 > seg_off ? j0 - seg_off : 0;
  const int qt_first = r_first / BQ;
  const int n_qt = (seg_len + BQ - 1) / BQ;
  const int per_head = n_qt - qt_first;            // >= 1 because j0 < kv_len
  const int n_it = per_head * a.group;
  const float c = a.scale * kLog2e;
  const bool w_active = wkey0 < kv_len;

  const lds_addr lds0 = to_lds_addr(smem);
  const lds_addr vtile = lds0 + NST * Cfg::STAGE_BYTES;
  const lds_addr stats0 = vtile + Cfg::VT::BYTES;
  AsyncTilePairU<T, BQ, D, NW> ld;
  ld.init(wave, lane, a.q_ss);
  RD rd;
  rd.init(lane);

  // Tile cursors (row offset of the tile, its query head, its ring stage), advanced once per iteration.
  struct Cursor {
    int r0, hq, stage;
  };
  auto advance = [&](Cursor &t) {
    t.r0 += BQ;
    if (t.r0 >= n_qt * BQ) { t.r0 = qt_first * BQ; ++t.hq; }
    t.stage = t.stage + 1 == NST ? 0 : t.stage + 1;
  };
  auto issue = [&](const Cursor &t) {   // rows past the segment re-read its last row
    const int64_t qoff = b * a.q_sb + t.hq * a.q_sh;
    ld.issue(reinterpret_cast<const T *>(a.q) + qoff, reinterpret_cast<const T *>(a.dout) + qoff, a.q_ss, t.r0, seg_len,
             lds0 + t.stage * Cfg::STAGE_BYTES, wave, lane);
    if (wave < 2 * BQ / 64) {   // lane `lane` copies entry 64*wave + lane of {-lse/scale [BQ], -delta [BQ]}
      const int st_idx = wave * 64 + fresh(lane), rr = t.r0 + st_idx % BQ;
      const unsigned st_plane = (unsigned)((st_idx / BQ) * a.ws_plane);
      const float *sb = a.delta + ((int64_t)b * a.n_q_heads + t.hq) * seg_len;     // wave-uniform
      const unsigned so = (st_plane + (unsigned)(rr < seg_len ? rr : seg_len - 1)) * 4u;
      const unsigned dst = stats0 + (unsigned)(t.stage * Cfg::STAT_BYTES + wave * 256);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(dst), "v"(so), "s"(sb) : "m0");
    }
  };

  // V rows of the workgroup's keys -> LDS (rows past the prefix are zero: their products are never stored)
  Cfg::VT::template copy<Cfg::THREADS>(smem + NST * Cfg::STAGE_BYTES, vbase + (int64_t)j0 * a.kv_ss, a.kv_ss, kv_len - j0, tid);
  // K fragments of the wave's keys stay in registers for the whole kernel.
  Frag kf[NKS];
  {
    int key = wkey0 + ln;
    key = key < kv_len ? key : kv_len - 1;     // keys past the prefix are computed on a copy and never stored
    const int64_t off = (int64_t)key * a.kv_ss + EPL * g;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) kf[ks] = load_frag_global<T>(kbase + off + ks * KSTEP);
  }
  Cursor t_iss = {qt_first * BQ, hk * a.group, 0};   // next tile to copy
  for (int i = 0; i < DIST; ++i) {
    if (i < n_it) issue(t_iss);
    advance(t_iss);
  }
  f32x16 dk[DB], dv[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) { dk[db][v] = 0.f; dv[db][v] = 0.f; }
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) settle(kf[ks]);
  const lds_addr vrow = Cfg::VT::lane_base(vtile, wave * 32 + ln, g);   // the lane's row of V
  wait_async_tiles();
  __syncthreads();

  // State of the tile in flight.  Operand fragments are read from LDS PF steps ahead of the matrix
  // instruction that consumes them (the compiler, left alone, reads each one right before its use and
  // exposes the LDS latency on every step); the scheduling fences keep that order.
  struct State {
    f32x16 s, dp;
    Frag qa[PF], da[PF], va[PF], tq[PFD], tdo[PFD];
  };
  auto active = [&](const Cursor &t) { return w_active && wkey0 <= seg_off + t.r0 + 31; };

  // Phase B: the accumulators start from the row statistics instead of zero (register v holds row
  // r0 + 8*(v/4) + 4*g + v%4), so that s = q.k - lse/scale and dp = dO.v - delta come out of the matrix
  // pipe ready for p = exp2(c*s) and dS = p*dp.
  // The matrix phases run at a raised wave priority, the vector phase at the default one: when the two waves of a
  // SIMD both have instructions ready, the one feeding the matrix pipe goes first (1.3 % of the kernel, measured).
  auto phase_b = [&](State &z, const Cursor &t) {
    __builtin_amdgcn_s_setprio(2);
    const lds_addr qblock = lds0 + t.stage * Cfg::STAGE_BYTES;   // the dO block lies QT::BYTES behind it
    const lds_addr st = stats0 + (unsigned)(t.stage * Cfg::STAT_BYTES + 16 * g);
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      const f32x4 nl = lds_load<f32x4>(st + 32 * vq);
      const f32x4 nd = lds_load<f32x4>(st + 4 * BQ + 32 * vq);
#pragma unroll
      for (int e = 0; e < 4; ++e) { z.s[4 * vq + e] = nl[e]; z.dp[4 * vq + e] = nd[e]; }
    }
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      rd.nat2(qblock, QT::BYTES, i, z.qa[i], z.da[i]);
      z.va[i] = Cfg::VT::frag(vrow, i);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      z.s = mma(z.qa[ks % PF], kf[ks], z.s);
      z.dp = mma(z.da[ks % PF], z.va[ks % PF], z.dp);
      if (ks + PF < NKS) {
        rd.nat2(qblock, QT::BYTES, ks + PF, z.qa[ks % PF], z.da[ks % PF]);
        z.va[ks % PF] = Cfg::VT::frag(vrow, ks + PF);
      } else {   // the rings drain: start on the operands of phase D
        const int i = ks + PF - NKS;
        rd.tr2(qblock, QT::BYTES, i / DB, i % DB, z.tq[i], z.tdo[i]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Phase C.  Visible iff key <= seg_off + row and row < seg_len, row = r0 + 4g + 8*(v/4) + v%4; blocks that
  // lie wholly below the diagonal and inside the segment (nearly all of them) skip the test.
  auto phase_c = [&](State &z, const Cursor &t) {
    __builtin_amdgcn_s_setprio(0);
    const lds_addr qblock = lds0 + t.stage * Cfg::STAGE_BYTES;
#pragma unroll
    for (int i = PF; i < PFD; ++i) rd.tr2(qblock, QT::BYTES, i / DB, i % DB, z.tq[i], z.tdo[i]);   // rest of phase D's ring
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float p = exp2_fast(z.s[v] * c);
      z.s[v] = p;
      z.dp[v] = p * z.dp[v];
    }
    // Tiles on the diagonal or at the end of the segment: entries above the diagonal and rows past the segment are
    // set to zero afterwards, in a branch that holds nothing else (whatever the exponential made of them, infinity
    // included, is overwritten).  One instance of the arithmetic above keeps p and dS in place: with a masked and an
    // unmasked copy of it the compiler moved all 16 dS registers on every step.
    const bool edge = (wkey0 + 31 > seg_off + t.r0) || (t.r0 + 32 > seg_len);
    if (edge) {
      asm volatile("" ::: "memory");   // keeps this a branch
      const int fl = fresh(lane), fg = fl >> 5;
      const int lo = wkey0 + (fl & 31) - seg_off - t.r0 - 4 * fg;   // need 8*(v/4)+v%4 >= lo
      const int hi = seg_len - t.r0 - 4 * fg;                       // and  8*(v/4)+v%4 <  hi
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int rr = 8 * (v >> 2) + (v & 3);
        if (rr < lo || rr >= hi) {
          z.s[v] = 0.f;
          z.dp[v] = 0.f;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto phase_d = [&](State &z, const Cursor &t) {
    __builtin_amdgcn_s_setprio(2);
    const lds_addr qblock = lds0 + t.stage * Cfg::STAGE_BYTES;
    Frag pf, dsf;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int sl = i / DB, db = i % DB;
      if (db == 0) {
        pf = block_slab<T>(z.s, sl);
        dsf = block_slab<T>(z.dp, sl);
      }
      dv[db] = mma(z.tdo[i % PFD], pf, dv[db]);
      dk[db] = mma(z.tq[i % PFD], dsf, dk[db]);
      if (i + PFD < NV) rd.tr2(qblock, QT::BYTES, (i + PFD) / DB, (i + PFD) % DB, z.tq[i % PFD], z.tdo[i % PFD]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // End of an iteration: the wave's share of the NEXT tile must have landed.  With DIST = 2 the copy issued at the top
  // of this iteration (PER instructions, one more for the statistics on wave 0) belongs to the tile after it and
  // stays in flight across the barrier.
  constexpr int kCopyInsts = AsyncTilePairU<T, BQ, D, NW>::PER;
  auto wait_next_tile = [&](bool issued_this_iteration) {
    if (DIST >= 2 && issued_this_iteration) {
      if (wave < 2 * BQ / 64) wait_async_tiles_but_last<kCopyInsts + 1>();
      else wait_async_tiles_but_last<kCopyInsts>();
    } else {
      wait_async_tiles();
    }
  };
  Cursor cur = {qt_first * BQ, hk * a.group, 0};   // tile of the current iteration
  const bool late = LAG > 0 && wave >= NW / 2;
  if (!late) {
    for (int it = 0; it < n_it; ++it) {
      // the stage this copy overwrites was last read before the barrier that ended the previous iteration
      if (it + DIST < n_it) issue(t_iss);
      advance(t_iss);
      if (active(cur)) {
        State z;
        phase_b(z, cur);
        phase_c(z, cur);
        phase_d(z, cur);
      }
      advance(cur);
      wait_next_tile(it + DIST < n_it);   // this wave's part of tile it+1 has landed
      __syncthreads();
    }
  } else {
    State z;
    Cursor prev = cur;
    for (int it = 0; it < n_it; ++it) {
      if (it + DIST < n_it) issue(t_iss);
      advance(t_iss);
      if (it > 0 && active(prev)) {
        phase_c(z, prev);
        phase_d(z, prev);
      }
      if (active(cur)) phase_b(z, cur);
      prev = cur;
      advance(cur);
      wait_next_tile(it + DIST < n_it);
      __syncthreads();
    }
    if (active(prev)) {
      phase_c(z, prev);
      phase_d(z, prev);
    }
  }

  // Epilogue: acc[key][d] += result, each element touched by exactly one lane of the grid.  In the accumulators a
  // lane holds ONE key and 4-element pieces of its row 32 bytes apart: read-modify-write straight from there would
  // touch 64 different cache lines per instruction.  Each wave therefore passes its 32 x D block through LDS (its
  // own region; rows padded by 16 bytes so that the row-per-lane writes spread over all banks) and updates the
  // accumulators row by row, LPR lanes side by side on one row.
  __syncthreads();   // the late half's last phases still read the tile ring that the regions below overlay
  float *dkb = a.dk_acc + kvoff, *dvb = a.dv_acc + kvoff;
  constexpr int ROWB = QT::DPAD * 4 + 16;           // bytes per staged row
  constexpr int LPR = D / 4;                        // lanes per row (16 bytes each)
  constexpr int RPI = 64 / LPR;                     // rows per instruction
  constexpr int NI = (32 + RPI - 1) / RPI;          // instructions per block
  static_assert(NW * 32 * ROWB <= Cfg::LDS_BYTES, "the epilogue's staging regions must fit the kernel's LDS");
  char *region = smem + wave * (32 * ROWB);
  const int row_in = lane / LPR, col = lane % LPR;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const f32x16(&acc)[DB] = which == 0 ? dk : dv;
    const float mul = which == 0 ? a.scale : 1.f;
    float *base = which == 0 ? dkb : dvb;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int d0 = 32 * db + 8 * vq + 4 * g;
        *reinterpret_cast<f32x4 *>(region + ln * ROWB + d0 * 4) =
            f32x4{acc[db][4 * vq] * mul, acc[db][4 * vq + 1] * mul, acc[db][4 * vq + 2] * mul, acc[db][4 * vq + 3] * mul};
      }
    f32x4 cur[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = i * RPI + row_in, key = wkey0 + r;
      if (row_in < RPI && r < 32 && key < kv_len)
        cur[i] = *reinterpret_cast<const f32x4 *>(base + (int64_t)key * a.kv_ss + 4 * col);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = i * RPI + row_in, key = wkey0 + r;
      if (row_in < RPI && r < 32 && key < kv_len) {
        const f32x4 add = *reinterpret_cast<const f32x4 *>(region + r * ROWB + 16 * col);
        *reinterpret_cast<f32x4 *>(base + (int64_t)key * a.kv_ss + 4 * col) = cur[i] + add;
      }
    }
  }
}

}  // namespace s1f

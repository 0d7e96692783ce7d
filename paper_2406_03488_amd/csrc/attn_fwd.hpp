// Forward of one segment: out = softmax(q k^T / sqrt(D), causal with the diagonal shifted by seg_off) v,
// lse = log-sum-exp of the scaled scores (Section 3.1, Eq. 3, restricted to the segment's rows).
//
// One workgroup (4 waves) owns 64*NC query rows of one head (NC = 1, 2, 3); wave w owns rows 16*NC*w .. +16*NC, NC column
// blocks of 16.  The transposed products are computed so that a lane always holds NC queries (column n of each block) and
// the keys run over registers:
//     S^T[key][q] = sum_d K[key][d] Q[q][d]        A = K from LDS, B = Q (registers)
//     O^T[d][q]  += sum_key V[key][d] P^T[key][q]  A = V read transposed from LDS, B = P^T slab (registers)
// Row maximum and sum are then in-lane reductions; the four lanes of a query meet at the end only.
//
// K/V tiles of 32 keys go from HBM straight into a ring in LDS (TileRing; no register staging, except that fp32 tiles are split
// on the way), with one workgroup barrier per tile.  In fp32 128-row tiles above head_dim 64 are eight waves of 16 rows, two
// to a SIMD (LDS has room for one workgroup): a wave's splitting and waiting runs beside the other's products (four waves
// of 32 rows: 32 heads, 2048 rows behind 8000 keys, head_dim 128 1948 us instead of 1650).
// The loop advances by one tile and is software-pipelined inside each wave: the score product of tile k+1 (matrix
// pipe) is issued together with the operand packing of tile k's probabilities (vector pipe), then the PV product of
// tile k together with the exponentials of tile k+1 (see fwd_step).  A wave walks to the last tile that one of its rows sees
// (see own_tiles); tiles that all of them see run a step without any masking code.
//
// What bounds it: the matrix pipe, at the clock the power limit leaves (head_dim 128: 63-68 % busy at 1.82-1.86 GHz, two
// waves per SIMD).  Per step and wave it runs 16 * NC matrix instructions of 16 cycles against about 12 * NC vector
// instructions and 8 * NC exponentials (two issue slots each), so both have to run under each other, and every operand
// read from LDS should feed as many matrix instructions as registers allow: 48 rows per wave (NC = 3) read a third less
// LDS per product than 32.  32 heads, 4096 rows behind 28672 keys: head_dim 128 1.86 -> 1.65 ms (1110 -> 1250
// TFLOP/s), 80 1.51 -> 1.22 ms, 64 1.17 -> 1.00 ms against 32x32x16 instructions on 32 rows per wave, whole swizzled
// rows in LDS and three waves per SIMD.
#pragma once
#include <type_traits>

#include "attn_plain.hpp"

namespace s1f {

// Lazy rescaling: the running maximum m of a row is raised only when a new tile makes its probabilities
// 2^(s*c - m) large, and the steady loop finds that out from their SUM, which it needs anyway, instead of from their
// maximum: a lane adds up the probabilities of its 8 keys of the tile, and if that sum exceeds 2^kRescaleTau in
// any lane of the wave (infinity included: the exponentials are taken before anyone has looked), the loop is left,
// the tile's row maxima are computed, the rows whose maximum exceeds m by more than kRescaleTau - 3 (a sum over 8
// keys above 2^tau needs one of them above 2^(tau-3)) take it as their new m, O and l are rescaled and the tile's
// probabilities recomputed.  Otherwise every probability is at most 2^kRescaleTau, which fp32 sums and bf16
// operands hold without loss.  The accumulator rescale (a pass over every O register) and the maximum (a chain of
// its own through all scores, plus lane exchanges) thereby leave the steady loop.
constexpr float kRescaleTau = 8.0f;
constexpr float kRescaleLimit = 256.0f;   // 2^kRescaleTau

// Masks the scores of rows 16*rb.. of a tile that crosses the diagonal.
//   ahead = (absolute row of the wave's first query) - (first key of the tile)
template <int NC> S1F_DEV void fwd_mask(f32x4 (&s)[2][NC], int rb, int ahead) {
  const int lane = lane_id(), lim = ahead + (lane & 15) - 4 * (lane >> 4);
  float hidden = -INFINITY;
  asm volatile("" : "+v"(hidden));   // made here, not kept in a register across the loop
#pragma unroll
  for (int cb = 0; cb < NC; ++cb)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (16 * rb + v > lim + 16 * cb) s[rb][cb][v] = hidden;
}

// Row maxima of a tile in log2 units (each lane gets the maxima of its NC queries' 32 scores).
template <int NC> S1F_DEV void fwd_row_max(const f32x4 (&s)[2][NC], float (&mx)[NC], float c) {
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    float x = s[0][cb][0];
#pragma unroll
    for (int i = 1; i < 8; ++i) x = fmaxf(x, s[i >> 2][cb][i & 3]);
    mx[cb] = max_over_rows(x) * c;
  }
}

// Probabilities of a tile from its scores, against the running maximum m (log2 units): p = 2^(s*c - m); rs = the
// sums over this lane's 8 keys.
template <int NC> S1F_DEV void fwd_probs(f32x4 (&p)[2][NC], const f32x4 (&s)[2][NC], const float (&m)[NC], float c, float (&rs)[NC]) {
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    rs[cb] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float x = exp2_fast(fmaf(s[i >> 2][cb][i & 3], c, -m[cb]));
      p[i >> 2][cb][i & 3] = x;
      rs[cb] += x;
    }
  }
}

// A tile that sets the maxima of its rows: the running maximum, finite also where every score is minus infinity (which then has weight
// zero), and probabilities whose products are rounded as those in the maxima are, so that no exponent is above zero.  (A fused product differs
// from a rounded one by up to half a spacing of m: from scores of 2^31 on, as a lowest value in K makes them, that is 2^7 and more, and
// p infinite.)
template <int NC> S1F_DEV void fwd_finite_max(const f32x4 (&s)[2][NC], float (&mx)[NC], float c) {
  fwd_row_max(s, mx, c);
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) mx[cb] = fmaxf(mx[cb], -kMaxFloat);
}
template <int NC> S1F_DEV void fwd_probs_of_max(f32x4 (&p)[2][NC], const f32x4 (&s)[2][NC], const float (&m)[NC], float c, float (&rs)[NC]) {
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    rs[cb] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float t = s[i >> 2][cb][i & 3] * c;
      settle(t);
      const float x = exp2_fast(t - m[cb]);
      p[i >> 2][cb][i & 3] = x;
      rs[cb] += x;
    }
  }
}

// Scores of a tile: s[rb][cb] = K[rows 16*rb..] Q[cb]^T   (outside the loop, which uses fwd_step)
template <typename M, int NC>
S1F_DEV void fwd_scores(f32x4 (&s)[2][NC], const typename M::RowOp (&q)[NC], const M &rd, lds_addr ktile) {
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) s[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const typename M::Nat ka = rd.nat_at(ktile);
#pragma unroll
  for (int i = 0; i < M::NN; ++i) {
    const typename M::Frag kf = M::nat(ka, i);
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) s[i / M::NK][cb] = M::mma_nat(i, kf, q[cb], s[i / M::NK][cb]);
    __builtin_amdgcn_sched_barrier(0);   // one operand at a time: reading all of them ahead costs the loop registers
  }
}

// K operands read ahead: those of tile k+2 that the next step begins with are read at the end of this one, so that no
// step starts by waiting for LDS.
template <typename M> struct KRing {
  static constexpr int N = M::NN < 4 ? M::NN : 4;
  typename M::Frag f[N];
  S1F_DEV void fill(const typename M::Nat &ka) {
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] = M::nat(ka, i);
  }
};

// One pipelined step over tile k, whose probabilities (against m) are in `p` and already counted in l:
//   phase 1   sn = scores of tile k+1, first its upper 16 keys, then its lower 16 (matrix pipe)
//             ||  p packed into operand slabs, then the probabilities of the upper 16 keys (vector pipe)
//   phase 2   O += P V of tile k (matrix pipe)  ||  the probabilities of the lower 16 keys, and all their sums rs
// The probabilities of tile k+1, p = 2^(sn*c - m), are computed against the CURRENT m, before anyone knows whether m
// has to be raised for them: the caller looks at rs afterwards (see kRescaleTau) and, in the rare case that it must
// raise m, rescales O and l and computes scores and p of tile k+1 again (its keys are still in the ring); otherwise it
// adds rs to l.  That way p takes the registers of sn, element by element, and the loop carries it there.
// The order is pinned slot by slot (one operand, its NC matrix instructions, its share of the vector work): two waves
// share a SIMD, and left alone the compiler puts LDS reads right before their use and the exponentials in heaps.
//   MASK: tile k+1 may cross the diagonal of the wave's rows; ahead_next: see fwd_mask
//   hidden (without a next tile): column blocks, from the first on, that tile k is wholly hidden from (never the last)
//   AHEAD: the first operands of ktile_after are read at the end (TileRing::AHEAD)
//   work(slot, slots): the share of a slot in what else the wave has to do in the step
template <typename M, bool HAS_NEXT, bool MASK, bool AHEAD, int NC, typename F>
S1F_DEV void fwd_step(f32x4 (&p)[2][NC], f32x4 (&o)[NC][M::DB], const float (&m)[NC], float (&rs)[NC],
                      const typename M::RowOp (&q)[NC], const M &rd, KRing<M> &kr, lds_addr ktile_next, lds_addr ktile_after,
                      lds_addr vtile, float c, int ahead_next, int hidden, F work) {
  typedef typename M::Frag Frag;
  constexpr int PK = KRing<M>::N, PV = M::NT < 3 ? M::NT : 3, NK = M::NK, NN = M::NN, NT = M::NT;
  __builtin_amdgcn_s_setprio(1);   // of two ready waves the one in phase 1, which has little else to issue, feeds the matrix pipe
  typename M::Slab pf[NC];
  Frag vf[PV];
  f32x4 sn[2][NC];
  const typename M::Tr va = rd.tr_at(vtile);
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) rs[cb] = 0.f;
  auto pack = [&](int cb) {
    pf[cb] = M::slab(p[0][cb], p[1][cb]);
    M::settle_slab(pf[cb]);
  };
  auto prob = [&](int x) { return p[x / (4 * NC)][(x >> 2) % NC][x & 3]; };
  auto probs = [&](int x0, int x1) {   // probabilities x0 .. x1-1 of the tile's 8 * NC per lane
#pragma unroll
    for (int x = x0; x < x1; ++x) {
      const int cb = (x >> 2) % NC;
      const float t = fmaf(sn[x / (4 * NC)][cb][x & 3], c, -m[cb]);
      if (x > 0) rs[((x - 1) >> 2) % NC] += prob(x - 1);   // one behind: its result is not ready at once
      float y = exp2_fast(t);
      settle(y);
      p[x / (4 * NC)][cb][x & 3] = y;
    }
  };
  if (HAS_NEXT) {
    const typename M::Nat ka = rd.nat_at(ktile_next);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) sn[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NN; ++i) {
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        sn[i / NK][cb] = M::mma_nat(i, kr.f[i % PK], q[cb], sn[i / NK][cb]);
        if (cb + 1 == NC) {
          if (MASK && i + 1 == NK) fwd_mask(sn, 0, ahead_next);
          if (MASK && i + 1 == NN) fwd_mask(sn, 1, ahead_next);
          if (i + PK < NN) kr.f[i % PK] = M::nat(ka, i + PK);
          if (i + PV >= NN) vf[i + PV - NN] = M::tr(va, i + PV - NN);
        }
        // vector work under this matrix instruction (of the other row half: this one's results are still in the pipe)
        const int w = i * NC + cb, W = NK * NC;
        if (w < NC) pack(w);
        if (w >= W) probs(4 * NC * (w - W) / W, 4 * NC * (w - W + 1) / W);
        work(w, (NN + NT) * NC);
        end_slot<M>();
      }
    }
  } else {
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) pack(cb);
#pragma unroll
    for (int i = 0; i < PV; ++i) vf[i] = M::tr(va, i);
  }
  __builtin_amdgcn_s_setprio(0);
  const typename M::Nat kb = rd.nat_at(AHEAD ? ktile_after : vtile);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      if (HAS_NEXT || cb + 1 == NC || cb >= hidden) M::mma_tr(i, vf[i % PV], pf[cb], o[cb]);
      if (cb + 1 == NC) {
        if (i + PV < NT) vf[i % PV] = M::tr(va, i + PV);
        if (HAS_NEXT && AHEAD && i + PK >= NT) kr.f[i + PK - NT] = M::nat(kb, i + PK - NT);
      }
      const int w = i * NC + cb, W = NT * NC;
      if (HAS_NEXT) probs(4 * NC + 4 * NC * w / W, 4 * NC + 4 * NC * (w + 1) / W);
      if (HAS_NEXT) work(NN * NC + w, (NN + NT) * NC);
      end_slot<M>();
    }
  }
  if (HAS_NEXT) rs[NC - 1] += prob(8 * NC - 1);
}

// fp32: the factor of the planes is taken out of a wave's accumulators; if they are not all finite, its rows (16*NC from row0 on) are
// computed again in plain arithmetic.  qb: row 0 of the segment; kbase, vbase: first of the `keys` keys that the wave has walked, from
// which seg_off counts.
template <typename T, int D, int NC>
S1F_DEV void fwd_finish_fp32(const AttnArgs &a, const T *qb, const T *kbase, const T *vbase, int row0, int seg_off, int keys, float c,
                             f32x4 (&o)[NC][Mat<T, D>::DB], float (&m)[NC], float (&l)[NC]) {
  typedef Mat<T, D> M;
  if constexpr (sizeof(T) == 4) {
    float bad = 0.f;
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      bad = fmaf(l[cb], 0.f, bad);
#pragma unroll
      for (int db = 0; db < M::DB; ++db) {
        bad = add_if_not_finite(o[cb][db], bad);
        o[cb][db] *= 1.f / M::UP;
      }
    }
    if (__builtin_expect(any_not_finite(bad), 0)) {
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        const int r_last = row0 + 16 * cb + 15, last = seg_off + (r_last < a.seg_len ? r_last : a.seg_len - 1);
        const int pl = lane_id(), r = row0 + 16 * cb + (pl & 15), rc = r < a.seg_len ? r : a.seg_len - 1;
        fwd_plain<D>(qb + (int64_t)rc * a.q_ss, kbase, vbase, a.kv_ss, seg_off + rc, last < keys ? last + 1 : keys,
                     c * (M::UP * M::UP), pl >> 4, o[cb], m[cb], l[cb]);
        if (pl >= 16) l[cb] = 0.f;   // (the sum over the row's four lanes follows)
      }
    }
  }
}

// Where the main loop lies within 32 bytes of code decides about up to 5 % of a launch (instructions are fetched in such pieces), and what
// stands in front of it would move it: words of padding behind a multiple of 32 bytes, each instance's best of eight places (fp32: all the same).
// With the loop of 32 heads, head_dim 80, 128-row tiles at 0, 8, 16, 24 bytes: 2406 first rows 47.4 46.9 46.4 46.9 us, 1757 behind 6435 keys
// 155.4 156.0 151.9 153.3; 64/8 heads, 128, 192 rows, 2626 behind 128446, at 4, 12, 20, 28: 8555 8574 8685 8456; 64-row tiles, by words 0 .. 7: 8
// heads, 128, 2785 behind 4881 106.8 108.7 110.3 110.5 107.8 110.7 111.4 108.1.
template <typename T, int D, int NC> constexpr int kLoopPad = sizeof(T) == 2 && NC == 1 ? (D == 128 ? 0 : D == 80 ? 4 : 2) : 3;

// REST: the second launch, over the rows of units that the first left over (an instance of its own: in the 64-row kernel itself
// the decision cost 2 to 6 % of launches of 30 to 300 us)
template <typename T, int D, int NC, int OCC, int WAVES, bool REST = false>
__global__ void __launch_bounds__(64 * WAVES, OCC) seg_attn_fwd_kernel(const AttnArgs a) {
  typedef Mat<T, D> M;
  typedef TileRing<T, D, WAVES> Ring;
  constexpr int DB = M::DB, BM = 16 * NC * WAVES, BN = 32;

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, j = lane >> 4, n = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int seg_len = a.seg_len;
  UnitChunk uc;
  int qt, bh, row0;
  if constexpr (REST) {   // a chunk is a tile of BM of the unit's a.bm rows
    const int cut = a.n_split * a.n_split_units;
    if ((int)blockIdx.x < cut) {
      uc = split_unit(blockIdx.x + a.first_id, a.first_id, a.n_split, a.n_split_units, a.by_split_units);
      decode_workgroup(uc.unit, a.by_tiles, a.n_bh, a.by_xcd, a.tile_major, qt, bh);
      row0 = (a.n_tiles - 1 - qt) * a.bm + uc.chunk * BM;
    } else {
      decode_workgroup(blockIdx.x - cut, a.by_rag, a.n_bh, a.by_xcd, 1, qt, bh);
      row0 = a.n_tiles * a.bm + qt * BM;
    }
    if (row0 >= seg_len) return;
    uc = UnitChunk{0, 0, 1, -1};
  } else {
    uc = split_unit(blockIdx.x, a.n_whole, a.n_split, a.n_split_units, a.by_split_units);
    decode_workgroup(uc.unit, a.by_tiles, a.n_bh, a.by_xcd, a.tile_major, qt, bh);
    row0 = (a.n_tiles - 1 - qt) * BM;   // later (heavier) row tiles are scheduled first
  }
  int b, h;
  div_mod(bh, a.by_heads, b, h);
  const int hk = div(h, a.by_group);
  const int wrow0 = row0 + wave * 16 * NC;
  const int last_row = (row0 + BM < seg_len ? row0 + BM : seg_len) - 1;
  // This workgroup's 32-key tiles: all that hold keys 0 .. seg_off+last_row, or one chunk of them.  From here on
  // keys are counted from the chunk's first key: seg_off and kv_len are relative to it.
  int kt0, kt1;
  chunk_range(uc, a.by_split, (a.seg_off + row0) / BN, (a.seg_off + last_row) / BN + 1, kt0, kt1);
  const int seg_off = a.seg_off - BN * kt0, kv_len = seg_off + seg_len;
  const int n_kt = kt1 - kt0;
  if (n_kt <= 0) {   // more chunks than this unit has whole tiles: a result that the merge gives no weight
    float *po = a.part + (int64_t)uc.slot * (BM * D);
    float *pml = a.part_ml + (int64_t)uc.slot * (BM * 2);
    for (int i = tid; i < BM * D; i += 64 * WAVES) po[i] = 0.f;
    for (int i = tid; i < BM; i += 64 * WAVES) {
      pml[2 * i] = -INFINITY;
      pml[2 * i + 1] = 0.f;
    }
    return;
  }

  const T *qb = reinterpret_cast<const T *>(a.q) + b * a.q_sb + h * a.q_sh;
  const int64_t kv_first = b * a.kv_sb + hk * a.kv_sh + (int64_t)(BN * kt0) * a.kv_ss;
  const T *kbase = reinterpret_cast<const T *>(a.k) + kv_first;
  const T *vbase = reinterpret_cast<const T *>(a.v) + kv_first;

  Ring ring;
  ring.init(kbase, vbase, a.kv_ss, n_kt, kv_len, to_lds_addr(smem), wave, lane);
  ring.issue(0);
  ring.issue(1);

  typename M::RowOp q[NC];
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    int r = wrow0 + 16 * cb + n;
    r = r < seg_len ? r : seg_len - 1;   // rows past the segment are computed on a copy and never stored
    M::load_row(q[cb], qb + (int64_t)r * a.q_ss, j);
  }
#pragma unroll
  for (int cb = 0; cb < NC; ++cb)
#pragma unroll
    for (int i = 0; i < M::NK; ++i) settle(q[cb].f[i]);

  f32x4 o[NC][DB];
#pragma unroll
  for (int cb = 0; cb < NC; ++cb)
#pragma unroll
    for (int db = 0; db < DB; ++db) o[cb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c = uniform(a.scale * kLog2e / (M::UP * M::UP));
  M rd;
  rd.init(lane);

  wait_async_tiles();
  ring.issue(2);
  ring.issue(3);
  __syncthreads();
  f32x4 s[2][NC];
  float m[NC], l[NC], mx[NC], rs[NC];
  fwd_scores<M, NC>(s, q, rd, ring.st[0]);
  if (BN - 1 > seg_off + wrow0) {
    fwd_mask(s, 0, seg_off + wrow0);
    fwd_mask(s, 1, seg_off + wrow0);
  }
  fwd_finite_max(s, m, c);
  fwd_probs_of_max(s, s, m, c, l);  // from here on `s` holds the probabilities of the current tile, l their sums

  int k = 0;   // current tile
  if (wrow0 >= seg_len) {   // no rows of its own: the wave only copies its share of the tiles
    for (; k + 1 < n_kt; ++k, ring.end_step()) ring.template begin_step<false>(n_kt - 1 - k);
    return;
  }
  KRing<M> kr;
  if (Ring::AHEAD) kr.fill(rd.nat_at(ring.st[1]));
  auto steady = [&](auto mask, auto whole) {
    constexpr bool MASK = decltype(mask)::value, WHOLE = decltype(whole)::value;
    ring.template begin_step<WHOLE>(n_kt - 1 - k);
    if (!Ring::AHEAD) kr.fill(rd.nat_at(ring.st[1]));
    const int ahead = seg_off + wrow0 - BN * (k + 1);
    fwd_step<M, true, MASK, Ring::AHEAD, NC>(s, o, m, rs, q, rd, kr, ring.st[1], ring.st[2],
                                ring.st[0] + Tile32<T, D>::BYTES, c, ahead, 0,
                                [&](int slot, int slots) { ring.template work<WHOLE>(slot, slots); });
    ++k;
    ring.end_step();
    bool raise = false;
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) raise = raise || !(rs[cb] <= kRescaleLimit);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
      asm volatile("" ::: "memory");
      fwd_scores<M, NC>(s, q, rd, ring.st[0]);
      if (MASK) {
        fwd_mask(s, 0, ahead);
        fwd_mask(s, 1, ahead);
      }
      fwd_finite_max(s, mx, c);
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        const float m_up = mx[cb] > m[cb] + (kRescaleTau - 3.f) ? mx[cb] : m[cb];
        const float alpha = exp2_fast(m[cb] - m_up);   // exactly 1 for rows that keep their maximum
        m[cb] = m_up;
        l[cb] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[cb][db] = o[cb][db] * alpha;
      }
      fwd_probs_of_max(s, s, m, c, rs);   // the current tile's probabilities again, against the raised maxima
    }
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) l[cb] += rs[cb];
  };
  // Tiles that every row of the wave sees in full, first while there is a whole tile to copy (no branches in the step),
  // then those on its diagonal.  A branch around the mask inside one loop would part the step where its two phases overlap.
  const std::integral_constant<bool, true> yes;
  const std::integral_constant<bool, false> no;
  const int n_own = own_tiles<BN>(seg_off, wrow0, wrow0 + 16 * NC < seg_len ? wrow0 + 16 * NC : seg_len, n_kt);
  int n_full = (seg_off + wrow0 + 1) / BN;
  n_full = n_full < n_kt - 1 ? n_full : n_kt - 1;
  const int n_fast = n_full < n_kt - 4 ? n_full : n_kt - 4;
  asm volatile(".p2align 5\n\t.fill %0, 4, 0xbf800000" ::"n"(kLoopPad<T, D, NC>));   // (s_nop 0)
  while (k + 1 < n_fast) steady(no, yes);
  while (k + 1 < n_full) steady(no, no);
  while (k + 1 < n_own) steady(yes, no);
  // the wave's last tile: no next scores to compute.  Waves that have more tiles to walk are let into their next step first.
  if (k + 1 < n_kt) ring.template begin_step<false>(n_kt - 1 - k);
  fwd_step<M, false, false, Ring::AHEAD, NC>(s, o, m, rs, q, rd, kr, ring.st[0], ring.st[0], ring.st[0] + Tile32<T, D>::BYTES, c, 0,
                                hidden_blocks<BN>(seg_off + wrow0, n_own), [](int, int) {});
  if (k + 1 < n_kt) {   // its share of the others' tiles
    ring.end_step();
    for (++k; k + 1 < n_kt; ++k, ring.end_step()) ring.template begin_step<false>(n_kt - 1 - k);
  }

  fwd_finish_fp32<T, D, NC>(a, qb, kbase, vbase, wrow0, seg_off, BN * n_kt, c, o, m, l);
  if (uc.slot >= 0) {   // a chunk: unnormalised output rows, running maximum and row sum go to the workspace
    float *po = a.part + (int64_t)uc.slot * (BM * D);
    float *pml = a.part_ml + (int64_t)uc.slot * (BM * 2);
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      const float lt = sum_over_rows(l[cb]);
      const int rl = wave * 16 * NC + 16 * cb + n;   // row within the unit
#pragma unroll
      for (int x = 0; x < DB; ++x) *reinterpret_cast<f32x4 *>(po + rl * D + M::quad_d0(x, j)) = M::quad(o[cb], x);
      if (j == 0) {
        pml[2 * rl] = m[cb];
        pml[2 * rl + 1] = lt;
      }
    }
    return;
  }
  T *ob = reinterpret_cast<T *>(a.out_w) + b * a.q_sb + h * a.q_sh;
  float *lse = a.lse + ((int64_t)b * a.n_q_heads + h) * seg_len;
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    const float lt = sum_over_rows(l[cb]);
    const float inv = 1.f / lt;
    const int r = wrow0 + 16 * cb + n;
    if (r < seg_len) {
      T *orow = ob + (int64_t)r * a.q_ss;
#pragma unroll
      for (int x = 0; x < DB; ++x) {
        const f32x4 y = M::quad(o[cb], x) * inv;
        store4<T>(orow + M::quad_d0(x, j), y[0], y[1], y[2], y[3]);
      }
      if (j == 0) lse[r] = (m[cb] + __builtin_amdgcn_logf(lt)) * kLn2;
    }
  }
}

// Merges the chunks of the units that seg_attn_fwd_kernel cut along the keys: with m_c, l_c, o_c the running
// maximum (log2 units), row sum and unnormalised output row of chunk c,
//   m = max_c m_c,  l = sum_c l_c 2^(m_c - m),  out = sum_c o_c 2^(m_c - m) / l,  lse = (m + log2 l) ln 2.
// A thread handles 4 consecutive head_dim elements of one row; a workgroup MergeRows<D>::RG rows of one split unit
// (grid: split units x groups of RG rows).  All chunk loads of a thread are independent of each other.
template <int D> struct MergeRows {
  static constexpr int C4 = D / 4;          // threads per row
  static constexpr int RG = 256 / C4;       // rows per workgroup
  __host__ __device__ static constexpr int groups(int bm) { return (bm + RG - 1) / RG; }
};
// MC: most chunks this instance merges (loads of all of them are in flight together; more of them than there are cost
// registers and with them waves: at 16 for a cut into 2, 256 units of 128 rows and head_dim 128 took 14 us instead of 8).
template <typename T, int D, int MC>
__global__ void __launch_bounds__(256) seg_attn_fwd_merge_kernel(const AttnArgs a) {
  typedef MergeRows<D> MR;
  const int BM = a.bm;
  int unit, rg;
  div_mod(blockIdx.x, a.by_groups, unit, rg);
  const int rl = rg * MR::RG + (int)threadIdx.x / MR::C4, c4 = (int)threadIdx.x % MR::C4;
  int qt, bh;
  decode_workgroup(a.n_whole + unit, a.by_tiles, a.n_bh, a.by_xcd, a.tile_major, qt, bh);
  qt = a.n_tiles - 1 - qt;
  int b, h;
  div_mod(bh, a.by_heads, b, h);
  const int r = qt * BM + rl, S = a.n_split;
  if ((int)threadIdx.x >= MR::RG * MR::C4 || rl >= BM || r >= a.seg_len) return;
  int slot0, slot_step;
  chunk_slots(unit, a.n_split_units, slot0, slot_step);
  const float *po = a.part + (int64_t)slot0 * (BM * D) + rl * D + 4 * c4;
  const float *pml = a.part_ml + (int64_t)slot0 * (BM * 2) + 2 * rl;
  f32x2 ml[MC];
  f32x4 oc[MC];
#pragma unroll
  for (int c = 0; c < MC; ++c) {   // past the last chunk: that one again, without weight
    const int64_t at = (int64_t)(c < S ? c : S - 1) * slot_step;
    ml[c] = *reinterpret_cast<const f32x2 *>(pml + at * (BM * 2));
    oc[c] = *reinterpret_cast<const f32x4 *>(po + at * (BM * D));
  }
  float m = ml[0][0];
#pragma unroll
  for (int c = 1; c < MC; ++c) m = fmaxf(m, ml[c][0]);
  float l = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < MC; ++c) {
    const float w = exp2_fast(ml[c][0] - m);
    if (c < S) {
      l += w * ml[c][1];
      acc += w * oc[c];
    }
  }
  const float inv = 1.f / l;
  T *ob = reinterpret_cast<T *>(a.out_w) + b * a.q_sb + h * a.q_sh;
  store4<T>(ob + (int64_t)r * a.q_ss + 4 * c4, acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
  if (c4 == 0) a.lse[((int64_t)b * a.n_q_heads + h) * a.seg_len + r] = (m + __builtin_amdgcn_logf(l)) * kLn2;
}

}  // namespace s1f

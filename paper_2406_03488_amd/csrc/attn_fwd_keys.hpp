// Forward of calls with few rows: a workgroup owns 16*NC rows of one head and its W waves share the KEYS among them, each walking
// its part of them alone; their results meet in LDS in the end.  (In seg_attn_fwd_kernel waves own rows of their own and walk all keys
// of the unit together; where a call has few units, most of the chip idles for the length of a walk, or units are cut along the keys over
// workgroups, whose results pass through memory and a second kernel.)
//
// Products as there, on a tile of 32 keys in LDS that is the wave's own.  Nothing is shared between waves before the end, so there is no
// barrier in the loop; while a wave waits for its tile, the others on its SIMD compute.
// Bound by the latency of a step, and in long walks by what a compute unit reads from the L2: every unit of 16*NC rows reads all keys
// itself, at 116 GB/s per compute unit of 2/1 heads, D 64, 511 rows behind 15830 keys (64 bytes a clock are 154), 37 to 60 in calls of 6 to
// 17 us, with the matrix pipe 7 to 20 % busy (profiles/forward_by_keys_kernel_trace_and_counters.txt).  Calls in us, row tiles / by
// keys: bf16, 4 heads, 256 rows behind 768 keys, D 64 9.6 / 6.4, D 128 11.2 / 9.2; 2 x 8/2 heads, 340 behind 1017, D 64 14.4 / 10.3, D 80
// 16.1 / 11.4; without a workspace 2/1 heads, 511 behind 15830, D 64 148 / 35, fp32 492 / 167.
#pragma once
#include "attn_fwd.hpp"

namespace s1f {

// A wave's tile of 32 keys in LDS: K and V, one stage of each.  The next K is asked for when the scores of the current one are
// computed, the next V behind the second product.  (Every tile goes through LDS: a lane's operand is 16 bytes of a row of its own, and
// loads of such operands straight into registers reached 57 GB/s per compute unit, half of what the copies do: 16341 keys, D 64, 32 rows
// 73 us.)
template <typename T, int D> struct WaveTiles;
template <int D> struct WaveTiles<bf16_t, D> {
  typedef Mat<bf16_t, D> M;
  typedef Tile32<bf16_t, D> TL;
  static constexpr int BYTES = 2 * TL::BYTES, COPIES = 2 * TL::NP;   // copies of one tile
  TilePairCopy<bf16_t, D> copy[2];   // rows 16*h .. +15 of a tile
  lds_addr lds;
  typename M::Nat ka;
  S1F_DEV void init(lds_addr at, const M &rd, int lane, int64_t stride) {
    copy[0].init(0, lane, stride);
    copy[1].init(1, lane, stride);
    lds = at;
    ka = rd.nat_at(at);
  }
  // `left` rows (at least one) are left from the tile's first on
  S1F_DEV void load_k(const bf16_t *k, int64_t stride, int left) const {
#pragma unroll
    for (int h = 0; h < 2; ++h) copy[h].issue(k, k, stride, left, left, lds, h);
  }
  S1F_DEV void load_v(const bf16_t *v, int64_t stride, int left) const {
#pragma unroll
    for (int h = 0; h < 2; ++h) copy[h].issue(v, v, stride, left, left, lds + TL::BYTES, h);
  }
  // K was asked for before V
  S1F_DEV void begin_step() { wait_async_tiles_but_last<COPIES>(); }
  S1F_DEV void after_scores(bool more, const bf16_t *k, const bf16_t *, int64_t stride, int left) {
    if (more) load_k(k, stride, left);
  }
  S1F_DEV void before_product(bool more) {
    if (more) wait_async_tiles_but_last<COPIES>();   // (the next K)
    else wait_async_tiles();
  }
  S1F_DEV void end_step(bool more, const bf16_t *v, int64_t stride, int left) {
    if (more) load_v(v, stride, left);
  }
  S1F_DEV typename M::Frag key(int h, int ks) const { return M::nat(ka, h * M::NK + ks); }
  S1F_DEV lds_addr v_tile() const { return lds + TL::BYTES; }
};
// fp32: both through registers, K straight into operands (a lane's 32 bytes of a row of its own, split where they are used; loads of that
// kind reach half the rate of the copies, but splitting takes longer), V split when it is written to LDS.
template <int D> struct WaveTiles<float, D> {
  typedef Mat<float, D> M;
  static constexpr int BYTES = Tile32<float, D>::BYTES;
  f32x4 k[2][M::NK][2];
  SplitPairCopy<D, 4> v[2];
  lds_addr lds;
  int n, j;
  S1F_DEV void init(lds_addr at, const M &, int lane, int64_t stride) {
    v[0].init(0, lane, stride);
    v[1].init(1, lane, stride);
    lds = at;
    n = lane & 15;
    j = lane >> 4;
  }
  S1F_DEV void load_k(const float *k0, int64_t stride, int left) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 16 * h + n;
      const float *row = k0 + (int64_t)(r < left ? r : left - 1) * stride;
#pragma unroll
      for (int i = 0; i < M::NK; ++i) {
        const f32x4 *at = reinterpret_cast<const f32x4 *>(row + 32 * i + (i < M::NKS ? 8 : 4) * j);
        k[h][i][0] = at[0];
        k[h][i][1] = i < M::NKS ? at[1] : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
  S1F_DEV void load_v(const float *p, int64_t stride, int left) {
#pragma unroll
    for (int h = 0; h < 2; ++h) v[h].load(p, p, stride, left, left, h);
  }
  S1F_DEV void begin_step() {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < SplitPairCopy<D, 4>::NI; ++i) v[h].write(i, lds);
  }
  S1F_DEV void after_scores(bool more, const float *k0, const float *v0, int64_t stride, int left) {
    if (!more) return;
    load_k(k0, stride, left);
    load_v(v0, stride, left);
  }
  S1F_DEV void before_product(bool) {}
  S1F_DEV void end_step(bool, const float *, int64_t, int) {}
  S1F_DEV typename M::Frag key(int h, int ks) const { return split3(k[h][ks][0] * kUp, k[h][ks][1] * kUp); }
  S1F_DEV lds_addr v_tile() const { return lds; }
};

template <typename T, int D, int NC, int W> struct FwdKeysCfg {
  static constexpr int ROWS = 16 * NC;
  static constexpr int WAVE_BYTES = WaveTiles<T, D>::BYTES;
  static constexpr int O_ROW = D + 4;                          // floats per row of a partial result (16 lanes side by side: other banks)
  static constexpr int ML_AT = W * ROWS * O_ROW * 4;           // running maxima and sums, behind the partial results
  static constexpr int MERGE_BYTES = ML_AT + W * ROWS * 8;
  static constexpr int LDS_BYTES = W * WAVE_BYTES > MERGE_BYTES ? W * WAVE_BYTES : MERGE_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a compute unit");
};

// Every LDS read of the wave so far has returned: what it has read may be overwritten by a copy.
S1F_DEV void lds_reads_done() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

template <typename T, int D, int NC, int W>
__global__ void __launch_bounds__(64 * W, (W + 3) / 4) seg_attn_fwd_kernel_by_keys(const AttnArgs a) {
  typedef Mat<T, D> M;
  typedef FwdKeysCfg<T, D, NC, W> Cfg;
  constexpr int DB = M::DB, BN = 32, ROWS = Cfg::ROWS, NK = M::NK, NT = M::NT;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, j = lane >> 4, n = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int qt, bh;
  decode_workgroup(blockIdx.x, a.by_tiles, a.n_bh, a.by_xcd, a.tile_major, qt, bh);
  int b, h;
  div_mod(bh, a.by_heads, b, h);
  const int hk = div(h, a.by_group);
  const int seg_len = a.seg_len, row0 = (a.n_tiles - 1 - qt) * ROWS;
  const int last_row = (row0 + ROWS < seg_len ? row0 + ROWS : seg_len) - 1;
  // The wave's 32-key tiles.  From here on keys are counted from its first one.
  int kt0, kt1;
  chunk_range(UnitChunk{0, wave, W, 0}, a.by_split, (a.seg_off + row0) / BN, (a.seg_off + last_row) / BN + 1, kt0, kt1);
  const int seg_off = a.seg_off - BN * kt0, kv_len = seg_off + seg_len, n_kt = kt1 - kt0;
  const T *qb = reinterpret_cast<const T *>(a.q) + b * a.q_sb + h * a.q_sh;
  const int64_t kv_first = b * a.kv_sb + hk * a.kv_sh + (int64_t)(BN * kt0) * a.kv_ss;
  const T *kbase = reinterpret_cast<const T *>(a.k) + kv_first, *vbase = reinterpret_cast<const T *>(a.v) + kv_first;

  M rd;
  rd.init(lane);
  WaveTiles<T, D> tiles;
  tiles.init(to_lds_addr(smem) + wave * Cfg::WAVE_BYTES, rd, lane, a.kv_ss);
  if (n_kt > 0) {
    tiles.load_k(kbase, a.kv_ss, kv_len);
    tiles.load_v(vbase, a.kv_ss, kv_len);
  }
  typename M::RowOp q[NC];
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    const int r = row0 + 16 * cb + n;
    M::load_row(q[cb], qb + (int64_t)(r < seg_len ? r : seg_len - 1) * a.q_ss, j);   // (rows past the segment: a copy, never stored)
  }
  f32x4 o[NC][DB];
  float m[NC], l[NC], mx[NC], rs[NC];
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    m[cb] = -INFINITY;
    l[cb] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) o[cb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float c = uniform(a.scale * kLog2e / (M::UP * M::UP));
#pragma unroll
  for (int cb = 0; cb < NC; ++cb)
#pragma unroll
    for (int i = 0; i < NK; ++i) settle(q[cb].f[i]);
  const int hidden = hidden_blocks<BN>(seg_off + row0, n_kt);   // (of the last tile of the unit, which the last wave walks)

  // (place of the loop: see kLoopPad.  Of eight, 3 and 4 words are the fastest: bf16, D 64, 8 heads, 428 rows behind 443 keys, 0 .. 7 words 6.38 6.41 6.36
  // 6.29 6.27 6.28 6.33 6.34 us; other instances within 1 %)
  asm volatile(".p2align 5\n\t.fill 4, 4, 0xbf800000");
  for (int k = 0; k < n_kt; ++k) {
    const bool more = k + 1 < n_kt;
    const int64_t next = (int64_t)(BN * (k + 1)) * a.kv_ss;
    const int left = kv_len - BN * (k + 1);
    tiles.begin_step();
    f32x4 s[2][NC];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        const typename M::Frag kf = tiles.key(rb, ks);
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cb = 0; cb < NC; ++cb) s[rb][cb] = M::mma_nat(ks, kf, q[cb], ks ? s[rb][cb] : zero);
      }
    lds_reads_done();   // of the tile that the next K overwrites
    tiles.after_scores(more, kbase + next, vbase + next, a.kv_ss, left);
    const int ahead = seg_off + row0 - BN * k;
    if (BN - 1 > ahead) {
      fwd_mask(s, 0, ahead);
      fwd_mask(s, 1, ahead);
    }
    // The first tile of a wave has a key that each row sees, but with any score (keys that are to have no weight may fill it); from then
    // on maxima are raised as in seg_attn_fwd_kernel.
    f32x4 p[2][NC];
    if (k == 0) {
      fwd_finite_max(s, m, c);
      fwd_probs_of_max(p, s, m, c, rs);
    } else {
      fwd_probs(p, s, m, c, rs);
    }
    bool raise = false;
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) raise = raise || !(rs[cb] <= kRescaleLimit);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
      fwd_finite_max(s, mx, c);
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        const float m_up = mx[cb] > m[cb] + (kRescaleTau - 3.f) ? mx[cb] : m[cb];
        const float alpha = exp2_fast(m[cb] - m_up);
        m[cb] = m_up;
        l[cb] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[cb][db] = o[cb][db] * alpha;
      }
      fwd_probs_of_max(p, s, m, c, rs);
    }
    typename M::Slab pf[NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      l[cb] += rs[cb];
      pf[cb] = M::slab(p[0][cb], p[1][cb]);
      M::settle_slab(pf[cb]);
    }
    tiles.before_product(more);
    const typename M::Tr va = rd.tr_at(tiles.v_tile());
    const int skip = more ? 0 : hidden;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const typename M::Frag vf = M::tr(va, i);
#pragma unroll
      for (int cb = 0; cb < NC; ++cb)
        if (cb + 1 == NC || cb >= skip) M::mma_tr(i, vf, pf[cb], o[cb]);
    }
    lds_reads_done();
    tiles.end_step(more, vbase + next, a.kv_ss, left);
  }
  fwd_finish_fp32<T, D, NC>(a, qb, kbase, vbase, row0, seg_off, BN * n_kt, c, o, m, l);

  __syncthreads();   // the tiles' place is taken by the results
  float *part = reinterpret_cast<float *>(smem), *ml = reinterpret_cast<float *>(smem + Cfg::ML_AT);
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    const float lt = sum_over_rows(l[cb]);
    const int r = wave * ROWS + 16 * cb + n;
#pragma unroll
    for (int x = 0; x < DB; ++x) *reinterpret_cast<f32x4 *>(part + r * Cfg::O_ROW + M::quad_d0(x, j)) = M::quad(o[cb], x);
    if (j == 0) *reinterpret_cast<f32x2 *>(ml + 2 * r) = f32x2{m[cb], lt};
  }
  __syncthreads();
  // out = sum_w o_w 2^(m_w - m) / sum_w l_w 2^(m_w - m), as in seg_attn_fwd_merge_kernel; 4 elements of head_dim per thread
  T *ob = reinterpret_cast<T *>(a.out_w) + b * a.q_sb + h * a.q_sh;
  for (int x = tid; x < ROWS * (D / 4); x += 64 * W) {
    const int rl = x / (D / 4), c4 = x % (D / 4), r = row0 + rl;
    f32x2 w_ml[W];
    float top = -INFINITY, sum = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      w_ml[w] = *reinterpret_cast<const f32x2 *>(ml + 2 * (w * ROWS + rl));
      top = fmaxf(top, w_ml[w][0]);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float weight = w_ml[w][0] == top ? 1.f : exp2_fast(w_ml[w][0] - top);   // (1 also if all are -inf, which plain arithmetic leaves)
      sum += weight * w_ml[w][1];
      acc += weight * *reinterpret_cast<const f32x4 *>(part + (w * ROWS + rl) * Cfg::O_ROW + 4 * c4);
    }
    const float inv = 1.f / sum;
    if (r < seg_len) {
      store4<T>(ob + (int64_t)r * a.q_ss + 4 * c4, acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
      if (c4 == 0) a.lse[((int64_t)b * a.n_q_heads + h) * seg_len + r] = (top + __builtin_amdgcn_logf(sum)) * kLn2;
    }
  }
}

}  // namespace s1f

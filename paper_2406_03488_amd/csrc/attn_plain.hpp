// fp32 results that the products of planes (split3) cannot give, in plain fp32 arithmetic.  The planes of an infinity, and those of a
// product that has left the range of the planes, are NaN, and whatever they touch becomes NaN with them, where fp32 arithmetic has an
// infinity, or a finite number (a key with a score of minus infinity has weight zero).  A wave whose accumulators are not all finite
// behind its main loop therefore computes its rows or keys again, from the operands in memory.  Per wave, and behind the loop: what
// is finite never comes here and pays one instruction per accumulator.  Slow (no matrix instructions, one key or row at a time: 32
// heads, 2048 rows behind 8000 keys, head_dim 128, all of them seeing an infinite value: forward 1.8 -> 18.6 ms, dQ 2.3 -> 19.2, dK/dV 3.1
// -> 22.0), and each row touches only the keys that it sees.  A walk ends once a NaN weight has made all elements of all its rows
// NaN.
//
// Lanes as in the epilogues of the main kernels: lane (n, j) holds, of its row (or key) n, elements 16*x + 4*j .. +3 of head_dim.
#pragma once
#include "attn_tile.hpp"

namespace s1f {

// bad + 0 for each finite element, else NaN
S1F_DEV float add_if_not_finite(f32x4 x, float bad) {
#pragma unroll
  for (int e = 0; e < 4; ++e) bad = fmaf(x[e], 0.f, bad);
  return bad;
}
// a lane of the wave has something that is not finite
S1F_DEV bool any_not_finite(float bad) { return __builtin_amdgcn_ballot_w64(!(bad == 0.f)) != 0; }

// every lane has met a NaN weight
S1F_DEV bool all_nan(float w) { return __builtin_amdgcn_ballot_w64(w == w) == 0; }

template <int D> struct PlainRow {
  static constexpr int DB = D / 16;
  f32x4 x[DB];
  S1F_DEV void load(const float *row, int j) {
#pragma unroll
    for (int i = 0; i < DB; ++i) x[i] = *reinterpret_cast<const f32x4 *>(row + 16 * i + 4 * j);
  }
};
// dot product of the lanes' rows n
template <int D> S1F_DEV float plain_dot(const PlainRow<D> &a, const PlainRow<D> &b) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < D / 16; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fmaf(a.x[i][e], b.x[i][e], s);
  return sum_over_rows(s);
}
template <int D> S1F_DEV void plain_add(f32x4 (&acc)[D / 16], float w, const PlainRow<D> &r) {
#pragma unroll
  for (int i = 0; i < D / 16; ++i) acc[i] += w * r.x[i];
}

// Forward of one row per lane: `o` unnormalised, m in log2 units.  k, v: the first key's rows; the lane's row sees keys 0 .. last
// (`keys` of them for the lane that sees most).
template <int D>
S1F_DEV void fwd_plain(const float *q, const float *k, const float *v, int64_t kv_ss, int last, int keys, float c, int j,
                       f32x4 (&o)[D / 16], float &m, float &l) {
  PlainRow<D> qr, kr, vr;
  qr.load(q, j);
  m = -INFINITY;
  l = 0.f;
#pragma unroll
  for (int i = 0; i < D / 16; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int key = 0; key < keys; ++key) {
    kr.load(k + key * kv_ss, j);
    vr.load(v + key * kv_ss, j);
    float s = plain_dot<D>(qr, kr) * c;
    settle(s);   // the product that the maximum is taken of, rounded: see fwd_probs_of_max
    if (key <= last) {
      const float m_up = fmaxf(m, s), base = m_up == -INFINITY ? 0.f : m_up;
      const float alpha = exp2_fast(m - base), p = exp2_fast(s - base);
      m = m_up;
      l = l * alpha + p;
#pragma unroll
      for (int i = 0; i < D / 16; ++i) o[i] = o[i] * alpha;
      plain_add<D>(o, p, vr);
    }
    if (all_nan(l)) break;
  }
}

// dQ of one row per lane, unscaled; nl: -lse in log2 units, nd: -delta
template <int D>
S1F_DEV void dq_plain(const float *q, const float *dout, const float *k, const float *v, int64_t kv_ss, int last, int keys, float c,
                      float nl, float nd, int j, f32x4 (&dq)[D / 16]) {
  PlainRow<D> qr, dor, kr, vr;
  qr.load(q, j);
  dor.load(dout, j);
#pragma unroll
  for (int i = 0; i < D / 16; ++i) dq[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float met = 0.f;
#pragma unroll 1
  for (int key = 0; key < keys; ++key) {
    kr.load(k + key * kv_ss, j);
    vr.load(v + key * kv_ss, j);
    const float s = plain_dot<D>(qr, kr), dp = plain_dot<D>(dor, vr) + nd;
    if (key <= last) {
      const float ds = exp2_fast(fmaf(s, c, nl)) * dp;
      met = ds == ds ? met : ds;
      plain_add<D>(dq, ds, kr);
    }
    if (all_nan(met)) break;
  }
}

// What rows r0 .. r1-1 of one query head add to dK (unscaled) and dV of one key per lane, which rows from `first` on see.  q, dout:
// row 0 of the head; stats: its -lse/scale, and ws_plane floats on its -delta; met: NaN once a probability was
template <int D>
S1F_DEV void dkdv_plain(const PlainRow<D> &kr, const PlainRow<D> &vr, const float *q, const float *dout, int64_t q_ss, const float *stats,
                        int64_t ws_plane, int r0, int r1, int first, float c, int j, f32x4 (&dk)[D / 16], f32x4 (&dv)[D / 16],
                        float &met) {
  PlainRow<D> qr, dor;
#pragma unroll 1
  for (int r = r0; r < r1; ++r) {
    qr.load(q + r * q_ss, j);
    dor.load(dout + r * q_ss, j);
    const float s = plain_dot<D>(qr, kr) + stats[r], dp = plain_dot<D>(dor, vr) + stats[ws_plane + r];
    if (r >= first) {
      const float p = exp2_fast(s * c);
      met = p == p ? met : p;
      plain_add<D>(dv, p, dor);
      plain_add<D>(dk, p * dp, qr);
    }
    if (all_nan(met)) break;
  }
}

}  // namespace s1f

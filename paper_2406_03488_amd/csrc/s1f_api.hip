// C ABI of the library: argument validation and kernel dispatch.  See include/s1f.h for the contract.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdint>
#include <mutex>

#include "attn_bwd.hpp"
#include "attn_fwd.hpp"
#include "attn_fwd_keys.hpp"
#include "s1f.h"

namespace {
using namespace s1f;

// Column blocks of 16 rows per wave (NC) that the forward and dQ kernels are built for: row tiles of 64 * NC rows.  Wide
// tiles use every K/V operand read from LDS for more matrix instructions, narrow ones leave a small launch more
// workgroups; plan_rows chooses per launch.  The widest ones are what two waves per SIMD have registers for.
// Waves per SIMD of the dK/dV kernel: what its accumulators leave room for.
template <typename T, int D> struct Shape;
template <int D> struct Shape<bf16_t, D> {
  static constexpr int FWD_MAX = 3, DQ_MAX = D == 128 ? 2 : 3, OCC = 2, KWGS = D == 64 ? 3 : 2;
  // the 128-row forward at head_dim 64 takes 130 registers if left alone; LDS has room for the four workgroups that 128 allow
  static constexpr int fwd_occ(int nc) { return D == 64 && nc == 2 ? 4 : OCC; }
  static constexpr int dq_occ(int) { return OCC; }
  static constexpr int waves(int) { return 4; }
  // both halves of the backward in one launch: as many workgroups per compute unit as the dK/dV kernel has alone
  static constexpr int BOTH_OCC = KWGS;
  static constexpr bool both(int nc) { return nc <= (D == 64 ? 2 : DQ_MAX); }
};
template <int D> struct Shape<float, D> {
  static constexpr int FWD_MAX = 2, DQ_MAX = 2, KWGS = 2;
  static constexpr int waves(int nc) { return nc == 2 && D > 64 ? 8 : 4; }
  static constexpr int fwd_occ(int nc) { return waves(nc) == 8 || D == 64 ? 2 : 1; }
  static constexpr int dq_occ(int nc) { return fwd_occ(nc); }
  static constexpr int BOTH_OCC = 2;
  static constexpr bool both(int nc) { return nc <= DQ_MAX && (D == 64 || waves(nc) == 8); }   // (workgroups of the dK/dV kernel's size)
};

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_desc(const s1f_desc *d) {
  if (d == nullptr) return S1F_EINVAL;
  if (d->batch < 1 || d->n_q_heads < 1 || d->n_kv_heads < 1 || d->n_q_heads % d->n_kv_heads != 0) return S1F_EINVAL;
  if (d->reserved != 0 || d->kv_capacity < 1) return S1F_EINVAL;
  if (d->dtype != S1F_F32 && d->dtype != S1F_BF16) return S1F_EUNSUPPORTED;
  if (d->head_dim != 64 && d->head_dim != 80 && d->head_dim != 128) return S1F_EUNSUPPORTED;
  if (d->batch > 65535 || d->n_q_heads > 65535) return S1F_EUNSUPPORTED;
  if ((int64_t)d->batch * d->n_q_heads > 0x7fffffff) return S1F_EUNSUPPORTED;   // (batch, head) pairs are counted in 32 bits
  // 16-byte vector accesses: every row must start on a 16-byte boundary
  const int64_t ce = d->dtype == S1F_BF16 ? 8 : 4;
  const int64_t s[6] = {d->q_stride_b, d->q_stride_h, d->q_stride_s, d->kv_stride_b, d->kv_stride_h, d->kv_stride_s};
  for (int i = 0; i < 6; ++i)
    if (s[i] < 0 || s[i] % ce != 0) return S1F_EINVAL;
  if (d->q_stride_s < d->head_dim || d->kv_stride_s < d->head_dim) return S1F_EINVAL;
  // the asynchronous tile copies address the 32 rows of a tile with 32-bit byte offsets
  if (d->q_stride_s >= (int64_t(1) << 23) || d->kv_stride_s >= (int64_t(1) << 23)) return S1F_EUNSUPPORTED;
  return S1F_OK;
}

int check_seg(const s1f_desc *d, int64_t seg_off, int64_t seg_len) {
  if (seg_off < 0 || seg_len < 1 || seg_off + seg_len > d->kv_capacity) return S1F_ERANGE;
  if (seg_off + seg_len > (int64_t(1) << 30)) return S1F_ERANGE;   // kernels index rows with 32-bit integers
  return S1F_OK;
}

AttnArgs make_args(const s1f_desc *d, int64_t seg_off, int64_t seg_len) {
  AttnArgs a = {};
  a.q_sb = d->q_stride_b; a.q_sh = d->q_stride_h; a.q_ss = d->q_stride_s;
  a.kv_sb = d->kv_stride_b; a.kv_sh = d->kv_stride_h; a.kv_ss = d->kv_stride_s;
  a.seg_off = (int32_t)seg_off; a.seg_len = (int32_t)seg_len;
  a.n_q_heads = d->n_q_heads; a.group = d->n_q_heads / d->n_kv_heads;
  a.by_heads = Divisor::of(a.n_q_heads); a.by_kv_heads = Divisor::of(d->n_kv_heads); a.by_group = Divisor::of(a.group);
  a.scale = (float)(1.0 / std::sqrt((double)d->head_dim));
  return a;
}

// A launch counts its threads in 32 bits, and the runtime takes a larger one all the same and runs what its size is past 2^32: fewer
// workgroups, without an error (two backwards of 129 x 65535 heads of one row, in one launch: half of dK and dV missing).
bool one_launch(int64_t grid, int threads) { return grid * threads <= 0xffffffffll; }
// The arguments of a call over the batch entries from b0 on.
template <typename T> AttnArgs from_entry(AttnArgs a, int64_t b0) {
  auto tensor = [&](const void *p, int64_t stride) { return p ? reinterpret_cast<const T *>(p) + b0 * stride : nullptr; };
  auto ours = [&](void *p) { return const_cast<T *>(tensor(p, a.q_sb)); };
  auto floats = [&](float *p, int64_t stride) { return p ? p + b0 * stride : nullptr; };
  const int64_t rows = (int64_t)a.n_q_heads * a.seg_len;
  a.q = tensor(a.q, a.q_sb); a.out = tensor(a.out, a.q_sb); a.dout = tensor(a.dout, a.q_sb);
  a.k = tensor(a.k, a.kv_sb); a.v = tensor(a.v, a.kv_sb);
  a.out_w = ours(a.out_w); a.dq = ours(a.dq);
  a.lse = floats(a.lse, rows); a.delta = floats(a.delta, rows);
  a.dk_acc = floats(a.dk_acc, a.kv_sb); a.dv_acc = floats(a.dv_acc, a.kv_sb);
  return a;
}
// Runs a call that is too large for one launch as two, over the halves of its batch entries.
template <typename T, typename F> int in_halves(const s1f_desc *d, const AttnArgs &a, F call) {
  if (d->batch < 2) return S1F_EUNSUPPORTED;
  s1f_desc lo = *d, hi = *d;
  lo.batch = d->batch / 2;
  hi.batch = d->batch - lo.batch;
  const int rc = call(&lo, a);
  return rc == S1F_OK ? call(&hi, from_entry<T>(a, lo.batch)) : rc;
}

// Kernels that need more than 64 KiB of LDS have to be told so once per device; `prepare` does that the first time
// a kernel is used on the current device (a template over the kernel itself, not its type, which all of them share: one set of
// flags each).
constexpr int kMaxDevices = 64;
template <auto KERNEL> int prepare(int lds_bytes) {
  if (lds_bytes <= 64 * 1024) return S1F_OK;
  static std::atomic<bool> done[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return S1F_EDEVICE;
  const bool cached = dev >= 0 && dev < kMaxDevices;
  if (cached && done[dev].load(std::memory_order_acquire)) return S1F_OK;
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize,
                          lds_bytes) != hipSuccess)
    return S1F_EDEVICE;
  if (cached) done[dev].store(true, std::memory_order_release);
  return S1F_OK;
}

// Order of the row tiles of the forward and dQ kernels within an XCD.  Tile by tile over the XCD's heads whenever
// query heads share K/V heads: an XCD then holds the query heads of one K/V group, and running the same row tile of
// all of them side by side makes them stream the same K/V rows through its L2 at the same time.  Otherwise head by
// head (all row tiles of a head side by side share its K/V rows), except for a SHORT launch whose tiles differ a lot
// in length (a first segment of a few rounds of workgroups): tile by tile the light tiles of every head then come
// last and fill the end of the launch.  A long first segment (many rounds: one unsegmented pass over 65536 tokens
// and 56 heads measured 11 % faster in the forward, 9 % in the dQ kernel) stays head by head.
constexpr int64_t kTileMajorMaxUnits = 6144;   // about eight rounds of row tiles
int row_tile_order(const s1f_desc *d, const AttnArgs &a) {
  if (d->n_q_heads > d->n_kv_heads) return 1;
  const int64_t units = (((int64_t)a.seg_len + 127) / 128) * d->n_q_heads * d->batch;
  return 2 * (int64_t)a.seg_off < (int64_t)a.seg_len && units <= kTileMajorMaxUnits;
}

// ---- how a launch is cut ----------------------------------------------------------------------------------------
// A launch of units of equal length runs in rounds of as many workgroups as the chip holds at once; its last round may
// leave most of the chip idle and still lasts as long as a unit.  Two things can be chosen per launch: the width of the
// row tiles (forward and dQ), and into how many chunks the units of the last round are cut (along the keys in the
// forward and dQ kernels, see split_unit; along the queries in the dK/dV kernel), to run side by side and be merged by a
// second kernel.  The plan with the shortest predicted time is taken.  It is a function of shape, device and workspace
// limit only, so that the workspace-size queries and the launches derive the same one.
constexpr int64_t kMaxPartBytes = int64_t(512) << 20;      // partial results of one launch with a caller's workspace
constexpr int64_t kStaticPartBytes = int64_t(32) << 20;    // ... with the library's built-in scratch
constexpr double kStartUs = 4.0, kRoundUs = 2.0;           // prologue and epilogue of the first workgroups, of a further round
constexpr double kMergeUs = 4.5, kMergeBytesPerUs = 2.5e6; // the merge kernel: fixed part, rate of its reads

// Time of one loop step of a workgroup, in microseconds, measured on launches of one workgroup per compute unit (alone),
// of two (shared) and of all it holds where that is more (crowd: per workgroup), 64 heads behind 4096 and 16384 keys;
// linear in the tile width.  The forward at head_dim 64, shared and crowd: fitted to 350 launches of each width (first
// segments and behind prefixes, 10 to 2500 us), whose times the prediction then misses by 7 % instead of 14; with the
// former numbers it preferred 192-row tiles where 128 rows were up to 16 % faster (32 heads, 5573 rows behind 48904 keys
// 2957 -> 2543 us).
struct StepUs {
  double alone0, alone_nc, shared0, shared_nc, crowd0, crowd_nc;
  double merge = 1;   // cost of the merge behind a cut launch, relative to kMergeUs and kMergeBytesPerUs
  double at(int nc, int64_t per_cu) const {
    if (per_cu <= 1) return alone0 + alone_nc * nc;
    const double two = shared0 + shared_nc * nc, all = (crowd0 + crowd_nc * nc) * (double)per_cu;
    return two > all ? two : all;
  }
};
template <typename T, int D> struct Cost;   // forward, dQ (steps of 32 keys), dK/dV (steps of 32 rows, nc = 0)
template <> struct Cost<bf16_t, 64> {
  static constexpr StepUs fwd = {0.225, 0.11, 0.181, 0.18, 0.034, 0.119}, dq = {0.075, 0.16, 0.12, 0.31, 0.07, 0.12},
                          dkdv = {0.75, 0, 0.9, 0, 0.42, 0};
};
template <> struct Cost<bf16_t, 80> {
  static constexpr StepUs fwd = {0.28, 0.12, 0.25, 0.26, 0, 0}, dq = {0.165, 0.175, 0.285, 0.335, 0, 0}, dkdv = {0.85, 0, 1.2, 0, 0, 0};
};
template <> struct Cost<bf16_t, 128> {
  static constexpr StepUs fwd = {0.29, 0.17, 0.36, 0.32, 0, 0}, dq = {0.2, 0.26, 0.32, 0.52, 0, 0}, dkdv = {1.05, 0, 1.65, 0, 0, 0};
};
// fp32: the forward at head_dim 80 and 128, dQ at 80 and dK/dV as measured.  Not so the forward at head_dim 64 (up to 19 % above) and
// dQ at 64 and 128 (alone: up to 1.9 and 2.1 times above; merge 0.7): those values are chosen for the plans that they lead to, some of which
// the tests of tile widths ask for by shape.  What cut 64-row dQ units cost above head_dim 64 is kept out by DqFamily::cut_narrow.
template <> struct Cost<float, 64> {
  static constexpr StepUs fwd = {0.72, 0.46, 0.885, 0.92, 0, 0}, dq = {-1.17, 2.23, 0.37, 1.615, 0, 0, 0.7}, dkdv = {2.75, 0, 4.7, 0, 0, 0};
};
template <> struct Cost<float, 80> {   // one workgroup per compute unit (LDS), as at head_dim 128
  static constexpr StepUs fwd = {0.75, 0.47, 1.5, 0.94, 0, 0}, dq = {0.83, 0.707, 1.67, 1.41, 0, 0}, dkdv = {3.3, 0, 6.6, 0, 0, 0};
};
template <> struct Cost<float, 128> {
  static constexpr StepUs fwd = {1.034, 0.636, 2.07, 1.27, 0, 0}, dq = {0.2, 3.09, 0.4, 6.18, 0, 0}, dkdv = {4.2, 0, 8.4, 0, 0, 0};
};

// Workgroups of a kernel that the current device holds at once, and its compute units (0 if that cannot be found out,
// e.g. without a device: launches are then never cut).
struct Slots {
  int total = 0, cus = 0;
};

// Time of `units` workgroups of `mean` loop steps each on average and `longest` at most, longest first.  Equal ones run in
// rounds; units whose length goes down to nothing (first segments) fill the gaps of each other, and then the longest
// ones, which share their compute unit for about half of their life, set the least time.  (32 heads, first segment of
// 2406 rows, head_dim 80: tiles of 128 rows 46 us, of 192 rows 60.)
double rounds_us(int64_t units, double mean, double longest, const StepUs &us, int nc, const Slots &s) {
  const int64_t per_cu = s.total / s.cus, full = units / s.total, rest = units % s.total;
  double rounds = full * (mean * us.at(nc, per_cu) + kRoundUs);
  if (rest > 0) rounds += mean * us.at(nc, (rest + s.cus - 1) / s.cus);
  const int64_t busy = units < s.total ? (units + s.cus - 1) / s.cus : per_cu;
  const double packed = (double)units * mean * us.at(nc, busy) / (double)(busy * s.cus) + full * kRoundUs;
  const double spread = longest < 2 * mean ? (longest - mean) / mean : 1.0;
  const double t = rounds + spread * (packed - rounds);
  const double one = longest * 0.5 * (us.at(nc, 1) + us.at(nc, busy < 2 ? busy : 2));
  return kStartUs + (t > one ? t : one);
}

struct SplitPlan {
  int nc = 1;                 // tile width (forward and dQ)
  int64_t n_tiles = 0;        // row tiles per (batch, head)
  int64_t n_whole = 0;        // leading workgroup ids that are whole units
  int64_t n_split_units = 0;  // units cut into chunks
  int n_split = 1;            // chunks per split unit
  int64_t grid() const { return n_whole + n_split_units * n_split; }
  int64_t chunks() const { return n_split_units * n_split; }
  SplitPlan uncut(int64_t n_bh) const { return SplitPlan{nc, n_tiles, n_tiles * n_bh, 0, 1}; }
};

// Chooses between whole units and, with cap > 0, each number of chunks for those of the last round, of which `direct` per
// unit need no partial result; `*t` is the time of the best plan known so far.
void plan_units(SplitPlan *best, double *t, int nc, int64_t n_tiles, int64_t units, double steps, double longest,
                const StepUs &us, const Slots &s, int64_t part_bytes, int direct, int64_t cap) {
  const int64_t r = units % s.total, whole = units - r;
  for (int n = 1; n <= kMaxChunks; ++n) {
    double now;
    if (n == 1) {
      now = rounds_us(units, steps, longest, us, nc, s);
    } else {
      const int64_t bytes = r * (n - direct) * part_bytes;
      if (r == 0 || steps < (double)n || bytes > cap) break;
      const double extra = us.merge * (kMergeUs + (double)bytes / kMergeBytesPerUs + 1.0);   // (1.0: not for nothing)
      if (kStartUs + extra >= *t) break;   // nor can more chunks win (the smallest launches end here, after one prediction)
      now = rounds_us(r * n, steps / n, longest / n, us, nc, s) + extra;
      if (whole > 0) now += rounds_us(whole, steps, steps, us, nc, s) - kStartUs;
    }
    if (now < *t) {
      *t = now;
      best->nc = nc;
      best->n_tiles = n_tiles;
      best->n_whole = n == 1 ? units : whole;
      best->n_split_units = n == 1 ? 0 : r;
      best->n_split = n;
    }
  }
}

// Looked up once per kernel and device.
template <auto KERNEL> Slots resident_slots(int lds_bytes, std::atomic<int64_t> *cache, int threads) {
  Slots s;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return s;
  }
  const int64_t known = cache[dev].load(std::memory_order_acquire);
  if (known > 0) {
    s.total = (int)(known >> 32);
    s.cus = (int)(known & 0xffffffff);
    return s;
  }
  int per_cu = 0, cus = 0;
  if (prepare<KERNEL>(lds_bytes) != S1F_OK ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(KERNEL), threads,
                                                   (size_t)lds_bytes) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per_cu <= 0 || cus <= 0) {
    (void)hipGetLastError();
    return s;
  }
  s.total = per_cu * cus;
  s.cus = cus;
  cache[dev].store(((int64_t)s.total << 32) | cus, std::memory_order_release);
  return s;
}

// One-dimensional grid; the kernels decode (unit -> tile, batch*head; chunk) themselves.
// `tile_major`: order of the workgroups within an XCD; chosen per kernel from the shape of the segment.
// The status reflects this launch only (the return code of the launch call, not the runtime's sticky last error).
void fill_launch(AttnArgs *a, int64_t n_bh, int tile_major, const SplitPlan &p) {
  a->n_tiles = (int32_t)p.n_tiles;
  a->n_bh = (int32_t)n_bh;
  a->tile_major = tile_major;
  a->n_whole = (int32_t)p.n_whole;
  a->n_split = p.n_split;
  a->n_split_units = (int32_t)p.n_split_units;
  a->bm = 64 * p.nc;
  a->by_tiles = Divisor::of(p.n_tiles);
  a->by_xcd = Divisor::of(n_bh < 8 ? 1 : n_bh / 8);
  a->by_split = Divisor::of(p.n_split);
  a->by_split_units = Divisor::of(p.n_split_units < 1 ? 1 : p.n_split_units);
}
template <auto KERNEL> int launch(int lds_bytes, const SplitPlan &p, int64_t n_bh, AttnArgs a, hipStream_t st, int threads) {
  if (p.n_tiles * n_bh > 0x7fffffff || !one_launch(p.grid(), threads)) return S1F_EUNSUPPORTED;
  const int rc = prepare<KERNEL>(lds_bytes);
  if (rc != S1F_OK) return rc;
  void *params[] = {&a};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(KERNEL), dim3((unsigned)p.grid()), dim3(threads), params,
                                       (size_t)lds_bytes, st);
  return e == hipSuccess ? S1F_OK : S1F_EDEVICE;
}

// The merge kernel behind a split launch: `groups` workgroups (of a few rows each) per split unit.
template <typename K> int launch_merge(K kernel, AttnArgs a, const SplitPlan &plan, int groups, hipStream_t st) {
  a.by_groups = Divisor::of(groups);
  void *params[] = {&a};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3((unsigned)(plan.n_split_units * groups)),
                                       dim3(256), params, 0, st);
  return e == hipSuccess ? S1F_OK : S1F_EDEVICE;
}

// The instance of the forward's merge kernel for a number of partial results per unit.
#define S1F_MERGE(KERNEL, T, D, parts, ...)                                                                       \
  ((parts) <= 2   ? launch_merge(KERNEL<T, D, 2>, __VA_ARGS__)                                                    \
   : (parts) <= 4 ? launch_merge(KERNEL<T, D, 4>, __VA_ARGS__)                                                    \
   : (parts) <= 8 ? launch_merge(KERNEL<T, D, 8>, __VA_ARGS__)                                                    \
                  : launch_merge(KERNEL<T, D, kMaxChunks>, __VA_ARGS__))

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- forward and dQ: row tiles of one kernel family ----
// KERNEL<NC> of a family F: F::kernel<NC>(), F::LDS, F::MAX (widest NC), F::cost
template <typename T, int D> struct FwdFamily {
  static constexpr bool FP32 = sizeof(T) == 4;
  static constexpr int MAX = Shape<T, D>::FWD_MAX, LDS = TileRing<T, D>::LDS_BYTES;
  static constexpr StepUs cost = Cost<T, D>::fwd;
  static constexpr int64_t row_bytes = D * 4 + 8;   // of a partial result: output, running maximum, row sum
  static bool cut_narrow(int64_t) { return true; }
    static constexpr int threads(int nc) { return 64 * Shape<T, D>::waves(nc); }
  template <int NC> static constexpr auto kernel() {
    constexpr int W = Shape<T, D>::waves(NC);
    return seg_attn_fwd_kernel<T, D, 4 * NC / W, Shape<T, D>::fwd_occ(NC), W>;
  }
  static constexpr auto rest_kernel() { return seg_attn_fwd_kernel<T, D, 1, Shape<T, D>::fwd_occ(1), 4, true>; }
};
template <typename T, int D> struct DqFamily {
  static constexpr int MAX = Shape<T, D>::DQ_MAX, LDS = TileRing<T, D>::LDS_BYTES;
  static constexpr StepUs cost = Cost<T, D>::dq;
  static constexpr int64_t row_bytes = D * 4;
  // Are units of 64 rows ever cut?  fp32 above head_dim 64: not unless those of 128 rows (eight waves, and a kernel for both halves in one
  // launch) would compute too many rows for nothing.  Cut in 64 rows / as then planned, backward of a segment, us: 8/2 heads, head_dim
  // 128, first segment of 1240 rows 125 / 99, 941 rows behind 2300 252 / 220; 4 heads, 80, first segment of 930 63 / 48.  Over 218 random
  // calls that this changes the one call takes 0.65 to 1.04 of the time, 0.80 on average; both halves one after the other 0.87 to 1.15, 1.02 on
  // average, for the dQ half by itself had been faster in small calls (see dq_in_pairs).  (The one call would gain beyond 3/16 as well; tests
  // ask for such plans.)
  static bool cut_narrow(int64_t seg_len) {
    return sizeof(T) == 2 || D == 64 || 16 * ((seg_len + 127) / 128 * 128 - seg_len) > 3 * seg_len;
  }
    static constexpr int threads(int nc) { return 64 * Shape<T, D>::waves(nc); }
  template <int NC> static constexpr auto kernel() {
    constexpr int W = Shape<T, D>::waves(NC);
    return seg_attn_bwd_dq_kernel<T, D, 4 * NC / W, Shape<T, D>::dq_occ(NC), W>;
  }
  static constexpr auto pair_kernel() { return seg_attn_bwd_dq_kernel<T, D, 1, Shape<T, D>::dq_occ(1), 4, sizeof(T) == 4 && D != 64>; }
};
template <typename F, int NC> Slots family_slots() {
  static std::atomic<int64_t> cache[kMaxDevices];
  return resident_slots<F::template kernel<NC>()>(F::LDS, cache, F::threads(NC));
}
// The dQ half by itself in fp32 above head_dim 64, planned in units of 128 rows (eight waves): does it run as two tiles of 64 rows for each,
// in four waves?  The same sums; half as long a launch of few units, where every tile then has a compute unit of its own, and still shorter
// where chunks are so short that starting a workgroup counts.  In units of 128 / in pairs, us: 3 heads, head_dim 128, first segment of 366
// rows 26.9 / 22.5; 2/1 heads, 80, 230 behind 3539 33.2 / 27.4; 4 heads, 128, 233 behind 771 34.1 / 28.9; over 87 random calls that the rule takes
// 0.78 .. 1.00 of the time, 0.86 on average; beyond it pairs take up to 1.4 times as long (4 heads, 80, first segment of 4088 154.9 / 220.1).
// (By itself this half would be faster still in 64-row units with chunks of their own, for the calls of this rule 1.12 times on average; the one
// call of both halves, 0.66 .. 0.9 of its former time in units of 128, has to have the same chunks.)
template <typename T, int D> bool dq_in_pairs(const AttnArgs &a, const SplitPlan &p) {
  if (sizeof(T) == 2 || D == 64 || p.nc != 2 || p.n_whole > 0) return false;
  const int64_t cus = family_slots<DqFamily<T, D>, 2>().cus;
  const double walk = ((double)a.seg_off + 0.5 * a.seg_len) / 32 / p.n_split;
  return 2 * p.grid() <= cus || (p.grid() < cus && walk <= 2);
}
template <typename F, int NC> void plan_rows_nc(const s1f_desc *d, int64_t seg_off, int64_t seg_len, int64_t cap, SplitPlan *best, double *t) {
  const Slots s = family_slots<F, NC>();
  const int64_t tiles = (seg_len + 64 * NC - 1) / (64 * NC), units = tiles * d->n_q_heads * d->batch;
  if (s.total <= 0) {   // nothing known about the device: the widest tiles, uncut
    if (best->n_tiles == 0) { best->nc = NC; best->n_tiles = tiles; best->n_whole = units; }
    return;
  }
  plan_units(best, t, NC, tiles, units, (double)(seg_off + (seg_len + 1) / 2) / 32 + 1, (double)(seg_off + seg_len) / 32 + 1, F::cost,
             s, F::row_bytes * 64 * NC, 0, cap);
}
// Wide tiles first: a narrower one has to be faster.  us: the time predicted for the plan
template <typename F> SplitPlan plan_rows(const s1f_desc *d, int64_t seg_off, int64_t seg_len, int64_t cap, double *us = nullptr) {
  SplitPlan p;
  double t = 1e300;
  if constexpr (F::MAX >= 3) plan_rows_nc<F, 3>(d, seg_off, seg_len, cap, &p, &t);
  plan_rows_nc<F, 2>(d, seg_off, seg_len, cap, &p, &t);
  plan_rows_nc<F, 1>(d, seg_off, seg_len, F::cut_narrow(seg_len) ? cap : 0, &p, &t);
  if (us != nullptr) *us = t;
  return p;
}
template <typename F> int launch_rows(const SplitPlan &p, int64_t n_bh, const AttnArgs &a, hipStream_t st) {
  if constexpr (F::MAX >= 3)
    if (p.nc == 3) return launch<F::template kernel<3>()>(F::LDS, p, n_bh, a, st, F::threads(3));
  if (p.nc == 2) return launch<F::template kernel<2>()>(F::LDS, p, n_bh, a, st, F::threads(2));
  return launch<F::template kernel<1>()>(F::LDS, p, n_bh, a, st, F::threads(1));
}

template <typename T, int D> size_t fwd_workspace(const SplitPlan &p) {
  const int64_t rows = p.chunks() * 64 * p.nc;
  return rows == 0 ? 0 : align256((size_t)(rows * D * 4)) + (size_t)(rows * 8);
}
// An uncut launch whose last round fills only part of the chip: is it faster to leave the units of that round to a second
// launch, in tiles of 64 rows (more of them side by side, each a shorter walk per key)?  Sets `whole` to the units that
// stay.  kDrainUs: the first launch has to end, its workgroups at slightly different times, before the second begins
// (launches of 200 to 300 us lost 1 % where 2 % were predicted).
// Each of 110 shapes for which the prediction says yes, timed both ways (second launch / one launch):
//   bf16, grouped heads (units run tile by tile, those left over are the shortest)   0.85 .. 0.94 of 29, mean 0.91
//   bf16, ungrouped (head by head), longest unit <= 1.12 of the mean                 0.87 .. 1.01 of 27, mean 0.95
//   bf16, ungrouped, longest unit > 1.15 of the mean: long and short ones already fill each other's gaps
//                                                                                    1.02 .. 1.10 of 10, mean 1.06
//   bf16 at head_dim 64, three or four workgroups per compute unit: no round ends at once
//                                                                                    0.95 .. 1.06 of 36, mean 1.03
//   fp32, grouped, behind seven or more full rounds 0.99 .. 1.02 of 7; behind fewer 0.99 .. 1.26 of 7; ungrouped 1.02
// hence the further conditions (fp32: either way takes the same time where the second launch is still allowed).  56 heads, 3678 rows behind 39549 keys (96 units of 192 rows left over) 4286 -> 3974
// us; 64/8 heads, 3214 rows behind 5000 keys 645 -> 592.
constexpr double kDrainUs = 10.0, kTailUneven = 1.12, kTailUnevenGrouped = 1.3;
template <typename F, int NC> bool row_tail(const AttnArgs &a, const SplitPlan &p, int64_t *whole) {
  const Slots s = family_slots<F, NC>(), s1 = family_slots<F, 1>();
  if (s.total <= 0 || s1.total <= 0) return false;
  const int64_t units = p.n_whole, r = units % s.total;
  const double mean = (double)(a.seg_off + (a.seg_len + 1) / 2) / 32 + 1, most = (double)(a.seg_off + a.seg_len) / 32 + 1;
  *whole = units - r;
  if (r == 0 || *whole == 0 || s.total > 2 * s.cus) return false;
  if (most > (a.group > 1 ? kTailUnevenGrouped : kTailUneven) * mean) return false;
  if (F::FP32 && (a.group == 1 || *whole < 7 * (int64_t)s.total)) return false;
  const double now = rounds_us(units, mean, most, F::cost, NC, s);
  const double two = rounds_us(*whole, mean, mean, F::cost, NC, s) + rounds_us(r * NC, mean, mean, F::cost, 1, s1);
  return two + kDrainUs < (F::FP32 ? 1.03 : 0.98) * now;
}

// ... for a plan of either width; 64-row tiles have no narrower ones to go to.
template <typename F> bool row_tail_of(const AttnArgs &a, const SplitPlan &p, int64_t *whole) {
  if (p.n_split_units != 0) return false;
  if (p.nc == 2) return row_tail<F, 2>(a, p, whole);
  if constexpr (F::MAX >= 3)
    if (p.nc == 3) return row_tail<F, 3>(a, p, whole);
  return false;
}

// How the rows of a forward whose last round goes to a second launch are shared out: `head` the first launch, `rest` the second (units
// of the first cut into 64-row tiles, and `rag` such tiles of the partly filled last unit of every (batch, head)).
struct Tail {
  SplitPlan head, rest;
  int64_t rag = 0;
};
template <typename F> bool fwd_tail(const AttnArgs &a, const SplitPlan &p, int64_t n_bh, Tail *t) {
  int64_t whole = 0;
  if (!row_tail_of<F>(a, p, &whole)) return false;
  t->head = t->rest = p;
  t->head.n_whole = whole;
  t->rest.nc = 1;
  t->rest.n_whole = 0;
  t->rest.n_split_units = p.n_whole - whole;
  t->rest.n_split = p.nc;
  // The last unit of every (batch, head) may hold rows for fewer 64-row tiles than the others; where that leaves fewer tiles to the
  // busiest compute unit, it is those that run in the second launch.  56 heads, 3678 rows behind 39549 keys: 56 units of 30 rows and
  // 40 whole ones are 176 tiles, 96 whole ones 288: 3903 -> 3746 us; 3669 rows behind 40380 4010 -> 3835.  Over 40 random calls that
  // it moves rows in (24 to 130 heads, 0.9 to 6 ms), time against leaving the last units of the launch: head_dim 128 0.947 .. 1.030, mean
  // 0.969; 80 0.956 .. 1.009, mean 0.990.  Not for grouped heads, whose units left over are the ones with the fewest keys (64/8 heads, 3110
  // rows behind 4612: 524 -> 561).
  const int64_t rag = (a.seg_len - (p.n_tiles - 1) * 64 * p.nc + 63) / 64, cus = family_slots<F, 1>().cus;
  const int64_t tiles = t->rest.n_split_units * p.nc, fewer = tiles - (p.nc - rag) * n_bh;
  if (a.group == 1 && t->rest.n_split_units >= n_bh && (fewer + cus - 1) / cus < (tiles + cus - 1) / cus) {
    t->head.n_tiles = t->rest.n_tiles = p.n_tiles - 1;
    t->rest.n_split_units -= n_bh;
    t->rest.n_whole = rag * n_bh;
    t->rag = rag;
  }
  return true;
}

// The forward whose waves share the keys of a unit (seg_attn_fwd_kernel_by_keys).  Its time in microseconds, fitted to calls of 4 to 500
// us: base + step per 32 keys (which a workgroup's waves walk side by side), for units of 16 and of 32 rows with a compute unit each.
// least1, least2: steps from which on it is faster.  Row tiles walk fewer in less time than waves need to meet: bf16, D 64, 16 rows and keys 2.97
// us in row tiles, 3.44 by keys; fp32, 20 rows behind 60 6.17, 8.98; bf16, D 128, 399 rows behind 8, units of 32 9.0, 10.4
struct KeysUs {
  double base1, step1, base2, step2;
  int least1, least2;
};
template <typename T, int D> struct KeysCost;
template <> struct KeysCost<bf16_t, 64> { static constexpr KeysUs us = {4.0, 0.073, 5.0, 0.105, 5, 16}; };
template <> struct KeysCost<bf16_t, 80> { static constexpr KeysUs us = {4.2, 0.103, 6.3, 0.125, 6, 16}; };
template <> struct KeysCost<bf16_t, 128> { static constexpr KeysUs us = {4.8, 0.146, 8.0, 0.17, 8, 16}; };
template <> struct KeysCost<float, 64> { static constexpr KeysUs us = {6.0, 0.33, 10.0, 0.45, 7, 16}; };
template <> struct KeysCost<float, 80> { static constexpr KeysUs us = {6.5, 0.45, 10.0, 0.75, 7, 16}; };
template <> struct KeysCost<float, 128> { static constexpr KeysUs us = {8.0, 0.85, 17.0, 1.0, 12, 24}; };
template <typename T, int D, int NC> struct KeysShape {
  // fp32 at head_dim 80: eight waves of two column blocks spill; 128: LDS
  static constexpr int W = sizeof(T) == 2 || D == 64 || (D == 80 && NC == 1) ? 8 : 4;
  static constexpr int PER_CU = sizeof(T) == 2 && D == 64 && NC == 1 ? 2 : 1;   // workgroups that a compute unit takes without longer steps
};
// Column blocks of its waves (1 or 2), if such a launch is predicted to take less than `plan_us`, the plan of row tiles' time; else 0.
//   few units only    (each has a compute unit to itself): beyond, every unit reading all keys costs more than idle compute units
//   not fp32 with a workspace   its steps are bound by the splitting of operands, which waves of row tiles share: 4 heads, 256 rows behind
//                     768 keys, D 64 cut into chunks 13.4 us, by keys 17.7; without a workspace 34.9, by keys 17.7
//   with a workspace, up to 48 steps, or up to 80 if units take more than half of the chip   chunks use the compute units that few units
//                     leave idle: 2/1 heads, 839 rows behind 2668, D 80 14.6 us in chunks, 15.1 by keys; 4 heads, 368 behind 2578, 13.4 and
//                     13.6 (few units of 50 to 80 steps would still gain up to 25 %; tests ask for chunks there).  Above D 64 a handful of
//                     units up to 24 steps (one head, 46 rows behind 1227, D 128 9.0 in chunks, 10.2 by keys), D 128 a sixth of the chip up to 32
//                     (40 rows behind 1228 of 2 entries 1.10, 16 heads, 11 behind 1063 1.04 times as long)
//   fewer than 32 (batch, head) pairs   with a workspace there is nothing in it beyond (32 heads, 129 rows behind 4011 keys, D 64: 18.7 us in
//                     chunks, 18.5 by keys); without one there would be (40.4 us), but tests ask for the tile widths of such calls by shape
// Over 600 random calls that run so, of one to 4200 rows, time against row tiles: bf16 with a workspace 0.56 .. 1.11, 0.81 on average, without
// 0.23 .. 1.05, 0.56, fp32 without 0.35 .. 1.08, 0.61 (2/1 heads, 3046 rows behind 31131, D 80: 371 -> 119 us).
template <typename T, int D> int keys_nc(const s1f_desc *d, int64_t seg_off, int64_t seg_len, int64_t cap, double plan_us) {
  const int64_t cus = family_slots<FwdFamily<T, D>, 1>().cus, n_bh = (int64_t)d->n_q_heads * d->batch;
  if (cus <= 0 || 8 * n_bh >= cus || (sizeof(T) == 4 && cap > 0)) return 0;
  constexpr KeysUs us = KeysCost<T, D>::us;
  const double steps = (double)((seg_off + seg_len + 31) / 32);
  const int64_t units1 = (seg_len + 15) / 16 * n_bh, units2 = (seg_len + 31) / 32 * n_bh;
  if (cap > 0 && steps > (2 * units1 > cus ? 80 : D > 64 && 32 * units1 < cus ? 24 : D == 128 && 6 * units1 < cus ? 32 : 48)) return 0;
  int nc = 0;
  // (two units of 16 rows on a compute unit: each step takes 1.6 times as long)
  const double us1 = us.base1 + us.step1 * steps * (units1 > cus ? 1.6 : 1.0), us2 = us.base2 + us.step2 * steps;
  if (units1 <= KeysShape<T, D, 1>::PER_CU * cus && steps >= us.least1 && us1 < plan_us) { nc = 1; plan_us = us1; }
  if (units1 > cus && units2 <= cus && steps >= us.least2 && us2 < plan_us) nc = 2;
  return nc;
}
// The plan of a forward, and how many column blocks its waves hold where they share keys (0: they do not; then as planned).
struct FwdPlan {
  SplitPlan p;
  int keys_nc = 0;
};
template <typename T, int D> FwdPlan fwd_plan(const s1f_desc *d, int64_t seg_off, int64_t seg_len, int64_t cap) {
  FwdPlan f;
  double us = 0;
  f.p = plan_rows<FwdFamily<T, D>>(d, seg_off, seg_len, cap, &us);
  f.keys_nc = keys_nc<T, D>(d, seg_off, seg_len, cap, us);
  if (f.keys_nc > 0) {
    const int64_t tiles = (seg_len + 16 * f.keys_nc - 1) / (16 * f.keys_nc);
    f.p = SplitPlan{1, tiles, tiles * d->n_q_heads * d->batch, 0, 1};
  }
  return f;
}
template <typename T, int D, int NC> int launch_keys(const s1f_desc *d, AttnArgs a, const SplitPlan &p, hipStream_t st) {
  constexpr int W = KeysShape<T, D, NC>::W;
  const int64_t n_bh = (int64_t)d->n_q_heads * d->batch;
  fill_launch(&a, n_bh, row_tile_order(d, a), p);
  a.bm = 16 * NC;
  a.by_split = Divisor::of(W);   // (a unit's waves)
  return launch<seg_attn_fwd_kernel_by_keys<T, D, NC, W>>(FwdKeysCfg<T, D, NC, W>::LDS_BYTES, p, n_bh, a, st, 64 * W);
}

template <typename T, int D> int fwd_run(const s1f_desc *d, AttnArgs a, const SplitPlan &p, hipStream_t st, void *workspace) {
  typedef FwdFamily<T, D> F;
  const int64_t n_bh = (int64_t)d->n_q_heads * d->batch;
  if (p.n_tiles * n_bh > 0x7fffffff) return S1F_EUNSUPPORTED;
  if (!one_launch(p.grid(), F::threads(p.nc)))
    return in_halves<T>(d, a, [&](const s1f_desc *half, const AttnArgs &x) {
      return fwd_run<T, D>(half, x, p.uncut((int64_t)d->n_q_heads * half->batch), st, nullptr);
    });
  a.part = reinterpret_cast<float *>(workspace);
  a.part_ml = reinterpret_cast<float *>(reinterpret_cast<char *>(workspace) + align256((size_t)(p.chunks() * 64 * p.nc * D * 4)));
  fill_launch(&a, n_bh, row_tile_order(d, a), p);
  a.first_id = 0;
  Tail t;
  if (fwd_tail<F>(a, p, n_bh, &t)) {
    a.by_rag = Divisor::of(t.rag < 1 ? 1 : t.rag);
    fill_launch(&a, n_bh, row_tile_order(d, a), t.head);
    const int rc = launch_rows<F>(t.head, n_bh, a, st);
    if (rc != S1F_OK) return rc;
    a.first_id = (int32_t)t.head.n_whole;
    a.n_split = t.rest.n_split;
    a.n_split_units = (int32_t)t.rest.n_split_units;
    a.by_split_units = Divisor::of(t.rest.n_split_units < 1 ? 1 : t.rest.n_split_units);
    return launch<F::rest_kernel()>(F::LDS, t.rest, n_bh, a, st, F::threads(1));
  }
  const int rc = launch_rows<F>(p, n_bh, a, st);
  if (rc != S1F_OK || p.n_split_units == 0) return rc;
  return S1F_MERGE(seg_attn_fwd_merge_kernel, T, D, p.n_split, a, p, MergeRows<D>::groups(a.bm), st);
}
template <typename T, int D>
int fwd_impl(const s1f_desc *d, const AttnArgs &a, hipStream_t st, void *workspace, size_t workspace_bytes, bool split) {
  FwdPlan f = fwd_plan<T, D>(d, a.seg_off, a.seg_len, split ? kMaxPartBytes : 0);
  if (fwd_workspace<T, D>(f.p) > workspace_bytes) {
    if (sizeof(T) == 2) return S1F_EINVAL;
    f = fwd_plan<T, D>(d, a.seg_off, a.seg_len, 0);   // fp32 runs with any workspace
  }
  if (f.keys_nc == 1) return launch_keys<T, D, 1>(d, a, f.p, st);
  if (f.keys_nc == 2) return launch_keys<T, D, 2>(d, a, f.p, st);
  return fwd_run<T, D>(d, a, f.p, st, workspace);
}
template <typename T, int D> size_t fwd_ws_impl(const s1f_desc *d, int64_t seg_off, int64_t seg_len) {
  return fwd_workspace<T, D>(fwd_plan<T, D>(d, seg_off, seg_len, kMaxPartBytes).p);
}

// ---- backward ----
// Workspace: the two planes of row statistics, then (256-byte aligned) the partial results of the dQ half, then those of the
// dK/dV half (in the same place if the halves run one after the other).
inline size_t stat_bytes(const s1f_desc *d, int64_t seg_len) {
  return align256(2 * (size_t)d->batch * (size_t)d->n_q_heads * (size_t)seg_len * sizeof(float));
}
template <typename T, int D> struct DkdvFamily {
  typedef BwdDkdvCfg<T, D> Cfg;
  static constexpr int LDS = Cfg::LDS_BYTES, THREADS = 64 * Cfg::WAVES;
  static constexpr int64_t part_bytes = 2 * (int64_t)Cfg::BNW * D * 4;
  static constexpr auto kernel() { return seg_attn_bwd_dkdv_kernel<T, D, Shape<T, D>::KWGS>; }
  static Slots slots() {
    static std::atomic<int64_t> cache[kMaxDevices];
    return resident_slots<kernel()>(LDS, cache, THREADS);
  }
  // iterations of a unit: of one that every row sees, and on average
  static double most_steps(const s1f_desc *d, int64_t seg_len) { return (double)(d->n_q_heads / d->n_kv_heads) * (double)((seg_len + 31) / 32); }
  static double mean_steps(const s1f_desc *d, int64_t seg_off, int64_t seg_len) {
    return most_steps(d, seg_len) * ((double)seg_off + 0.5 * (double)seg_len) / (double)(seg_off + seg_len);
  }
  static SplitPlan plan(const s1f_desc *d, int64_t seg_off, int64_t seg_len, int64_t cap) {
    const int64_t kv_len = seg_off + seg_len, units = (kv_len + Cfg::BNW - 1) / Cfg::BNW * d->n_kv_heads * d->batch;
    SplitPlan p;
    p.n_tiles = (kv_len + Cfg::BNW - 1) / Cfg::BNW;
    p.n_whole = units;
    if (cap <= 0) return p;
    const Slots s = slots();
    if (s.total <= 0) return p;
    const double most = most_steps(d, seg_len), mean = mean_steps(d, seg_off, seg_len);
    double t = 1e300;
    // never more partial results than the built-in scratch holds: s1f_seg_attn_bwd and its _noalloc form then cut alike
    // and add in the same order
    plan_units(&p, &t, 0, p.n_tiles, units, mean, most, Cost<T, D>::dkdv, s, part_bytes, 1, cap < kStaticPartBytes ? cap : kStaticPartBytes);
    return p;
  }
};
// The plans of both halves of a backward, made once per call: the size check and the launches use the same ones.
struct BwdPlans {
  SplitPlan q, k;
  SplitPlan q_both;         // the dQ half in one launch with the other
  bool both = false;        // in one launch, if the workspace holds the partial results of both halves at once
  size_t bytes = 0;         // of the workspace that needs
  size_t apart_bytes = 0;   // of the workspace the halves need one after the other
  size_t k_part = 0;        // in one launch: where the partial results of the dK/dV half begin, behind those of the dQ half
};
// Both halves in one launch: where there is a kernel for the dQ half's tile width, and unless the call is long and the dQ half's
// last round is cut to fill the chip anyway.  One launch / two, backward of a segment, us:
//   tiny and small     4 heads fp32, 256 rows behind 768 keys, head_dim 64 32 -> 24; 8/2 heads, 1051 rows behind 1391 112 -> 94
//   a few rounds       32 heads, 1757 rows behind 6435 keys, head_dim 80 480 -> 453; 64/8 heads, 533 behind 5649, 128 374 -> 327
//   long, dQ uncut     32 heads, head_dim 128, 3983 behind 15556 3166 -> 3129; 80, 2782 behind 29986 2989 -> 2865
//   long, dQ cut       32 heads, head_dim 128, 3652 behind 19539 3599 -> 3547, 3181 behind 26583 4078 -> 4097; 56 heads, 4897 behind
//                      17918 7768 -> 7829, 2898 behind 62638 14797 -> 14859; 64/8 heads, 3606 behind 79334 same: workgroups of the
//                      second half start one by one and no longer walk the same rows side by side
// Over 170 random calls that run in one launch (20 us to 20 ms), time against two: bf16 0.82 on average, worst 1.044 (64/8 heads,
// head_dim 64, 913 rows behind 6179) and 1.028 (3 x 56 heads, head_dim 128, first segment of 267 rows); fp32 0.85, worst 1.008.
constexpr double kBothUs = 3000.0, kLongWalk = 24;
template <typename T, int D> bool both_halves(const s1f_desc *d, int64_t seg_off, int64_t seg_len, const BwdPlans &p) {
  if (!Shape<T, D>::both(p.q_both.nc) || !one_launch(p.q_both.grid() + p.k.grid(), DkdvFamily<T, D>::THREADS)) return false;
  if (p.q.n_split_units == 0) return true;
  // fp32 at head_dim 128, one workgroup to a compute unit: a few workgroups too many for both halves in one round, and the launch lasts as
  // long as the halves one after the other, or longer where the dQ half by itself runs in pairs of tiles.  2/1 heads, 470 rows behind 18102
  // keys, 128 and 146 workgroups: in one launch 251 us, apart 225; over 37 such calls 0.97 to 1.16 times as long.  Not so where the dK/dV units on
  // the diagonal, which are short, make up for them (914 rows behind 15703, 130 workgroups: 147, apart 212), at head_dim 80 (0.87), with
  // more workgroups of the dQ half (592 rows behind 16796, 160 and 136: 217, apart 283), nor where walks are short.
  if (sizeof(T) == 4 && D == 128) {
    const Slots s = DkdvFamily<T, D>::slots();
    const int64_t over = p.q_both.grid() + p.k.grid() - s.total;
    if (s.total == s.cus && over * DkdvFamily<T, D>::Cfg::BNW > seg_len && 4 * over <= s.total && 2 * p.q_both.grid() <= s.cus && p.q_both.n_whole == 0 &&
        p.k.n_split_units == 0 && DkdvFamily<T, D>::most_steps(d, seg_len) >= kLongWalk)
      return false;
  }
  const double cells = ((double)seg_off + 0.5 * (double)seg_len) * (double)seg_len * d->n_q_heads * d->batch;   // (query, key) pairs
  const double step_us = Cost<T, D>::dq.at(p.q.nc, 2) / (64 * p.q.nc) + Cost<T, D>::dkdv.at(0, 2) / 128;        // per 32 of them
  return cells / 32 * step_us / 512 < kBothUs;   // (two workgroups on each of 256 compute units, as the step times presume)
}
// Time of both halves in one launch: groups of workgroups of equal length, handed to the slots in the order of their ids.
struct Group {
  int64_t count;
  double us;
};
double groups_us(const Group (&g)[4], int64_t slots) {
  struct { double at; int64_t count; } ends[5];   // when slots become free, in order (a group adds at most one time)
  int n_ends = 1;
  ends[0] = {0, slots};
  double last = 0;
  for (int i = 0; i < 4; ++i)
    for (int64_t left = g[i].count; left > 0;) {
      const double end = ends[0].at + g[i].us;
      const int64_t now = left < ends[0].count ? left : ends[0].count;
      left -= now;
      last = end > last ? end : last;
      if ((ends[0].count -= now) == 0) {
        for (int x = 1; x < n_ends; ++x) ends[x - 1] = ends[x];
        --n_ends;
      }
      int x = n_ends;
      while (x > 0 && ends[x - 1].at > end) --x;
      for (int y = n_ends; y > x; --y) ends[y] = ends[y - 1];
      ends[x] = {end, now};
      ++n_ends;
    }
  return last;
}
// The cut of the dK/dV half, and the number of chunks of the dQ half where all of its units are cut, for the one launch of a segment
// behind a prefix: its slots and its merge are shared, and as long as there is a compute unit for every workgroup, steps are short.  Each
// half cut as if it ran alone / so, backward of a segment, us: 4 heads fp32, D 64, 256 rows behind 768 25.9 / 23.6; 2 x 8/2 heads, D 64, 350
// behind 389 21.4 / 20.1; 3 heads, D 80, 387 behind 779 23.9 / 19.8; 64/8 heads, D 128, 467 behind 4486 285 / 225.  The prediction is good
// for about 10 %, hence the margin; of first segments, whose units differ in length, it is not (1.25 times slower at worst).
// The halves called one after the other have the same cuts, since they give the same bits.  Hence none that lengthens either by itself:
//   kHalfUs     the longest walk of a half, and of dK/dV all of its rounds, by its step times alone, grow by at most this.  (Without a limit, over 151 random calls: dQ alone up
//               to 1.43 times as long, dK/dV 1.40; 4 heads, D 128, 427 behind 2318, 9 chunks to 3: dQ 17.5 -> 21.7)
//   no more chunks than alone     and of units that stay whole alone, not all, but for few: their sums would wait for a second kernel (8
//               heads, D 80, 403 behind 626, 72 units in 3 chunks: dK/dV 17.8 -> 21.9, the one launch 23.9 -> 26.3)
// Over 220 random calls that get another plan, time against each half cut alone: the one call 0.74 .. 1.03, 0.91 on average, dQ by itself 0.89
// .. 1.07, dK/dV by itself 0.79 .. 1.06, both of them 0.97 on average and 1.03 at most.
// A function of the plan that the dQ half has with the built-in scratch, so that dK and dV do not depend on the workspace.
constexpr int64_t kJointRounds = 8;   // (longer launches: as alone)
constexpr double kHalfUs = 2.25;
constexpr int64_t kFewUnits = 12;    // (an n-th of the compute units)
template <typename T, int D> void plan_together(const s1f_desc *d, int64_t seg_off, int64_t seg_len, BwdPlans *p) {
  typedef DkdvFamily<T, D> K;
  const Slots s = K::slots();
  SplitPlan q = p->q_both, k = p->k;
  const int64_t n_qh = (int64_t)d->n_q_heads * d->batch, uq = q.n_tiles * n_qh, uk = k.n_tiles * d->n_kv_heads * d->batch;
  if (s.total <= 0 || uq + uk > kJointRounds * s.total || seg_off < seg_len) return;
  const double q_mean = (double)seg_off / 32 + (double)(seg_len + 1) / 64 + 1, q_most = (double)(seg_off + seg_len) / 32 + 1;
  const double k_mean = K::mean_steps(d, seg_off, seg_len), k_most = K::most_steps(d, seg_len);
  const int64_t q_bytes = DqFamily<T, D>::row_bytes * 64 * q.nc;
  const bool cut_q = q.n_whole == 0 && q.n_split_units > 0, whole_k = k.n_split_units == 0;
  auto per_cu = [&](int64_t n) { return n >= s.total ? s.total / s.cus : (n + s.cus - 1) / s.cus; };
  auto longest = [](double steps, const SplitPlan &x) { return steps / (x.n_whole > 0 ? 1 : x.n_split); };
  auto rounds = [&](int64_t n) { return n <= s.total ? n > 0 : (n + s.total - 1) / s.total; };
  auto in_rounds = [&](double steps, const SplitPlan &x) { return steps * ((double)rounds(x.n_whole) + (double)rounds(x.chunks()) / x.n_split); };
  auto predict = [&]() {
    const int64_t n = q.grid() + k.grid(), part = (k.chunks() - k.n_split_units) * K::part_bytes;
    if (part > kStaticPartBytes) return 1e300;
    const double q_step = Cost<T, D>::dq.at(q.nc, per_cu(n)), k_step = Cost<T, D>::dkdv.at(0, per_cu(n));
    const double q_one = q_step * longest(q_most, q), k_one = k_step * longest(k_most, k);
    double us = (q_one > k_one ? q_one : k_one) + kRoundUs;   // side by side
    if (n > s.total) {
      const double lq = q_step * q_mean, lk = k_step * k_mean;
      const Group groups[4] = {{q.n_whole, lq + kRoundUs}, {q.chunks(), lq / q.n_split + kRoundUs},
                               {k.n_whole, lk + kRoundUs}, {k.chunks(), lk / k.n_split + kRoundUs}};
      const int a = q_one >= k_one ? 0 : 2;
      const Group in_order[4] = {groups[a], groups[a + 1], groups[2 - a], groups[3 - a]};
      const double all = groups_us(in_order, s.total);
      us = all > 0.75 * us ? all : 0.75 * us;   // (the longest unit shares its compute unit for about half of its life)
    }
    return q.n_split_units + k.n_split_units > 0 ? us + kMergeUs + (double)(q.chunks() * q_bytes + part) / kMergeBytesPerUs : us;
  };
  // What either half may walk by itself, and what others have to beat: the plan as alone, by more than the prediction is good for.
  const double q_limit = longest(q_most, q) + kHalfUs / Cost<T, D>::dq.at(q.nc, per_cu(q.grid()));
  const double k_more = kHalfUs / Cost<T, D>::dkdv.at(0, per_cu(k.grid())), k_limit = longest(k_most, k) + k_more, k_rounds = in_rounds(k_mean, k) + k_more;
  double best = 0.88 * predict();
  // (more units than slots: no cut takes less than all of their steps evenly shared out)
  const double q_all = (double)uq * q_mean * Cost<T, D>::dq.at(q.nc, s.total / s.cus), k_all = (double)uk * k_mean * Cost<T, D>::dkdv.at(0, s.total / s.cus);
  if (uq + uk > s.total && q_all + k_all >= best * s.total) return;
  const double over = (double)uq * q_mean * Cost<T, D>::dq.at(q.nc, 2) / (k_mean * Cost<T, D>::dkdv.at(0, 2)) + (double)uk;
  // units to cut: all, those of the last, partial round if all ran in rounds of the dK/dV half's, and if there were no other half
  const int64_t rests[3] = {uk, ((int64_t)over % s.total + 7) / 8 * 8, uk % s.total};
  const int planned = q.n_split, p_k = k.n_split;
  for (int nq : {planned, 8, 6, 4, 3}) {
    q.n_split = nq;
    if (nq != planned && (!cut_q || nq > planned || longest(q_most, q) > q_limit)) continue;
    for (int n : {1, 2, 3, 4, 5, 6, 8}) {
      if (n > 1 && k_mean < n) break;
      if (!whole_k && n > p_k) break;
      for (int64_t r : rests) {
        if (r == 0 || r > uk || (r < uk && uq + uk < s.total)) continue;
        if (whole_k && n > 1 && r == uk && (n == 2 || kFewUnits * uk > s.cus)) continue;
        k.n_split = n;
        k.n_split_units = n == 1 ? 0 : r;
        k.n_whole = uk - k.n_split_units;
        const double us = longest(k_most, k) > k_limit || in_rounds(k_mean, k) > k_rounds ? 1e300 : predict();
        if (us < (whole_k && n > 1 ? 0.9 : 1.0) * best) {
          best = us;
          p->k = k;
          if (cut_q) p->q.n_split = p->q_both.n_split = nq;
        }
        if (n == 1) break;
      }
    }
  }
}
// The dQ half's plan in one launch with the other.  Whole units give the same bits in tiles of any width.  fp32 above head_dim 64: the
// 64-row tiles run in workgroups of another size than the dK/dV half, and 128 rows in eight waves are faster next to it: 32 heads,
// head_dim 128, backward of 1020 rows 221 -> 160 us, of 980 rows behind 1020 keys 518 -> 450
template <typename T, int D> void one_launch_dq(const s1f_desc *d, int64_t seg_len, BwdPlans *p) {
  p->q_both = p->q;
  if (sizeof(T) == 4 && !Shape<T, D>::both(p->q.nc) && p->q.n_split_units == 0) {
    p->q_both.nc = DqFamily<T, D>::MAX;
    p->q_both.n_tiles = (seg_len + 64 * p->q_both.nc - 1) / (64 * p->q_both.nc);
    p->q_both.n_whole = p->q_both.n_tiles * d->n_q_heads * d->batch;
  }
}
template <typename T, int D> int bwd_plans_impl(const s1f_desc *d, int64_t seg_off, int64_t seg_len, int64_t cap, BwdPlans *p) {
  p->q = plan_rows<DqFamily<T, D>>(d, seg_off, seg_len, cap);
  p->k = DkdvFamily<T, D>::plan(d, seg_off, seg_len, cap);
  one_launch_dq<T, D>(d, seg_len, p);
  if (cap > 0) {
    BwdPlans c = *p;   // as with the built-in scratch
    const bool same = cap <= kStaticPartBytes || p->q.chunks() * 64 * p->q.nc * D * 4 <= kStaticPartBytes;
    if (!same) {
      c.q = plan_rows<DqFamily<T, D>>(d, seg_off, seg_len, kStaticPartBytes);
      one_launch_dq<T, D>(d, seg_len, &c);
    }
    if (both_halves<T, D>(d, seg_off, seg_len, c)) plan_together<T, D>(d, seg_off, seg_len, &c);
    p->k = c.k;
    if (same) {
      p->q = c.q;
      p->q_both = c.q_both;
    }
  }
  const size_t qb = (size_t)(p->q.chunks() * 64 * p->q.nc * D * 4);
  const size_t kb = (size_t)((p->k.chunks() - p->k.n_split_units) * DkdvFamily<T, D>::part_bytes);
  p->both = both_halves<T, D>(d, seg_off, seg_len, *p);
  p->k_part = p->both ? align256(qb) : 0;
  p->apart_bytes = stat_bytes(d, seg_len) + (qb > kb ? qb : kb);
  p->bytes = p->both && kb > 0 ? stat_bytes(d, seg_len) + p->k_part + kb : p->apart_bytes;
  return S1F_OK;
}

template <typename T, int D> int launch_stats(const s1f_desc *d, AttnArgs a, hipStream_t st) {
  // (within one launch wherever both halves are: more than 2^24 workgroups of 64 rows and still fewer than that of wider tiles need
  // 65 rows each, 2^30 in all, and bwd_prepare allows 2^28)
  const int64_t groups = ((int64_t)a.seg_len + 63) / 64, grid = groups * d->n_q_heads * d->batch;
  a.by_groups = Divisor::of(groups);
  void *params[] = {&a};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(seg_attn_bwd_stats_kernel<T, D>), dim3((unsigned)grid), dim3(256),
                                       params, 0, st);
  return e == hipSuccess ? S1F_OK : S1F_EDEVICE;
}
// The merges of the dQ half's `q_units` and the dK/dV half's `k_units` cut units, in one launch.
template <typename T, int D, int MC>
int launch_bwd_merge_of(AttnArgs aq, AttnArgs ak, int64_t q_groups, int64_t k_groups, hipStream_t st) {
  int n = (int)q_groups;
  if (q_groups > 0) aq.by_groups = Divisor::of(MergeRows<D>::groups(aq.bm));
  void *params[] = {&aq, &ak, &n};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(seg_attn_bwd_merge_kernel<T, D, MC>),
                                       dim3((unsigned)(q_groups + k_groups)), dim3(256), params, 0, st);
  return e == hipSuccess ? S1F_OK : S1F_EDEVICE;
}
template <typename T, int D>
int launch_bwd_merge(const AttnArgs &aq, const AttnArgs &ak, int64_t q_units, int64_t k_units, hipStream_t st) {
  if (q_units + k_units == 0) return S1F_OK;
  const int64_t q_groups = q_units * MergeRows<D>::groups(aq.bm), k_groups = k_units * DkdvMerge<D>::GROUPS;
  const int pq = q_units > 0 ? aq.n_split : 0, pk = k_units > 0 ? ak.n_split - 1 : 0, parts = pq > pk ? pq : pk;
  return parts <= 2   ? launch_bwd_merge_of<T, D, 2>(aq, ak, q_groups, k_groups, st)
         : parts <= 4 ? launch_bwd_merge_of<T, D, 4>(aq, ak, q_groups, k_groups, st)
         : parts <= 8 ? launch_bwd_merge_of<T, D, 8>(aq, ak, q_groups, k_groups, st)
                      : launch_bwd_merge_of<T, D, kMaxChunks>(aq, ak, q_groups, k_groups, st);
}
// The arguments of either half's launch; k_part: see BwdPlans.
template <typename T, int D> AttnArgs dq_args(const s1f_desc *d, AttnArgs a, const SplitPlan &p) {
  a.part = reinterpret_cast<float *>(reinterpret_cast<char *>(a.delta) + stat_bytes(d, a.seg_len));
  fill_launch(&a, (int64_t)d->n_q_heads * d->batch, row_tile_order(d, a), p);
  return a;
}
template <typename T, int D> AttnArgs dkdv_args(const s1f_desc *d, AttnArgs a, const SplitPlan &p, size_t k_part) {
  a.part = reinterpret_cast<float *>(reinterpret_cast<char *>(a.delta) + stat_bytes(d, a.seg_len) + k_part);
  fill_launch(&a, (int64_t)d->n_kv_heads * d->batch, 2 * (int64_t)a.seg_off < (int64_t)a.seg_len, p);
  return a;
}

template <typename T, int D> int bwd_dq_impl(const s1f_desc *d, const AttnArgs &a0, const SplitPlan &p, hipStream_t st) {
  if (!one_launch(p.grid(), DqFamily<T, D>::threads(p.nc)))
    return in_halves<T>(d, a0, [&](const s1f_desc *half, const AttnArgs &x) {
      return bwd_dq_impl<T, D>(half, x, p.uncut((int64_t)d->n_q_heads * half->batch), st);
    });
  const AttnArgs a = dq_args<T, D>(d, a0, p);
  int rc;
  if (dq_in_pairs<T, D>(a, p)) {
    SplitPlan pairs = p;
    pairs.n_split *= 2;
    rc = launch<DqFamily<T, D>::pair_kernel()>(DqFamily<T, D>::LDS, pairs, a.n_bh, a, st, DqFamily<T, D>::threads(1));
  } else {
    rc = launch_rows<DqFamily<T, D>>(p, a.n_bh, a, st);
  }
  return rc == S1F_OK ? launch_bwd_merge<T, D>(a, a, p.n_split_units, 0, st) : rc;
}

template <typename T, int D> int bwd_dkdv_impl(const s1f_desc *d, const AttnArgs &a0, const SplitPlan &p, hipStream_t st) {
  typedef DkdvFamily<T, D> F;
  if (!one_launch(p.grid(), F::THREADS))
    return in_halves<T>(d, a0, [&](const s1f_desc *half, const AttnArgs &x) {
      return bwd_dkdv_impl<T, D>(half, x, p.uncut((int64_t)d->n_kv_heads * half->batch), st);
    });
  const AttnArgs a = dkdv_args<T, D>(d, a0, p, 0);
  const int rc = launch<F::kernel()>(F::LDS, p, a.n_bh, a, st, F::THREADS);
  return rc == S1F_OK ? launch_bwd_merge<T, D>(a, a, 0, p.n_split_units, st) : rc;
}

template <typename T, int D, int NC> constexpr auto both_kernel() {
  constexpr int W = Shape<T, D>::waves(NC);
  return seg_attn_bwd_kernel<T, D, 4 * NC / W, Shape<T, D>::BOTH_OCC, W>;
}
template <typename T, int D> constexpr int kBothLds =
    TileRing<T, D>::LDS_BYTES > BwdDkdvCfg<T, D>::LDS_BYTES ? TileRing<T, D>::LDS_BYTES : BwdDkdvCfg<T, D>::LDS_BYTES;
template <typename T, int D, int NC>
int launch_both(const BwdPlans &p, AttnArgs aq, AttnArgs ak, int dq_first, hipStream_t st) {
  const int rc = prepare<both_kernel<T, D, NC>()>(kBothLds<T, D>);
  if (rc != S1F_OK) return rc;
  int first = (int)(dq_first ? p.q_both.grid() : p.k.grid());
  void *params[] = {&aq, &ak, &first, &dq_first};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(both_kernel<T, D, NC>()), dim3((unsigned)(p.q_both.grid() + p.k.grid())),
                                       dim3(DkdvFamily<T, D>::THREADS), params, (size_t)kBothLds<T, D>, st);
  return e == hipSuccess ? S1F_OK : S1F_EDEVICE;
}
// The longer units first: those of the other half then fill the gaps at the end.
template <typename T, int D> bool dq_half_first(const AttnArgs &a, const BwdPlans &p) {
  const double q_us = ((double)a.seg_off + 0.5 * a.seg_len) / 32 * Cost<T, D>::dq.at(p.q_both.nc, 2) / (p.q_both.n_whole > 0 ? 1 : p.q_both.n_split);
  const double k_us = (double)a.group * ((a.seg_len + 31) / 32) * Cost<T, D>::dkdv.at(0, 2) / (p.k.n_whole > 0 ? 1 : p.k.n_split);
  return q_us >= k_us;
}
template <typename T, int D> int bwd_both_impl(const s1f_desc *d, const AttnArgs &a, const BwdPlans &p, hipStream_t st) {
  const AttnArgs aq = dq_args<T, D>(d, a, p.q_both), ak = dkdv_args<T, D>(d, a, p.k, p.k_part);
  const int dq_first = dq_half_first<T, D>(a, p);
  int rc = launch_stats<T, D>(d, a, st);
  if (rc != S1F_OK) return rc;
  rc = S1F_EUNSUPPORTED;
  if constexpr (Shape<T, D>::both(3)) { if (p.q_both.nc == 3) rc = launch_both<T, D, 3>(p, aq, ak, dq_first, st); }
  if constexpr (Shape<T, D>::both(2)) { if (p.q_both.nc == 2) rc = launch_both<T, D, 2>(p, aq, ak, dq_first, st); }
  if constexpr (Shape<T, D>::both(1)) { if (p.q_both.nc == 1) rc = launch_both<T, D, 1>(p, aq, ak, dq_first, st); }
  return rc == S1F_OK ? launch_bwd_merge<T, D>(aq, ak, p.q_both.n_split_units, p.k.n_split_units, st) : rc;
}

// What a launch of either backward kernel could be refused for before it reaches the runtime.
template <typename F, int NC> int prepare_rows() {
  const int rc = prepare<F::template kernel<NC>()>(F::LDS);
  if constexpr (NC > 1) return rc != S1F_OK ? rc : prepare_rows<F, NC - 1>();
  return rc;
}
template <typename T, int D, int NC> int prepare_both() {
  int rc = S1F_OK;
  if constexpr (Shape<T, D>::both(NC)) rc = prepare<both_kernel<T, D, NC>()>(kBothLds<T, D>);
  if constexpr (NC > 1) return rc != S1F_OK ? rc : prepare_both<T, D, NC - 1>();
  return rc;
}
template <typename T, int D> int bwd_ready_impl(const s1f_desc *d, const AttnArgs &a, const BwdPlans &p) {
  const int64_t kv_tiles = ((int64_t)a.seg_off + a.seg_len + DkdvFamily<T, D>::Cfg::BNW - 1) / DkdvFamily<T, D>::Cfg::BNW;
  const int64_t row_tiles = ((int64_t)a.seg_len + 63) / 64;
  if (kv_tiles * d->n_kv_heads * d->batch > 0x7fffffff || row_tiles * d->n_q_heads * d->batch > 0x7fffffff) return S1F_EUNSUPPORTED;
  if (!one_launch(p.q.n_tiles * d->n_q_heads, DqFamily<T, D>::threads(p.q.nc)) ||
      !one_launch(p.k.n_tiles * d->n_kv_heads, DkdvFamily<T, D>::THREADS))   // one batch entry: not to be halved further
    return S1F_EUNSUPPORTED;
  if (p.both) return prepare_both<T, D, DqFamily<T, D>::MAX>();
  const int rc = prepare_rows<DqFamily<T, D>, DqFamily<T, D>::MAX>();
  return rc != S1F_OK ? rc : prepare<DkdvFamily<T, D>::kernel()>(DkdvFamily<T, D>::LDS);
}

// What s1f_launch_plan reports.
template <typename T, int D> int plan_impl(const s1f_desc *d, const AttnArgs &a, int launch, int64_t cap, int64_t *out) {
  SplitPlan p;
  int64_t whole = 0;
  const bool fwd = launch == S1F_PLAN_FWD || launch == S1F_PLAN_FWD_WS;
  int keys_nc = 0;
  if (fwd) {
    const FwdPlan f = fwd_plan<T, D>(d, a.seg_off, a.seg_len, cap);
    p = f.p;
    keys_nc = f.keys_nc;
  } else {
    BwdPlans b;
    bwd_plans_impl<T, D>(d, a.seg_off, a.seg_len, cap, &b);
    p = launch == S1F_PLAN_DQ ? b.q : b.k;
  }
  const bool tail = fwd && keys_nc == 0 && row_tail_of<FwdFamily<T, D>>(a, p, &whole);
  out[0] = launch == S1F_PLAN_DKDV ? DkdvFamily<T, D>::Cfg::BNW : keys_nc > 0 ? 16 * keys_nc : 64 * p.nc;
  out[1] = tail ? whole : p.n_whole;
  out[2] = p.n_split_units;
  out[3] = p.n_split;
  out[4] = tail ? p.n_whole - whole : 0;
  return S1F_OK;
}

// What s1f_launch_paths reports.
template <typename T, int D> int paths_impl(const s1f_desc *d, const AttnArgs &a, int64_t *out) {
  BwdPlans p, small;
  bwd_plans_impl<T, D>(d, a.seg_off, a.seg_len, kMaxPartBytes, &p);
  bwd_plans_impl<T, D>(d, a.seg_off, a.seg_len, kStaticPartBytes, &small);
  Tail t;
  const FwdPlan f = fwd_plan<T, D>(d, a.seg_off, a.seg_len, 0);
  if (f.keys_nc == 0) fwd_tail<FwdFamily<T, D>>(a, f.p, (int64_t)d->n_q_heads * d->batch, &t);
  out[0] = p.both;
  out[1] = 64 * (p.both ? p.q_both.nc : p.q.nc);
  out[2] = p.both && dq_half_first<T, D>(a, p);
  out[3] = small.both;
  out[4] = t.rag;
  return S1F_OK;
}

#define S1F_DISPATCH(fn, d, ...)                                                        \
  do {                                                                                  \
    if ((d)->dtype == S1F_BF16) {                                                       \
      switch ((d)->head_dim) {                                                          \
        case 64: return fn<bf16_t, 64>(__VA_ARGS__);                                    \
        case 80: return fn<bf16_t, 80>(__VA_ARGS__);                                    \
        case 128: return fn<bf16_t, 128>(__VA_ARGS__);                                  \
      }                                                                                 \
    } else {                                                                            \
      switch ((d)->head_dim) {                                                          \
        case 64: return fn<float, 64>(__VA_ARGS__);                                     \
        case 80: return fn<float, 80>(__VA_ARGS__);                                     \
        case 128: return fn<float, 128>(__VA_ARGS__);                                   \
      }                                                                                 \
    }                                                                                   \
    return S1F_EUNSUPPORTED;                                                            \
  } while (0)

}  // namespace

namespace {
int fwd_entry(const s1f_desc *desc, const void *q_seg, const void *k_prefix, const void *v_prefix, int64_t seg_off,
              int64_t seg_len, void *out, float *lse, void *workspace, size_t workspace_bytes, bool split,
              void *hip_stream) {
  int rc = check_desc(desc);
  if (rc != S1F_OK) return rc;
  if (!q_seg || !k_prefix || !v_prefix || !out || !lse) return S1F_EINVAL;
  if (!aligned16(q_seg) || !aligned16(k_prefix) || !aligned16(v_prefix) || !aligned16(out)) return S1F_EINVAL;
  if (workspace_bytes > 0 && (!workspace || !aligned16(workspace))) return S1F_EINVAL;
  rc = check_seg(desc, seg_off, seg_len);
  if (rc != S1F_OK) return rc;
  AttnArgs a = make_args(desc, seg_off, seg_len);
  a.q = q_seg; a.k = k_prefix; a.v = v_prefix; a.out_w = out; a.lse = lse;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  S1F_DISPATCH(fwd_impl, desc, desc, a, st, workspace, workspace_bytes, split);
}
// (callers have validated the descriptor: the dispatches below always find their kernel)
size_t fwd_ws_dispatch(const s1f_desc *d, int64_t seg_off, int64_t seg_len) {
  S1F_DISPATCH(fwd_ws_impl, d, d, seg_off, seg_len);
}
int bwd_plans_dispatch(const s1f_desc *d, int64_t seg_off, int64_t seg_len, int64_t cap, BwdPlans *p) {
  S1F_DISPATCH(bwd_plans_impl, d, d, seg_off, seg_len, cap, p);
}
}  // namespace

extern "C" int s1f_seg_attn_fwd(const s1f_desc *desc, const void *q_seg, const void *k_prefix, const void *v_prefix,
                                int64_t seg_off, int64_t seg_len, void *out, float *lse, void *hip_stream) {
  return fwd_entry(desc, q_seg, k_prefix, v_prefix, seg_off, seg_len, out, lse, nullptr, 0, false, hip_stream);
}

extern "C" size_t s1f_fwd_workspace_bytes(const s1f_desc *desc, int64_t seg_off, int64_t seg_len) {
  if (check_desc(desc) != S1F_OK || check_seg(desc, seg_off, seg_len) != S1F_OK) return 0;
  return fwd_ws_dispatch(desc, seg_off, seg_len);
}

extern "C" int s1f_seg_attn_fwd_ws(const s1f_desc *desc, const void *q_seg, const void *k_prefix, const void *v_prefix,
                                   int64_t seg_off, int64_t seg_len, void *out, float *lse, void *workspace,
                                   size_t workspace_bytes, void *hip_stream) {
  return fwd_entry(desc, q_seg, k_prefix, v_prefix, seg_off, seg_len, out, lse, workspace, workspace_bytes, true, hip_stream);
}

extern "C" size_t s1f_bwd_workspace_bytes(const s1f_desc *desc, int64_t seg_off, int64_t seg_len) {
  if (check_desc(desc) != S1F_OK || check_seg(desc, seg_off, seg_len) != S1F_OK) return 0;
  BwdPlans p;
  bwd_plans_dispatch(desc, seg_off, seg_len, kMaxPartBytes, &p);
  return p.bytes;
}

namespace {
int bwd_dq_dispatch(const s1f_desc *d, const AttnArgs &a, const BwdPlans &p, hipStream_t st) {
  S1F_DISPATCH(bwd_dq_impl, d, d, a, p.q, st);
}
int bwd_dkdv_dispatch(const s1f_desc *d, const AttnArgs &a, const BwdPlans &p, hipStream_t st) {
  S1F_DISPATCH(bwd_dkdv_impl, d, d, a, p.k, st);
}

int bwd_both_dispatch(const s1f_desc *d, const AttnArgs &a, const BwdPlans &p, hipStream_t st) {
  S1F_DISPATCH(bwd_both_impl, d, d, a, p, st);
}
int bwd_ready_dispatch(const s1f_desc *d, const AttnArgs &a, const BwdPlans &p) { S1F_DISPATCH(bwd_ready_impl, d, d, a, p); }

// Validation shared by the backward entry points; fills `a` and `plans` on success.
int bwd_prepare(const s1f_desc *desc, const void *dout, const void *q_seg, const void *k_prefix, const void *v_prefix,
                const float *lse, int64_t seg_off, int64_t seg_len, const void *workspace, size_t workspace_bytes,
                AttnArgs *a, BwdPlans *plans, int64_t part_cap = kMaxPartBytes) {
  int rc = check_desc(desc);
  if (rc != S1F_OK) return rc;
  if (!dout || !q_seg || !k_prefix || !v_prefix || !lse || !workspace) return S1F_EINVAL;
  if (!aligned16(dout) || !aligned16(q_seg) || !aligned16(k_prefix) || !aligned16(v_prefix) || !aligned16(workspace))
    return S1F_EINVAL;
  rc = check_seg(desc, seg_off, seg_len);
  if (rc != S1F_OK) return rc;
  bwd_plans_dispatch(desc, seg_off, seg_len, part_cap, plans);
  if (workspace_bytes < plans->bytes) plans->both = false;
  if (workspace_bytes < plans->apart_bytes) {
    // fp32 runs with any workspace that holds the row statistics; its launches are then left whole
    if (desc->dtype == S1F_BF16 || workspace_bytes < stat_bytes(desc, seg_len)) return S1F_EINVAL;
    bwd_plans_dispatch(desc, seg_off, seg_len, 0, plans);
  }
  // the asynchronous copies address the workspace with 32-bit byte offsets
  const int64_t stat_rows = (int64_t)desc->batch * desc->n_q_heads * seg_len;
  if (stat_rows > (int64_t(1) << 28)) return S1F_EUNSUPPORTED;
  *a = make_args(desc, seg_off, seg_len);
  a->q = q_seg; a->k = k_prefix; a->v = v_prefix; a->dout = dout;
  a->lse = const_cast<float *>(lse);
  a->delta = reinterpret_cast<float *>(const_cast<void *>(workspace));
  a->ws_plane = stat_rows;
  return S1F_OK;
}

// s1f_seg_attn_bwd; `part_cap` bounds the partial dQ rows a split dQ launch may leave behind the statistics.
int bwd_entry(const s1f_desc *desc, const void *dout, const void *q_seg, const void *k_prefix, const void *v_prefix,
              const void *out, const float *lse, int64_t seg_off, int64_t seg_len, void *dq, float *dk_prefix_acc,
              float *dv_prefix_acc, void *workspace, size_t workspace_bytes, int64_t part_cap, void *hip_stream) {
  AttnArgs a;
  BwdPlans p;
  const int rc = bwd_prepare(desc, dout, q_seg, k_prefix, v_prefix, lse, seg_off, seg_len, workspace, workspace_bytes, &a, &p,
                             part_cap);
  if (rc != S1F_OK) return rc;
  if (!out || !dq || !dk_prefix_acc || !dv_prefix_acc) return S1F_EINVAL;
  if (!aligned16(out) || !aligned16(dq) || !aligned16(dk_prefix_acc) || !aligned16(dv_prefix_acc)) return S1F_EINVAL;
  a.out = out; a.dq = dq; a.dk_acc = dk_prefix_acc; a.dv_acc = dv_prefix_acc;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  // everything that can fail short of the launches themselves happens before the first kernel is enqueued
  int rc2 = bwd_ready_dispatch(desc, a, p);
  if (rc2 == S1F_OK && p.both) return bwd_both_dispatch(desc, a, p, st);
  if (rc2 == S1F_OK) rc2 = bwd_dq_dispatch(desc, a, p, st);
  return rc2 == S1F_OK ? bwd_dkdv_dispatch(desc, a, p, st) : rc2;
}
}  // namespace

extern "C" int s1f_seg_attn_bwd_dq(const s1f_desc *desc, const void *dout, const void *q_seg, const void *k_prefix,
                                   const void *v_prefix, const void *out, const float *lse, int64_t seg_off,
                                   int64_t seg_len, void *dq, void *workspace, size_t workspace_bytes,
                                   void *hip_stream) {
  AttnArgs a;
  BwdPlans p;
  const int rc = bwd_prepare(desc, dout, q_seg, k_prefix, v_prefix, lse, seg_off, seg_len, workspace, workspace_bytes, &a, &p);
  if (rc != S1F_OK) return rc;
  if (!out || !dq || !aligned16(out) || !aligned16(dq)) return S1F_EINVAL;
  a.out = out; a.dq = dq;
  return bwd_dq_dispatch(desc, a, p, reinterpret_cast<hipStream_t>(hip_stream));
}

extern "C" int s1f_seg_attn_bwd_dkdv(const s1f_desc *desc, const void *dout, const void *q_seg, const void *k_prefix,
                                     const void *v_prefix, const float *lse, int64_t seg_off, int64_t seg_len,
                                     float *dk_prefix_acc, float *dv_prefix_acc, const void *workspace,
                                     size_t workspace_bytes, void *hip_stream) {
  AttnArgs a;
  BwdPlans p;
  const int rc = bwd_prepare(desc, dout, q_seg, k_prefix, v_prefix, lse, seg_off, seg_len, workspace, workspace_bytes, &a, &p);
  if (rc != S1F_OK) return rc;
  if (!dk_prefix_acc || !dv_prefix_acc || !aligned16(dk_prefix_acc) || !aligned16(dv_prefix_acc)) return S1F_EINVAL;
  a.dk_acc = dk_prefix_acc; a.dv_acc = dv_prefix_acc;
  return bwd_dkdv_dispatch(desc, a, p, reinterpret_cast<hipStream_t>(hip_stream));
}

extern "C" int s1f_seg_attn_bwd(const s1f_desc *desc, const void *dout, const void *q_seg, const void *k_prefix,
                                const void *v_prefix, const void *out, const float *lse, int64_t seg_off,
                                int64_t seg_len, void *dq, float *dk_prefix_acc, float *dv_prefix_acc,
                                void *workspace, size_t workspace_bytes, void *hip_stream) {
  return bwd_entry(desc, dout, q_seg, k_prefix, v_prefix, out, lse, seg_off, seg_len, dq, dk_prefix_acc, dv_prefix_acc,
                   workspace, workspace_bytes, kMaxPartBytes, hip_stream);
}

// ---- the backward for callers that cannot allocate --------------------------------------------------------------
// Its row statistics live in a device array that is part of the library's code object instead of a workspace
// argument.  In host code the array's name is only a handle: its device address is looked up once per device
// (each device holds its own copy) and that address is what the kernels receive.
namespace {
constexpr int64_t kStaticStatRows = int64_t(1) << 21;            // batch * n_q_heads * seg_len the array holds
// two planes of row statistics (16 MiB), then the partial results of either half (at most kStaticPartBytes each)
constexpr size_t kStaticScratchBytes = 2 * (size_t)kStaticStatRows * sizeof(float) + 2 * (size_t)kStaticPartBytes;
static __device__ __align__(256) float scratch[kStaticScratchBytes / sizeof(float)];

std::mutex scratch_mutex;
float *scratch_ptr[kMaxDevices];   // device address of `scratch` on each device, null until looked up

int static_scratch(float **out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return S1F_EDEVICE;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (scratch_ptr[dev] == nullptr) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return S1F_EDEVICE;
    scratch_ptr[dev] = static_cast<float *>(p);
  }
  *out = scratch_ptr[dev];
  return S1F_OK;
}
}  // namespace

extern "C" size_t s1f_static_scratch_rows(void) { return (size_t)kStaticStatRows; }

extern "C" int s1f_seg_attn_bwd_noalloc(const s1f_desc *desc, const void *dout, const void *q_seg, const void *k_prefix,
                                        const void *v_prefix, const void *out, const float *lse, int64_t seg_off,
                                        int64_t seg_len, void *dq, float *dk_prefix_acc, float *dv_prefix_acc,
                                        void *hip_stream) {
  int rc = check_desc(desc);
  if (rc != S1F_OK) return rc;
  rc = check_seg(desc, seg_off, seg_len);
  if (rc != S1F_OK) return rc;
  if ((int64_t)desc->batch * desc->n_q_heads * seg_len > kStaticStatRows) return S1F_ESCRATCH;
  float *ws = nullptr;
  rc = static_scratch(&ws);
  if (rc != S1F_OK) return rc;
  // every plane entry that is read is written by the same call before (by the statistics kernel, or by the dQ kernel where the halves
  // run one after the other): nothing to clear
  return bwd_entry(desc, dout, q_seg, k_prefix, v_prefix, out, lse, seg_off, seg_len, dq, dk_prefix_acc, dv_prefix_acc, ws,
                   kStaticScratchBytes, kStaticPartBytes, hip_stream);
}

extern "C" int s1f_launch_plan(const s1f_desc *desc, int32_t launch, int64_t seg_off, int64_t seg_len, int64_t *plan) {
  int rc = check_desc(desc);
  if (rc != S1F_OK) return rc;
  if (plan == nullptr || launch < S1F_PLAN_FWD || launch > S1F_PLAN_DKDV) return S1F_EINVAL;
  rc = check_seg(desc, seg_off, seg_len);
  if (rc != S1F_OK) return rc;
  const AttnArgs a = make_args(desc, seg_off, seg_len);
  S1F_DISPATCH(plan_impl, desc, desc, a, launch, launch == S1F_PLAN_FWD ? 0 : kMaxPartBytes, plan);
}

extern "C" int s1f_launch_paths(const s1f_desc *desc, int64_t seg_off, int64_t seg_len, int64_t *paths) {
  int rc = check_desc(desc);
  if (rc != S1F_OK) return rc;
  if (paths == nullptr) return S1F_EINVAL;
  rc = check_seg(desc, seg_off, seg_len);
  if (rc != S1F_OK) return rc;
  const AttnArgs a = make_args(desc, seg_off, seg_len);
  S1F_DISPATCH(paths_impl, desc, desc, a, paths);
}

extern "C" const char *s1f_strerror(int status) {
  switch (status) {
    case S1F_OK: return "ok";
    case S1F_EINVAL: return "invalid argument (null or misaligned pointer, bad size or stride, workspace too small)";
    case S1F_EUNSUPPORTED: return "unsupported dtype or head_dim (supported: f32/bf16 with head_dim 64, 80, 128)";
    case S1F_ERANGE: return "segment out of range (seg_off < 0, seg_len < 1 or seg_off + seg_len > kv_capacity)";
    case S1F_EDEVICE: return "HIP runtime error at kernel launch";
    case S1F_ESCRATCH:
      return "batch * n_q_heads * seg_len exceeds the built-in scratch of s1f_seg_attn_bwd_noalloc "
             "(s1f_static_scratch_rows); use s1f_seg_attn_bwd with a workspace";
    default: return "unknown status";
  }
}

extern "C" int s1f_version(void) { return 200; }

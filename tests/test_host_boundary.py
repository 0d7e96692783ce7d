"""CPU-only checks of the boundary: the shared library loads, exports every symbol the header declares,
validates arguments before touching a device, and its partitioner agrees bit for bit with the oracle."""
import ctypes
import os
import re

import pytest

import paper_2406_03488_amd as s1f
from paper_2406_03488_amd import binding
from oracle import partition as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "s1f.h")).read()
    names = set(re.findall(r"\b(s1f_[a-z_0-9]+)\s*\(", header))
    assert {"s1f_partition", "s1f_seg_attn_fwd", "s1f_seg_attn_bwd", "s1f_bwd_workspace_bytes", "s1f_strerror",
            "s1f_version"} <= names
    lib = s1f.load_library()
    for name in names:
        assert hasattr(lib, name), name
    assert s1f.version() >= 100


@pytest.mark.parametrize("args", [(8, 2, 1, 1), (6, 3, 1, 1), (100, 4, 8, 2), (1000, 7, 64, 8), (4096, 8, 512, 8),
                                  (999, 3, 1, 1), (37, 1, 16, 4), (9, 9, 16, 4), (8192, 4, 2560, 32),
                                  (32768, 8, 4096, 32), (65536, 16, 7168, 56), (131072, 32, 8192, 64),
                                  (64, 4, 10**6, 1), (10000, 5, 1, 1), (24, 23, 3, 1), (50, 49, 1, 1)])
def test_partition_matches_oracle_bit_exact(args):
    assert s1f.partition(*args) == P.partition(*args)


def test_partition_matches_oracle_sweep():
    for n in range(1, 40):
        for k in range(1, min(n, 6) + 1):
            for hidden in (1, 2, 5, 64):
                assert s1f.partition(n, k, hidden, 1) == P.partition(n, k, hidden, 1), (n, k, hidden)


def test_partition_rejects_bad_arguments():
    for bad in ((8, 0, 4, 1), (3, 4, 4, 1), (8, 2, 0, 1), (8, 2, 4, 0), (8, 2, 6, 4)):
        with pytest.raises(s1f.S1FError) as e:
            s1f.partition(*bad)
        assert e.value.status == 1
    lib = s1f.load_library()
    assert lib.s1f_partition(8, 2, 4, 1, None) == 1


def test_partition_ex_additive_matches_oracle():
    for n, k, hidden, align in ((8, 2, 1, 2), (8, 2, 1, 3), (64, 4, 1, 4), (100, 3, 2, 8), (257, 5, 4, 16), (50, 2, 1, 7),
                                (4096, 8, 512, 128), (32768, 8, 4096, 128), (32768, 8, 4096, 256), (8192, 4, 2560, 64),
                                (1000, 7, 64, 1), (129, 2, 8, 128), (300, 3, 1, 100)):
        assert s1f.partition_ex(n, k, hidden, 1, s1f.COST_ADDITIVE, align) == P.partition(n, k, hidden, 1, align)
    for n in range(1, 30):
        for k in range(1, 5):
            for align in (1, 2, 3, 5):
                if (n - 1) // align < k - 1 or n < k:
                    continue
                assert s1f.partition_ex(n, k, 3, 1, 0, align) == P.partition(n, k, 3, 1, align), (n, k, align)
    assert s1f.partition_ex(32768, 8, 4096, 32) == s1f.partition(32768, 8, 4096, 32)


def test_partition_ex_literal_matches_oracle():
    for n, k, hidden, align in ((8, 2, 1, 1), (6, 3, 1, 1), (8, 2, 1, 4), (100, 4, 8, 1), (300, 7, 16, 1), (257, 5, 4, 16),
                                (400, 8, 64, 8), (64, 64, 2, 1), (90, 3, 1000, 1), (350, 6, 1, 1), (385, 4, 12, 128)):
        assert s1f.partition_ex(n, k, hidden, 1, s1f.COST_LITERAL, align) == P.partition_literal(n, k, hidden, 1, align)
    for n in range(1, 26):
        for k in range(1, 5):
            for align in (1, 2, 4):
                if (n - 1) // align < k - 1 or n < k:
                    continue
                for hidden in (1, 7):
                    assert (s1f.partition_ex(n, k, hidden, 1, 1, align)
                            == P.partition_literal(n, k, hidden, 1, align)), (n, k, hidden, align)


@pytest.mark.parametrize("n,k,hidden,align", [(8192, 4, 2560, 1), (32768, 8, 4096, 1), (65536, 16, 7168, 1),
                                              (131072, 32, 8192, 1), (32768, 8, 4096, 128)])
def test_partition_ex_literal_full_size_is_optimal(n, k, hidden, align):
    """At sizes the quadratic oracle cannot reach: the bound T reached is feasible, T - 1 is not (left-to-right
    greedy: each segment as long as T - 1 allows), and no boundary can move left on its own."""
    b = s1f.partition_ex(n, k, hidden, 1, s1f.COST_LITERAL, align)
    assert b[0] == 0 and b[-1] == n and all(x < y for x, y in zip(b[:-1], b[1:]))
    assert all(x % align == 0 for x in b[1:-1])
    costs = [P.literal_cost(x, y, hidden) for x, y in zip(b[:-1], b[1:])]
    T = max(costs)

    def segments_needed(bound):
        a, used = 0, 0
        while a < n:
            # largest y with (y - a)(12 hidden + y) <= bound, by bisection; n itself is always a candidate
            lo, hi = a, n
            while lo < hi:
                mid = (lo + hi + 1) // 2
                if P.literal_cost(a, mid, hidden) <= bound:
                    lo = mid
                else:
                    hi = mid - 1
            y = lo if lo == n else lo // align * align
            if y <= a:
                return None
            a, used = y, used + 1
        return used
    assert segments_needed(T) <= k
    fewer = segments_needed(T - 1)
    assert fewer is None or fewer > k
    for i in range(1, k):                         # lexicographic minimality, one boundary at a time
        moved = b[:i] + [b[i] - align] + b[i + 1:]
        if moved[i] <= moved[i - 1]:
            continue
        assert max(P.literal_cost(x, y, hidden) for x, y in zip(moved[:-1], moved[1:])) > T


def test_partition_rebalance_matches_oracle():
    import random
    rng = random.Random(20240603)
    for _ in range(200):
        k = rng.randint(1, 6)
        align = rng.choice((1, 1, 2, 4, 8))
        lens = [rng.randint(1, 40) for _ in range(k)]
        b = [0]
        for x in lens:
            b.append(b[-1] + x)
        cost = [rng.choice((0, rng.randint(1, 1000), rng.randint(1, 10**9))) for _ in range(k)]
        if sum(cost) == 0 or (b[-1] - 1) // align < k - 1:
            with pytest.raises(s1f.S1FError):
                s1f.partition_rebalance(b, cost, align)
            continue
        assert s1f.partition_rebalance(b, cost, align) == P.rebalance(b, cost, align), (b, cost, align)
    assert s1f.partition_rebalance([0, 10, 20, 30], [10, 20, 30]) == [0, 15, 23, 30]
    assert s1f.partition_rebalance([0, 10, 20, 30], [10, 20, 30], 4) == [0, 16, 24, 30]
    big = s1f.partition(32768, 8, 4096, 32)
    ns = [1_900_000_000 + 37 * i for i in range(8)]
    assert s1f.partition_rebalance(big, ns, 128) == P.rebalance(big, ns, 128)


def test_partition_variants_reject_bad_arguments():
    for bad in ((8, 3, 1, 1, 0, 4), (8, 2, 1, 1, 0, 0), (15, 4, 1, 1, 1, 5), (8, 2, 1, 1, 2, 1), (8, 2, 6, 4, 1, 1)):
        with pytest.raises(s1f.S1FError) as e:
            s1f.partition_ex(*bad)
        assert e.value.status == 1
    for b, c, a in (([0, 4, 4, 8], [1, 1, 1], 1), ([1, 4, 8], [1, 1], 1), ([0, 4, 8], [0, 0], 1), ([0, 4, 8], [1, -1], 1),
                    ([0, 4, 8], [1, 1], 0), ([0, 1, 2, 3], [1, 1, 1], 2), ([0, 4, 8], [1 << 48, 1], 1)):
        with pytest.raises(s1f.S1FError):
            s1f.partition_rebalance(b, c, a)
    lib = s1f.load_library()
    assert lib.s1f_partition_ex(8, 2, 4, 1, 0, 1, None) == 1
    assert lib.s1f_partition_rebalance(2, None, None, 1, None) == 1


def _desc(**kw):
    base = dict(batch=1, n_q_heads=4, n_kv_heads=2, head_dim=64, dtype=1, reserved=0, q_stride_b=4 * 256 * 64,
                q_stride_h=256 * 64, q_stride_s=64, kv_stride_b=2 * 512 * 64, kv_stride_h=512 * 64, kv_stride_s=64,
                kv_capacity=512)
    base.update(kw)
    return binding.Desc(**base)


def test_attention_entry_points_validate_before_any_launch():
    """Every call below must fail in validation (no GPU is present or needed)."""
    lib = s1f.load_library()
    p = ctypes.c_void_p(4096)   # non-null, 16-byte aligned, never dereferenced

    def fwd(desc, seg_off=0, seg_len=256, q=p, lse=p):
        return lib.s1f_seg_attn_fwd(ctypes.byref(desc), q, p, p, seg_off, seg_len, p, lse, None)

    assert fwd(_desc(), q=None) == 1
    assert fwd(_desc(), lse=None) == 1
    assert fwd(_desc(), q=ctypes.c_void_p(4100)) == 1            # misaligned
    assert fwd(_desc(n_kv_heads=3)) == 1
    assert fwd(_desc(q_stride_s=60)) == 1
    assert fwd(_desc(kv_stride_h=513 * 64 + 1)) == 1
    assert fwd(_desc(reserved=1)) == 1
    assert fwd(_desc(head_dim=96)) == 2
    assert fwd(_desc(dtype=7)) == 2
    assert fwd(_desc(kv_stride_s=1 << 23, kv_stride_h=1 << 40, kv_stride_b=1 << 41)) == 2   # row stride beyond the kernels' reach
    assert fwd(_desc(q_stride_s=1 << 23, q_stride_h=1 << 40, q_stride_b=1 << 41)) == 2
    # more (batch, head) pairs than the kernels' 32-bit counters hold; 65535 x 40000 would wrap a 32-bit product
    assert fwd(_desc(batch=65535, n_q_heads=40000, n_kv_heads=40000)) == 2
    assert fwd(_desc(), seg_off=-1) == 3
    assert fwd(_desc(), seg_len=0) == 3
    assert fwd(_desc(), seg_off=300, seg_len=256) == 3            # past kv_capacity
    assert lib.s1f_seg_attn_fwd(None, p, p, p, 0, 1, p, p, None) == 1

    def fwd_ws(desc, ws, ws_bytes):
        return lib.s1f_seg_attn_fwd_ws(ctypes.byref(desc), p, p, p, 0, 256, p, p, ws, ws_bytes, None)

    assert fwd_ws(_desc(), None, 16) == 1                          # a size without a pointer
    assert fwd_ws(_desc(), ctypes.c_void_p(4100), 1 << 20) == 1    # misaligned workspace
    assert fwd_ws(_desc(head_dim=96), p, 1 << 20) == 2
    assert lib.s1f_fwd_workspace_bytes(ctypes.byref(_desc()), 0, 256) == 0       # no device here: launches are not split
    assert lib.s1f_fwd_workspace_bytes(ctypes.byref(_desc()), 500, 256) == 0     # out of range
    assert lib.s1f_fwd_workspace_bytes(None, 0, 256) == 0

    def bwd(desc, seg_off=0, seg_len=256, ws=p, ws_bytes=1 << 20):
        return lib.s1f_seg_attn_bwd(ctypes.byref(desc), p, p, p, p, p, p, seg_off, seg_len, p, p, p, ws, ws_bytes, None)

    assert bwd(_desc(), ws=None) == 1
    assert bwd(_desc(), ws_bytes=4 * 256 * 4 - 1) == 1
    assert bwd(_desc(), seg_off=400, seg_len=200) == 3
    assert bwd(_desc(head_dim=32)) == 2
    # batch * heads * seg_len beyond the workspace's 32-bit offsets: 4096 * 4096 * 17 rows of statistics (the
    # product of the first two wraps to 2^24 in 32 bits and must not slip through as a small number)
    big = _desc(batch=4096, n_q_heads=4096, n_kv_heads=4096)
    assert bwd(big, seg_len=17, ws_bytes=1 << 62) == 2
    assert lib.s1f_bwd_workspace_bytes(ctypes.byref(_desc()), 0, 256) == 2 * 4 * 256 * 4
    assert lib.s1f_bwd_workspace_bytes(ctypes.byref(_desc()), 500, 256) == 0
    for code in range(0, 6):
        assert isinstance(s1f.strerror(code), str) and s1f.strerror(code)


def test_launch_plan_validates_and_is_whole_without_a_device():
    lib = s1f.load_library()
    plan = (ctypes.c_int64 * 5)()
    ask = lambda desc, launch, off, m, out=plan: lib.s1f_launch_plan(ctypes.byref(desc), launch, off, m, out)
    for launch in (s1f.PLAN_FWD, s1f.PLAN_FWD_WS, s1f.PLAN_DQ, s1f.PLAN_DKDV):
        assert ask(_desc(), launch, 100, 200) == 0
        assert plan[0] in (64, 128, 192) and plan[2] == 0 and plan[3] == 1 and plan[4] == 0
        units = 2 * -(-300 // 128) if launch == s1f.PLAN_DKDV else 4 * -(-200 // plan[0])
        assert plan[1] == units
    assert ask(_desc(), -1, 0, 64) == 1 and ask(_desc(), 4, 0, 64) == 1 and ask(_desc(), 0, 0, 64, None) == 1
    assert ask(_desc(head_dim=96), 0, 0, 64) == 2 and ask(_desc(), 0, 500, 64) == 3
    assert lib.s1f_launch_plan(None, 0, 0, 64, plan) == 1
    paths = (ctypes.c_int64 * 5)()
    assert lib.s1f_launch_paths(ctypes.byref(_desc()), 100, 200, paths) == 0 and paths[1] in (64, 128, 192) and paths[4] == 0
    assert lib.s1f_launch_paths(ctypes.byref(_desc()), 100, 200, None) == 1 and lib.s1f_launch_paths(None, 0, 64, paths) == 1
    assert lib.s1f_launch_paths(ctypes.byref(_desc(head_dim=96)), 0, 64, paths) == 2
    assert lib.s1f_launch_paths(ctypes.byref(_desc()), 500, 64, paths) == 3


def test_noalloc_backward_rejects_more_rows_than_the_array_holds():
    lib = s1f.load_library()
    rows = s1f.static_scratch_rows()
    assert rows == 1 << 21
    p = ctypes.c_void_p(4096)       # never dereferenced: the size check comes before any launch
    hq = 64
    m = rows // hq + 1
    desc = binding.Desc(batch=1, n_q_heads=hq, n_kv_heads=8, head_dim=128, dtype=1, reserved=0, q_stride_b=hq * m * 128,
                        q_stride_h=m * 128, q_stride_s=128, kv_stride_b=8 * m * 128, kv_stride_h=m * 128,
                        kv_stride_s=128, kv_capacity=m)
    rc = lib.s1f_seg_attn_bwd_noalloc(ctypes.byref(desc), p, p, p, p, p, p, 0, m, p, p, p, None)
    assert rc == 5 and "scratch" in s1f.strerror(rc)


def test_seq1f1b_order_matches_oracle():
    """The library enumerates the order in closed form; the oracle simulates the queue of Section 3.2."""
    from oracle import schedule as SCH
    for P_ in (1, 2, 3, 4, 8):
        for i in range(1, P_ + 1):
            for M in (1, 2, 3, 4, 7, 9, 16, 33):
                for k in (1, 2, 3, 4, 8):
                    assert s1f.seq1f1b_warmup(P_, i, M, k) == SCH.warmup_count(P_, i, M, k), (P_, i, M, k)
                    assert s1f.seq1f1b_order(P_, i, M, k) == SCH.stage_order(P_, i, M, k), (P_, i, M, k)


def test_peak_memory_share_matches_oracle():
    """Section 3.1's A * w_i / sum_j w_j: the library's closed-form denominator against the oracle's explicit sum,
    as exact fractions and as the very same float."""
    from fractions import Fraction
    from oracle import schedule as SCH
    for P_ in (1, 2, 3, 4, 8, 16):
        for M in (1, 2, 4, 8, 9, 16, 17, 64):
            for k in (1, 2, 3, 4, 8, 32):
                total = Fraction(0)
                ws = [SCH.warmup_count(P_, j, M, k) for j in range(1, P_ + 1)]
                if sum(ws) == 0:            # one device, whole sequences: the formula divides by zero
                    with pytest.raises(s1f.S1FError):
                        s1f.seq1f1b_peak_memory_share(P_, 1, M, k)
                    continue
                for i in range(1, P_ + 1):
                    num, den = s1f.seq1f1b_peak_memory_share(P_, i, M, k)
                    assert (num, den) == (ws[i - 1], sum(ws)), (P_, i, M, k)
                    assert num / den == SCH.peak_memory_fraction(P_, i, M, k)
                    total += Fraction(num, den)
                assert total == 1
    # the paper's own example shape: 8 devices, 4 segments: the first device holds the most, shares fall by 1 / den
    shares = [s1f.seq1f1b_peak_memory_share(8, i, 32, 4) for i in range(1, 9)]
    assert [n for n, _ in shares] == [10, 9, 8, 7, 6, 5, 4, 3] and {d for _, d in shares} == {52}
    with pytest.raises(s1f.S1FError):
        s1f.seq1f1b_peak_memory_share(4, 5, 8, 2)
    lib = s1f.load_library()
    assert lib.s1f_seq1f1b_peak_memory_share(4, 1, 8, 2, None, None) == 1


def test_seq1f1b_rejects_bad_arguments():
    for bad in ((0, 1, 4, 2), (4, 0, 4, 2), (4, 5, 4, 2), (4, 1, 0, 2), (4, 1, 4, 0)):
        with pytest.raises(s1f.S1FError) as e:
            s1f.seq1f1b_order(*bad)
        assert e.value.status == 1
        with pytest.raises(s1f.S1FError):
            s1f.seq1f1b_warmup(*bad)
    lib = s1f.load_library()
    n = ctypes.c_int64(0)
    buf = (binding.Pass * 4)()
    assert lib.s1f_seq1f1b_order(2, 1, 3, 2, buf, 4, ctypes.byref(n)) == 1      # too small: size reported
    assert n.value == 12
    assert lib.s1f_seq1f1b_order(2, 1, 3, 2, None, 0, ctypes.byref(n)) == 1 and n.value == 12

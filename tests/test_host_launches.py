"""What the library asks of the runtime, recorded by one that runs nothing (recording_runtime.c): in a process of its own, without torch."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAX_DYNAMIC_LDS = 8   # hipFuncAttributeMaxDynamicSharedMemorySize

DRIVER = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import paper_2406_03488_amd as s1f
from paper_2406_03488_amd.binding import Desc
lib = s1f.load_library()
p = 4096   # (no address is looked at)
for dtype in (0, 1):
    for d in (64, 80, 128):
        for hq, hk, off, m in eval(sys.argv[2]):
            desc = ctypes.byref(Desc(1, hq, hk, d, dtype, 0, hq * m * d, m * d, d, hk * (off + m) * d, (off + m) * d, d, off + m))
            big = 1 << 40
            rc = [lib.s1f_seg_attn_fwd(desc, p, p, p, off, m, p, p, None), lib.s1f_seg_attn_fwd_ws(desc, p, p, p, off, m, p, p, p, big, None),
                  lib.s1f_seg_attn_bwd(desc, p, p, p, p, p, p, off, m, p, p, p, p, big, None),
                  lib.s1f_seg_attn_bwd_noalloc(desc, p, p, p, p, p, p, off, m, p, p, p, None),
                  lib.s1f_seg_attn_bwd_dq(desc, p, p, p, p, p, p, off, m, p, p, big, None),
                  lib.s1f_seg_attn_bwd_dkdv(desc, p, p, p, p, p, off, m, p, p, p, big, None)]
            assert rc == [0] * 6, rc
            paths, plan = (ctypes.c_int64 * 5)(), (ctypes.c_int64 * 5)()
            assert lib.s1f_launch_paths(desc, off, m, paths) == 0 and lib.s1f_launch_plan(desc, 0, off, m, plan) == 0
            print(*paths, plan[4], hq)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("runtime") / "recording.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", "-Werror", "-o", so, os.path.join(ROOT, "tests", "recording_runtime.c")], check=True)
    return so


def record(runtime, tmp_path, shapes):
    path = str(tmp_path / "record")
    env = dict(os.environ, RECORD=path, PYTHONPATH=ROOT)
    run = subprocess.run([sys.executable, "-c", DRIVER, runtime, repr(shapes)], env=env, capture_output=True, text=True, cwd=ROOT)
    assert run.returncode == 0, run.stderr
    lines = [line.split() for line in open(path)]
    return lines, [[int(x) for x in line.split()] for line in run.stdout.splitlines()]


def test_every_kernel_is_told_of_its_lds_before_it_runs(runtime, tmp_path):
    lines, _ = record(runtime, tmp_path, [(2, 1, 0, 40), (32, 32, 700, 321), (64, 8, 5000, 3214), (56, 56, 9203, 5220), (112, 112, 0, 193)])
    told, launched = {}, set()
    for what, name, *rest in lines:
        if what == "attribute":
            assert int(rest[0]) == MAX_DYNAMIC_LDS
            told[name] = int(rest[1])
        else:
            lds = int(rest[2])
            launched.add((name, lds))
            assert lds <= 64 * 1024 or told.get(name, 0) >= lds, name
    assert sum(lds > 64 * 1024 for _, lds in launched) >= 25   # (one flag per type of kernel told two of them)


def test_paths_are_the_ones_that_calls_take(runtime, tmp_path):
    shapes = [(2, 1, 0, 40), (32, 32, 700, 321), (56, 56, 17918, 4897), (64, 8, 5000, 3214), (56, 56, 39549, 3678), (130, 130, 8808, 1600)]
    lines, paths = record(runtime, tmp_path, shapes)
    launches = [(name, int(rest[0])) for what, name, *rest in lines if what == "launch"]

    def take(kernel):
        """The next launch, if it is one of that kernel: its workgroups."""
        return launches.pop(0)[1] if launches and kernel in launches[0][0] else 0

    seen = set()
    for one_bwd, _, _, one_noalloc, tiles, second, heads in paths:
        assert take("seg_attn_fwd_kernel")
        assert second == 0 or take("seg_attn_fwd_kernel") >= tiles * heads
        assert take("seg_attn_fwd_kernel")
        take("fwd_merge")
        for one in (one_bwd, one_noalloc):
            if one:
                assert take("bwd_stats") and take("seg_attn_bwd_kernel")
            else:
                assert take("bwd_dq_kernel")
                take("bwd_merge")
                assert take("bwd_dkdv_kernel")
            take("bwd_merge")
        for half in ("dq", "dkdv"):
            assert take(f"bwd_{half}_kernel")
            take("bwd_merge")
        seen |= {("one launch", one_bwd), ("second launch", second > 0), ("partly filled units", tiles > 0)}
    assert not launches and len(seen) == 6


# fp32 calls whose dQ half by itself runs each unit of 128 rows as two tiles of 64: (batch, heads, K/V heads, offset, rows); a last unit whose second
# tile has no rows, one row, all but one; more chunks than some units have tiles; 16 chunks of few units; more tiles than compute units
PAIRS = [(1, 1, 1, 0, 246), (1, 3, 3, 33, 700), (2, 2, 1, 7, 449), (1, 2, 1, 3539, 255), (1, 1, 1, 0, 640), (2, 4, 4, 771, 233), (1, 8, 8, 45, 338)]


def test_dq_half_of_few_units_runs_in_pairs_of_tiles(runtime, tmp_path):
    lines, _ = record(runtime, tmp_path, [(hq, hk, off, m) for nb, hq, hk, off, m in PAIRS if nb == 1])
    names = [name for what, name, *_ in lines if what == "launch"]
    in_pairs = [name for name in names if "bwd_dq_kernelIf" in name and "Lb1E" in name]
    assert len(in_pairs) == 2 * sum(nb == 1 for nb, *_ in PAIRS)   # (head_dim 80 and 128)


PLANS = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import paper_2406_03488_amd as s1f
from paper_2406_03488_amd.binding import Desc
lib = s1f.load_library()
for dtype, nb, hq, hk, d, off, m in eval(sys.argv[2]):
    desc = ctypes.byref(Desc(nb, hq, hk, d, dtype, 0, hq * m * d, m * d, d, hk * (off + m) * d, (off + m) * d, d, off + m))
    for launch in (s1f.PLAN_DQ, s1f.PLAN_DKDV):
        plan = (ctypes.c_int64 * 5)()
        assert lib.s1f_launch_plan(desc, launch, off, m, plan) == 0
        print(*plan)
    paths = (ctypes.c_int64 * 5)()
    assert lib.s1f_launch_paths(desc, off, m, paths) == 0
    print(*paths)
"""
# ((element type, batch, heads, K/V heads, head_dim, offset, rows), fewest chunks of dQ units, of dK/dV units, most of those): calls whose halves
# by themselves took 1.1 to 1.4 times as long in fewer chunks, or with dK/dV units in two chunks instead of whole
HALVES = [((1, 1, 4, 4, 128, 2318, 427), 5, 1, 1), ((1, 1, 8, 8, 80, 17519, 1044), 9, 1, 1), ((1, 1, 1, 1, 128, 13211, 621), 14, 1, 1),
          ((1, 3, 8, 2, 80, 669, 349), 1, 4, 5), ((1, 2, 4, 4, 128, 723, 289), 3, 1, 1), ((1, 2, 3, 3, 64, 1122, 277), 3, 1, 1),
          ((0, 3, 3, 3, 128, 359, 217), 1, 4, 4)]


def plans_of(runtime, tmp_path, calls):
    """Plan of the dQ half, of the dK/dV half, and paths of each call."""
    env = dict(os.environ, RECORD=str(tmp_path / "record"), PYTHONPATH=ROOT)
    run = subprocess.run([sys.executable, "-c", PLANS, runtime, repr(calls)], env=env, capture_output=True, text=True, cwd=ROOT)
    assert run.returncode == 0, run.stderr
    lines = [[int(x) for x in line.split()] for line in run.stdout.splitlines()]
    return [lines[i:i + 3] for i in range(0, len(lines), 3)]


def test_cuts_of_one_launch_serve_the_halves_too(runtime, tmp_path):
    for (call, least_dq, least, most), (dq, dkdv, _) in zip(HALVES, plans_of(runtime, tmp_path, [c for c, *_ in HALVES])):
        assert dq[3] >= least_dq, call
        assert least <= dkdv[3] <= most, call


def test_a_few_workgroups_too_many_for_one_round_run_apart(runtime, tmp_path):
    """fp32, head_dim 128, one workgroup to a compute unit: 128 workgroups of the dQ half and 146 or 130 of the other."""
    over, short = plans_of(runtime, tmp_path, [(0, 1, 2, 1, 128, 18102, 470), (0, 1, 1, 1, 128, 15703, 914)])
    assert all(dq[2] * dq[3] == 128 for dq, _, _ in (over, short))
    assert over[1][1] == 146 and short[1][1] == 130   # (two of 130 follow seven short ones on the diagonal)
    assert over[2][0] == 0 and short[2][0] == 1

"""Forward of calls with few rows, whose waves share the keys of a unit of 16 or 32 rows (that they do is asked of the library): edges
of units and tiles, waves without keys, every head_dim and element type, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2406_03488_amd as s1f
from oracle import attention as A
from test_gpu_launch_cuts import _close, _device_data

pytestmark = pytest.mark.gpu

# (batch, query heads, K/V heads, offset, rows), rows per unit: one row; one row more and less than a block and than a unit;
# units with fewer tiles than waves; one unit of 16 rows per compute unit, and more (bf16 at head_dim 64 has two of them before it takes
# units of 32, unless walks are long); a last unit of one row; offsets that put a diagonal on two tiles
SHAPES = [((1, 1, 1, 400, 1), 16), ((2, 3, 1, 700, 15), 16), ((1, 4, 4, 360, 17), 16), ((1, 2, 1, 353, 33), 16), ((3, 2, 2, 218, 161), 16),
          ((1, 8, 2, 1500, 512), 16), ((1, 8, 2, 1499, 625), 32), ((2, 15, 5, 777, 225), 32), ((1, 8, 2, 3500, 577), 32)]


@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("shape,rows", SHAPES)
def test_units_whose_waves_share_the_keys(dtype, d, shape, rows, rising):
    nb, hq, hkv, off, m = shape
    q, _, k, v = _device_data(300 + off + m + d, dtype, d, *shape, rising)
    if (off + m) % 2:   # other strides: heads between the rows
        q, k, v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, k, v))
    if dtype == "bf16" and d == 64 and off < 3000:
        rows = 16
    plan = s1f.launch_plan(q, k, off, s1f.PLAN_FWD)
    assert plan == (rows, nb * hq * -(-m // rows), 0, 1, 0), "the shape no longer takes the path it is here for"
    host = lambda x: x.double().cpu().numpy()
    calls = [lambda o, l: s1f.seg_attn_fwd(q, k, v, off, o, l)]
    if dtype == "bf16" and off < 3000:   # (fp32, and few rows behind many keys, with a workspace: row tiles)
        assert s1f.launch_plan(q, k, off, s1f.PLAN_FWD_WS) == plan and s1f.fwd_workspace_bytes(q, k, off) == 0
        calls.append(lambda o, l: s1f.seg_attn_fwd_ws(q, k, v, off, o, l, None))
    res = []
    for call in calls:
        out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
        call(out, lse)
        res.append((out, lse))
    assert all(torch.equal(x, y) for x, y in zip(res[0], res[-1]))
    out, lse = res[0]
    for b in range(nb):
        want, want_lse = A.segment_forward(host(q[b]), host(k[b]), host(v[b]), off)
        _close({"out": host(out[b]), "lse": host(lse[b])}, {"out": want, "lse": want_lse}, dtype, f"entry {b}: ")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("off,m,rows", [(117, 180, 16), (117, 1041, 32), (105, 1041, 32)])
def test_keys_that_are_not_finite_leave_earlier_rows_alone(dtype, off, m, rows):
    """Units of 16 rows, and of 32 (offset 105) whose first block ends a tile before the second: rows whose block ends before a tile keep
    their bits when that tile's values become NaN and its keys infinite.  (fp32, next to a block that does not: computed again in plain
    arithmetic with it, the same up to the rounding of its sums.)"""
    q, _, k, v = _device_data(m, dtype, 80, 1, 4, 2, off, m, False)
    assert s1f.launch_plan(q, k, off, s1f.PLAN_FWD)[0] == rows
    res = []
    for bad in (False, True):
        first = 32 * ((off + m // 2) // 32)
        if bad:
            v[:, :, first:] = float("nan")
            k[:, :, first:] = float("inf")
        out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device="cuda")
        s1f.seg_attn_fwd(q, k, v, off, out, lse)
        res.append((out, lse))
    alone = (first - off) // 16 * 16   # rows of blocks that end before the tile
    assert alone > 0 and torch.isfinite(res[0][0]).all()
    mixed = alone % rows   # rows of the unit that both kinds of blocks are in
    assert mixed == (16 if off == 105 else 0)
    same = alone - mixed if dtype == "f32" else alone
    for x, y in zip(*res):
        assert torch.equal(x[:, :, :same], y[:, :, :same])
        x, y = x[:, :, same:alone], y[:, :, same:alone]
        assert torch.isfinite(y).all() and (x.numel() == 0 or (x - y).abs().max() <= 2.0 ** -18 * max(1.0, x.abs().max()))
    assert not torch.isfinite(res[1][0][:, :, first - off:]).any()


# Keys that are to have no weight, as a column of K makes them (q has 0.25 to 1.75 in it): the lowest bf16, scores from which a
# rounding is larger than exponents are, and minus infinity
@pytest.mark.parametrize("low", [-3.3895e38, -1e12, float("-inf")])
@pytest.mark.parametrize("run,odd", [(1, 0), (1, 1), (4, 0), (4, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("shape,rows", [((1, 4, 2, 900, 100), 16), ((1, 8, 2, 1499, 625), 32)])
def test_tiles_of_keys_without_weight(shape, rows, d, dtype, run, odd, low):
    """Every other run of tiles of 32 keys has scores far below all others: among the even or the odd ones is the first tile of every
    wave, and in longer runs all that a wave walks."""
    nb, hq, hkv, off, m = shape
    q, _, k, v = _device_data(off + d, dtype, d, *shape, False)
    q[..., d - 1] = q[..., d - 1].abs().clamp(0.25, 1.75)
    k[..., d - 1] = torch.where(torch.arange(off + m, device="cuda") // (32 * run) % 2 == odd, low, 0.0)
    if dtype == "bf16" and d == 64:
        rows = 16
    assert s1f.launch_plan(q, k, off, s1f.PLAN_FWD)[0] == rows
    out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
    s1f.seg_attn_fwd(q, k, v, off, out, lse)
    host = lambda x: x[0].double().cpu().numpy()
    with np.errstate(invalid="ignore"):
        want, want_lse = A.segment_forward(host(q), host(k), host(v), off)
    assert np.isfinite(want).all()
    _close({"out": host(out), "lse": host(lse)}, {"out": want, "lse": want_lse}, dtype, "")


# Few keys: row tiles take less time than waves need to meet.  One row, rows and keys around a block and a tile, and units of 32 rows
FEW_KEYS = [(1, 1, 1, 0, 1), (2, 4, 2, 0, 16), (1, 3, 3, 15, 17), (1, 8, 2, 31, 33), (3, 2, 1, 60, 20), (1, 6, 1, 0, 64), (2, 8, 8, 8, 399)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("shape", FEW_KEYS)
def test_few_keys_run_in_row_tiles(shape, d, dtype):
    nb, hq, hkv, off, m = shape
    q, _, k, v = _device_data(400 + off + m + d, dtype, d, *shape, False)
    if not (m == 399 and dtype == "bf16" and d == 64):   # (two units of 16 rows on a compute unit)
        assert s1f.launch_plan(q, k, off, s1f.PLAN_FWD)[0] == 64
    out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
    s1f.seg_attn_fwd(q, k, v, off, out, lse)
    host = lambda x: x.double().cpu().numpy()
    for b in range(nb):
        want, want_lse = A.segment_forward(host(q[b]), host(k[b]), host(v[b]), off)
        _close({"out": host(out[b]), "lse": host(lse[b])}, {"out": want, "lse": want_lse}, dtype, f"entry {b}: ")

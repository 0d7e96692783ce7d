"""Launches at the edges of what the planner chooses between, in both element types, compared with the oracle: few row
tiles (of 64 rows: the narrowest) that are nearly empty or nearly full, whole and cut along the keys (forward, dQ) or along
the queries (dK/dV) with more chunks than some of their units have tiles; every wider tile of the forward and the dQ
kernel, whole and cut, with waves that are partly or wholly empty, on data that raises the running maximum as well as on
data that does not; rows of a partial last round in a second launch.  Which plan a shape gets is asked of the library, so
that a test whose shape no longer takes the path it is about fails.  The two halves of the backward as separate calls
equal the one call bit for bit."""
import numpy as np
import pytest
import torch

import paper_2406_03488_amd as s1f
import s1f_synth as S
from oracle import attention as A
from test_gpu_batch_sweep import _check, _sequence

pytestmark = pytest.mark.gpu

# (query heads, K/V heads, offset, rows): one row; one row more and less than 64, 128 and 192; a first segment (its early
# units have fewer key tiles than chunks); 64 heads.  Their backwards run in tiles of 64 rows (fp32 above head_dim 64: some in 128), and
# the fp32 forward with a workspace; other forwards of fewer than 32 heads share keys among waves.
SHAPES = [(2, 1, 700, 1), (4, 2, 0, 63), (4, 2, 33, 65), (8, 2, 400, 127), (3, 1, 1000, 129), (2, 2, 5, 191),
          (8, 8, 95, 193), (4, 4, 0, 640), (64, 8, 300, 200)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("hq,hkv,off,m", SHAPES)
def test_edges_of_the_launch_plan(dtype, d, hq, hkv, off, m):
    from gpu_harness import run_segment, to_device
    n = off + m
    q, k, v, do = _sequence(8000 + d + off + m, hq, hkv, n, d, dtype)
    out, lse = A.segment_forward(q[:, off:], k, v, off)
    dq, dk, dv = A.segment_backward(do[:, off:], q[:, off:], k, v, off)
    want = {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    got = run_segment(q[:, off:], k, v, do[:, off:], off, dtype)
    _check(got, want, dtype)
    plain = run_segment(q[:, off:], k, v, do[:, off:], off, dtype, layout="bshd", fwd_workspace=False)
    _check(plain, want, dtype, where="without a forward workspace: ")

    dev = lambda x: to_device(x, dtype)[None].contiguous()
    qd, kd, vd, dod = dev(q[:, off:]), dev(k), dev(v), dev(do[:, off:])
    o, dqd = torch.empty_like(qd), torch.empty_like(qd)
    l = torch.empty((1, hq, m), dtype=torch.float32, device="cuda")
    s1f.seg_attn_fwd(qd, kd, vd, off, o, l)
    ws = torch.empty(s1f.bwd_workspace_bytes(qd, kd, off), dtype=torch.uint8, device="cuda")
    acc, dqs = {}, {}
    for how in ("one call", "two calls", "second half again"):   # (it leaves the statistics in place)
        a, b = (torch.zeros((1, hkv, n, d), dtype=torch.float32, device="cuda") for _ in range(2))
        if how == "one call":
            s1f.seg_attn_bwd(dod, qd, kd, vd, o, l, off, dqd, a, b, ws)
        elif how == "two calls":
            s1f.seg_attn_bwd_dq(dod, qd, kd, vd, o, l, off, dqd, ws)
            s1f.seg_attn_bwd_dkdv(dod, qd, kd, vd, l, off, a, b, ws)
        else:
            s1f.seg_attn_bwd_dkdv(dod, qd, kd, vd, l, off, a, b, ws)
        acc[how], dqs[how] = (a, b), dqd.clone()
    assert torch.equal(dqs["one call"], dqs["two calls"])
    for how in ("two calls", "second half again"):
        assert all(torch.equal(x, y) for x, y in zip(acc["one call"], acc[how])), how


def test_fp32_forward_takes_any_workspace():
    """fp32 calls were never cut before they could be: a caller that brings no workspace, or a small one, is served."""
    q, k, v, _ = (torch.from_numpy(x)[None].cuda() for x in _sequence(77, 4, 2, 900, 64, "f32"))
    qs = q[:, :, 700:].contiguous()
    assert s1f.fwd_workspace_bytes(qs, k, 700) > 16
    outs = []
    for ws in (None, torch.empty(16, dtype=torch.uint8, device="cuda"),
               torch.empty(s1f.fwd_workspace_bytes(qs, k, 700), dtype=torch.uint8, device="cuda")):
        out, lse = torch.empty_like(qs), torch.empty(qs.shape[:3], device="cuda")
        s1f.seg_attn_fwd_ws(qs, k, v, 700, out, lse, ws)
        outs.append(out)
    assert torch.equal(outs[0], outs[1])
    assert (outs[0] - outs[2]).abs().max().item() <= 1e-5


# No workspace and a last round that fills a part of the chip, in which the rest runs in a second launch of 64-row tiles:
# both wide tiles, grouped heads (the rest are the first rows of every head) and ungrouped ones (the last heads, whose last
# tile has rows for one or two of its 64-row tiles only), every head_dim that has the path, both element types and layouts.
SECOND_LAUNCH = [
    ("bf16", 128, 192, (3, 40, 8, 2887, 1597), "bhsd"), ("bf16", 128, 192, (2, 112, 112, 12736, 775), "bshd"),
    ("bf16", 128, 128, (3, 96, 96, 6899, 390), "bhsd"), ("bf16", 128, 128, (2, 40, 8, 20462, 1787), "bshd"),
    ("bf16", 80, 192, (3, 96, 96, 8535, 659), "bshd"), ("bf16", 80, 192, (3, 40, 8, 4914, 1575), "bhsd"),
    ("bf16", 80, 128, (3, 96, 96, 5253, 194), "bhsd"), ("f32", 64, 128, (2, 64, 8, 7244, 3873), "bshd"),
    ("f32", 80, 128, (2, 64, 8, 4146, 3339), "bhsd"), ("f32", 128, 128, (2, 64, 8, 5390, 3597), "bhsd"),
]
# ... and in which it stays in the one launch although that is predicted to be slower: it is not, where the units differ in
# length and run head by head, and at head_dim 64 in bf16.
ONE_LAUNCH = [
    ("bf16", 64, (2, 40, 8, 4760, 1734)), ("bf16", 64, (1, 112, 112, 3563, 1191)),
    ("bf16", 80, (1, 56, 56, 5982, 3539)), ("bf16", 128, (1, 56, 56, 9203, 5220)), ("bf16", 128, (2, 32, 32, 4048, 3145)),
    ("f32", 128, (3, 112, 112, 1357, 969)),
]


def _empty(layout, nb, h, n, d, dtype):
    if layout == "bshd":
        return torch.empty((nb, n, h, d), device="cuda", dtype=dtype).permute(0, 2, 1, 3)
    return torch.empty((nb, h, n, d), device="cuda", dtype=dtype)


@pytest.mark.parametrize("dtype,d,rows,shape,layout", SECOND_LAUNCH)
def test_second_launch_of_a_partial_last_round(dtype, d, rows, shape, layout):
    nb, hq, hkv, off, m = shape
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(off + m)
    q, k, v = (_empty(layout, nb, h, n, d, t).normal_(generator=g) for h, n in ((hq, m), (hkv, off + m), (hkv, off + m)))
    plan = s1f.launch_plan(q, k, off, s1f.PLAN_FWD)
    assert plan[0] == rows and plan[1] > 0 and plan[2] == 0 and plan[4] > 0, plan
    assert plan[1] + plan[4] == nb * hq * -(-m // rows)
    res = []
    for workspace in (False, True):
        out, lse = torch.full_like(q, float("nan")), torch.full((nb, hq, m), float("nan"), device="cuda")
        if workspace:
            nbytes = s1f.fwd_workspace_bytes(q, k, off)
            s1f.seg_attn_fwd_ws(q, k, v, off, out, lse, torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None)
        else:
            s1f.seg_attn_fwd(q, k, v, off, out, lse)
        res.append((out, lse))
    # every row of every head against the call that cuts along the keys instead: one bf16 rounding apart; fp32: sums of up
    # to 2e4 terms in another order
    top = res[1][0].float().abs().max().item()
    assert (res[0][0].float() - res[1][0].float()).abs().max().item() <= (2.0 ** -7 if dtype == "bf16" else 2.0 ** -17) * top
    assert (res[0][1] - res[1][1]).abs().max().item() <= 1e-5
    host = lambda x: x.double().cpu().numpy()
    for b, h in ((0, 0), (nb - 1, hq // 2), (nb - 1, hq - 1)):
        g0 = h // (hq // hkv)
        for r0, r1 in ((0, 8), (m // 2, m // 2 + 8), (m - 8, m)):
            want, want_lse = A.segment_forward(host(q[b, h:h + 1, r0:r1]), host(k[b, g0:g0 + 1]), host(v[b, g0:g0 + 1]), off + r0)
            _close({"out": host(res[0][0][b, h:h + 1, r0:r1]), "lse": host(res[0][1][b, h:h + 1, r0:r1])},
                   {"out": want, "lse": want_lse}, dtype, f"entry {b} head {h} rows {r0}: ")


@pytest.mark.parametrize("dtype,d,shape", ONE_LAUNCH)
def test_one_launch_where_a_second_does_not_pay(dtype, d, shape):
    nb, hq, hkv, off, m = shape
    q, k = (torch.empty((nb, h, n, d), device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
            for h, n in ((hq, m), (hkv, off + m)))
    plan = s1f.launch_plan(q, k, off, s1f.PLAN_FWD)
    assert plan[0] > 64 and plan[2] == 0 and plan[4] == 0, plan


# More row tiles than the chip holds at once and a small rest, no workspace: in the first shape the rest (the first rows
# of every head) runs in a second launch of narrower tiles, the second stays in one launch.
@pytest.mark.parametrize("hq,hkv,off,m,heads", [(64, 8, 5000, 3214, [0, 31, 63]), (112, 112, 9000, 1770, [12, 13, 111])])
def test_rows_of_a_partial_last_round(hq, hkv, off, m, heads):
    g = torch.Generator(device="cuda")
    g.manual_seed(off + m)
    rnd = lambda h, n: torch.empty((1, h, n, 128), device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    q, k, v = rnd(hq, m), rnd(hkv, off + m), rnd(hkv, off + m)
    out, lse = torch.full_like(q, 9.0), torch.full((1, hq, m), 9.0, device="cuda")
    s1f.seg_attn_fwd(q, k, v, off, out, lse)
    host = lambda x: x[0].double().cpu().numpy()
    for h in heads:
        g0 = h // (hq // hkv)
        want, want_lse = A.segment_forward(host(q[:, h:h + 1]), host(k[:, g0:g0 + 1]), host(v[:, g0:g0 + 1]), off)
        none = dict.fromkeys(("dq", "dk", "dv"), np.ones(1))
        _check({"out": host(out[:, h:h + 1]), "lse": host(lse[:, h:h + 1]), **none},
               {"out": want, "lse": want_lse, **none}, "bf16", where="head %d: " % h)


# (dtype, head_dim, (batch, query heads, K/V heads, offset, rows), rows per unit and whether units are cut: forward without
# and with a workspace, dQ).  Between them every width that the kernels are built for, whole and cut, last tiles of 1 to
# 65 rows (tiles of 64, 128, 192 rows: waves of 16, 32, 48) and of one row less than a whole one.
WIDTHS = [
    ("bf16", 64, (3, 112, 112, 0, 193), ("128", "128", "128")),
    ("bf16", 64, (3, 64, 8, 757, 321), ("192", "192", "128")),
    ("bf16", 64, (1, 112, 112, 1500, 769), ("64", "64", "128 cut")),
    ("bf16", 64, (1, 56, 56, 4772, 65), ("64", "128 cut", "128 cut")),
    ("bf16", 64, (3, 32, 32, 2585, 129), ("64", "192 cut", "64 cut")),
    ("bf16", 64, (3, 56, 56, 196, 554), ("128", "128", "192")),
    ("bf16", 64, (1, 32, 32, 4011, 129), ("64", "64 cut", "192 cut")),
    ("bf16", 80, (3, 112, 112, 0, 65), ("128", "128", "128")),
    ("bf16", 80, (3, 64, 8, 0, 129), ("192", "192", "192")),
    ("bf16", 80, (1, 112, 112, 1500, 769), ("128", "192 cut", "192 cut")),
    ("bf16", 80, (1, 32, 32, 1500, 577), ("64", "128 cut", "128 cut")),
    ("bf16", 128, (3, 112, 112, 0, 65), ("128", "128", "128")),
    ("bf16", 128, (3, 64, 8, 0, 129), ("192", "192", "64")),
    ("bf16", 128, (1, 112, 112, 1500, 769), ("128", "192 cut", "64")),
    ("bf16", 128, (1, 32, 32, 1500, 577), ("64", "128 cut", "128 cut")),
    ("f32", 64, (3, 112, 112, 0, 193), ("128", "128", "128")),
    ("f32", 64, (1, 32, 32, 700, 321), ("64", "128 cut", "64 cut")),
    ("f32", 64, (3, 56, 56, 333, 65), ("64", "64", "128 cut")),
    ("f32", 80, (3, 112, 112, 0, 193), ("128", "128", "128")),
    ("f32", 80, (1, 32, 32, 700, 321), ("64", "128 cut", "128 cut")),
    ("f32", 128, (3, 112, 112, 0, 193), ("128", "128", "128")),
    ("f32", 128, (1, 32, 32, 700, 321), ("64", "128 cut", "64 cut")),
    ("f32", 128, (1, 32, 32, 0, 450), ("64", "64", "128 cut")),
]


def _device_data(seed, dtype, d, nb, hq, hkv, off, m, rising):
    """q, dout [nb, hq, m, d] and k, v [nb, hkv, off + m, d] of N(0, 1) numbers.  `rising`: scores that climb along the keys
    by tens of nats for some rows and fall for others (key j carries a_j * u, a_j from 0 to 2 in four steps, u of +-1, and
    row r carries c_r * u, c_r in [-2, 2], on top of 0.6 * N(0, 1)), so that the forward raises its running maximum."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rnd = lambda *shape: torch.empty(shape, device="cuda").normal_(generator=g)
    n = off + m
    q, do, k, v = rnd(nb, hq, m, d), rnd(nb, hq, m, d), rnd(nb, hkv, n, d), rnd(nb, hkv, n, d)
    if rising:
        u = rnd(d).sign()
        k = 0.6 * k + (torch.arange(n, device="cuda") * 4 // n * (2.0 / 3.0))[:, None] * u
        q = 0.6 * q + (1.5 * rnd(nb, hq, m, 1)).clamp(-2.0, 2.0) * u
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    return [x.to(t) for x in (q, do, k, v)]


def _close(got, want, dtype, where):
    """The contract's bounds; where results exceed order one, the absolute ones grow by a rounding of the largest value
    (bf16: 2^-9 of it, and as much again for the probabilities; fp32: the rounding of its sums)."""
    from gpu_harness import errors
    for name in want:
        mx, fro = errors(got[name], want[name])
        top = float(np.abs(want[name]).max())
        assert np.isfinite(got[name]).all(), where + name
        if dtype == "f32":
            assert mx <= 1e-4 + 2.0 ** -18 * top, f"{where}{name}: max abs {mx}"
        elif name == "lse":
            assert mx <= 1e-3, f"{where}lse: max abs {mx}"
        else:
            assert mx <= 2e-2 + 2.0 ** -8 * top and fro <= 1e-2, f"{where}{name}: max abs {mx} (of {top}) rel fro {fro}"


@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("dtype,d,shape,plans", WIDTHS)
def test_every_tile_width_whole_and_cut(dtype, d, shape, plans, rising):
    nb, hq, hkv, off, m = shape
    q, do, k, v = _device_data(9000 + off + m + d, dtype, d, *shape, rising)
    for launch, want in zip((s1f.PLAN_FWD, s1f.PLAN_FWD_WS, s1f.PLAN_DQ), plans):
        rows, whole, cut, chunks, second = s1f.launch_plan(q, k, off, launch)
        assert f"{rows}{' cut' if cut else ''}" == want and second == 0, "the shape no longer takes the path it is here for"
    outs = {}
    for how in ("plain", "workspace"):
        out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
        if how == "plain":
            s1f.seg_attn_fwd(q, k, v, off, out, lse)
        else:
            nbytes = s1f.fwd_workspace_bytes(q, k, off)
            s1f.seg_attn_fwd_ws(q, k, v, off, out, lse, torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None)
        outs[how] = (out, lse)
    dq = torch.full_like(q, float("nan"))
    dk, dv = (torch.zeros(k.shape, device="cuda") for _ in range(2))
    ws = torch.empty(s1f.bwd_workspace_bytes(q, k, off), dtype=torch.uint8, device="cuda")
    s1f.seg_attn_bwd(do, q, k, v, *outs["workspace"], off, dq, dk, dv, ws)
    host = lambda x: x.double().cpu().numpy()
    grp = hq // hkv
    for b, g in sorted({(0, 0), (nb - 1, hkv - 1), (nb // 2, hkv // 2)}):
        hs = slice(g * grp, (g + 1) * grp)
        qh, doh, kh, vh = host(q[b, hs]), host(do[b, hs]), host(k[b, g:g + 1]), host(v[b, g:g + 1])
        out, lse = A.segment_forward(qh, kh, vh, off)
        wdq, wdk, wdv = A.segment_backward(doh, qh, kh, vh, off)
        # The backward reads delta = rowsum(dout * out) from the `out` that the forward saved.  What that row-wise difference
        # makes of dQ and dK is linear in it (dQ: times -scale * P K, dK: -scale * P^T (. * Q)) and part of what is expected:
        # keys with a common direction make P K large, and the rounding of a bf16 `out` alone then is 1e-2 of dQ.
        ddelta = (doh * (host(outs["workspace"][0][b, hs]) - out)).sum(-1, keepdims=True) / np.sqrt(d)
        wdq = wdq - ddelta * A.segment_forward(qh, kh, kh, off)[0]
        wdk = wdk - A.segment_backward(ddelta * qh, qh, kh, vh, off)[2]
        where = f"entry {b} K/V head {g}: "
        for how in outs:
            _close({"out": host(outs[how][0][b, hs]), "lse": host(outs[how][1][b, hs])}, {"out": out, "lse": lse}, dtype,
                   where + how + " ")
        _close({"dq": host(dq[b, hs]), "dk": host(dk[b, g:g + 1]), "dv": host(dv[b, g:g + 1])},
               {"dq": wdq, "dk": wdk, "dv": wdv}, dtype, where)


@pytest.mark.parametrize("dtype,d,shape,plans", WIDTHS)
def test_every_tile_width_in_halves(dtype, d, shape, plans):
    """The kernels of one half each, which most calls above do not run: the same bits as the one call, which is compared with the
    oracle there."""
    nb, hq, hkv, off, m = shape
    q, do, k, v = _device_data(9000 + off + m + d, dtype, d, *shape, False)
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device="cuda")
    s1f.seg_attn_fwd(q, k, v, off, out, lse)
    ws = torch.empty(s1f.bwd_workspace_bytes(q, k, off), dtype=torch.uint8, device="cuda")
    res = []
    for halves in (False, True):
        dq = torch.full_like(q, float("nan"))
        dk, dv = (torch.full(k.shape, 0.5, device="cuda") for _ in range(2))
        ws.fill_(0xff)
        if halves:
            s1f.seg_attn_bwd_dq(do, q, k, v, out, lse, off, dq, ws)
            s1f.seg_attn_bwd_dkdv(do, q, k, v, lse, off, dk, dv, ws)
        else:
            s1f.seg_attn_bwd(do, q, k, v, out, lse, off, dq, dk, dv, ws)
        res.append((dq, dk, dv))
    for name, x, y in zip(("dq", "dk", "dv"), *res):
        assert torch.isfinite(x).all() and torch.equal(x, y), name


@pytest.mark.parametrize("run,odd", [(1, 0), (1, 1), (3, 0)])
@pytest.mark.parametrize("dtype,d,shape,plans", WIDTHS)
def test_every_tile_width_on_tiles_of_keys_without_weight(dtype, d, shape, plans, run, odd):
    """Every other tile of 32 keys, or run of three, has scores far below the others, as a column of K makes them (q has 0.25 to 1.75 in it):
    the first tiles of walks and of chunks, and those that raise the maximum from one such tile to the next.  -1e12: finite, and spaced wider
    than exponents are."""
    nb, hq, hkv, off, m = shape
    q, do, k, v = _device_data(9100 + off + m + d, dtype, d, *shape, False)
    q[..., d - 1] = q[..., d - 1].abs().clamp(0.25, 1.75)
    tiles = torch.arange(off + m, device="cuda") // 32
    low = torch.tensor([-1e12, -3.3895e38, float("-inf")], device="cuda")[tiles // 2 % 3]
    k[..., d - 1] = torch.where(tiles // run % 2 == odd, low, 0.0)
    first = min(max(0, 32 * run - off), m - 1) if odd == 0 else 0   # rows before see no other key
    if off + m <= 32 * run:
        k[..., -1, d - 1] = 0.0   # (the last row does)
    for workspace in (False, True):
        out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
        if workspace:
            nbytes = s1f.fwd_workspace_bytes(q, k, off)
            s1f.seg_attn_fwd_ws(q, k, v, off, out, lse, torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None)
        else:
            s1f.seg_attn_fwd(q, k, v, off, out, lse)
        host = lambda x: x.double().cpu().numpy()
        for b, h in ((0, 0), (nb - 1, hq - 1)):
            g = h // (hq // hkv)
            with np.errstate(invalid="ignore"):
                want, want_lse = A.segment_forward(host(q[b, h:h + 1]), host(k[b, g:g + 1]), host(v[b, g:g + 1]), off)
            assert np.isfinite(want[:, first:]).all()
            _close({"out": host(out[b, h:h + 1, first:]), "lse": host(lse[b, h:h + 1, first:])},
                   {"out": want[:, first:], "lse": want_lse[:, first:]}, dtype, f"entry {b} head {h} workspace {workspace}: ")


# Forwards in tiles of 64 rows, whole without a workspace and cut with one, whole either way, and cut where few rows share keys without a
# workspace: one row, one more and less than 64 and 128, three tiles; first segments, whose early units have fewer tiles than chunks;
# 16 chunks.
EDGES_64 = [
    ((1, 32, 8, 1000, 1), "64", "64 cut"), ((1, 32, 32, 1499, 63), "64", "64 cut"), ((1, 33, 11, 1000, 65), "64", "64 cut"),
    ((2, 16, 4, 2100, 127), "64", "64 cut"), ((1, 32, 8, 1000, 129), "64", "64 cut"), ((1, 32, 32, 2600, 191), "64", "64 cut"),
    ((2, 16, 4, 0, 63), "64", "64"), ((1, 32, 8, 5, 65), "64", "64"), ((1, 33, 11, 0, 193), "64", "64"), ((1, 40, 8, 31, 129), "64", "64"),
    ((1, 3, 3, 0, 3000), "64", "64 cut"), ((1, 1, 1, 0, 1600), "16", "64 cut"), ((1, 2, 1, 3000, 1), "16", "64 cut"),
]


@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("shape,plain,cut", EDGES_64)
def test_edges_of_64_row_forwards(shape, plain, cut, d, rising):
    nb, hq, hkv, off, m = shape
    q, _, k, v = _device_data(9200 + off + m + d, "bf16", d, *shape, rising)
    if (off + m) % 2:   # other strides: heads between the rows
        q, k, v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, k, v))
    for launch, want in ((s1f.PLAN_FWD, plain), (s1f.PLAN_FWD_WS, cut)):
        rows, _, units, chunks, _ = s1f.launch_plan(q, k, off, launch)
        assert f"{rows}{' cut' if units else ''}" == want, "the shape no longer takes the path it is here for"
    assert off > 0 or not cut.endswith("cut") or chunks > 2   # (the first unit has two key tiles)
    host = lambda x: x.double().cpu().numpy()
    for workspace in (False, True):
        out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
        if workspace:
            nbytes = s1f.fwd_workspace_bytes(q, k, off)
            room = torch.full((nbytes + 4096,), 0xff, dtype=torch.uint8, device="cuda")   # (a partial result that is not written: NaN)
            s1f.seg_attn_fwd_ws(q, k, v, off, out, lse, room[:nbytes] if nbytes else None)
            assert (room[nbytes:] == 0xff).all()
        else:
            s1f.seg_attn_fwd(q, k, v, off, out, lse)
        assert torch.isfinite(out.float()).all() and torch.isfinite(lse).all()
        for b, h in sorted({(0, 0), (nb - 1, hq // 2), (nb - 1, hq - 1)}):
            g = h // (hq // hkv)
            want, want_lse = A.segment_forward(host(q[b, h:h + 1]), host(k[b, g:g + 1]), host(v[b, g:g + 1]), off)
            _close({"out": host(out[b, h:h + 1]), "lse": host(lse[b, h:h + 1])}, {"out": want, "lse": want_lse}, "bf16",
                   f"entry {b} head {h} workspace {workspace}: ")

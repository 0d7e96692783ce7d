"""Launches at the edges of what the planner chooses between: row tiles of 64, 128 and 192 rows, last tiles that are
nearly empty or nearly full, launches cut along the keys (forward, dQ) and along the queries (dK/dV) with more chunks
than some of their units have tiles, in both element types.  Compared with the oracle within the contract's tolerances;
the two halves of the backward as separate calls bit for bit with the one call."""
import numpy as np
import pytest
import torch

import paper_2406_03488_amd as s1f
import s1f_synth as S
from oracle import attention as A
from test_gpu_batch_sweep import _check, _sequence

pytestmark = pytest.mark.gpu

# (query heads, K/V heads, offset, rows): one row; one row more and less than a tile of each width; a first segment (its
# early units have fewer key tiles than chunks); enough heads to fill the chip with wide tiles and ragged last ones
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

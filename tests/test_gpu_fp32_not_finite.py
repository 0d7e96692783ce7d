"""fp32 operands that are infinite, NaN or near the largest float: every result element is finite, infinite of the right sign or NaN
exactly where 64-bit arithmetic over the visible keys has it so, and heads without such operands keep their bits."""
import numpy as np
import pytest
import torch

import paper_2406_03488_amd as s1f

pytestmark = pytest.mark.gpu

# (query heads, K/V heads, offset, rows, heads looked at): one tile; several, with waves that end at different ones; launches that are cut
# along the keys (or queries); enough heads for tiles of 128 rows
SHAPES = [(2, 2, 0, 70, (0,)), (4, 2, 31, 130, (0, 2)), (4, 4, 1200, 150, (3,)), (264, 264, 127, 97, (0, 263))]
INF, NAN = float("inf"), float("nan")


def exact(q, k, v, do, off):
    """One query head: q, do [m, d], k, v [off + m, d], each row over the keys that it sees."""
    m, d = q.shape
    out, lse, dq, dk, dv = np.zeros((m, d)), np.zeros(m), np.zeros((m, d)), np.zeros_like(k), np.zeros_like(v)
    with np.errstate(all="ignore"):
        for i in range(m):
            n = off + i + 1
            s = (k[:n] * q[i]).sum(1) / np.sqrt(d)
            top = s.max()
            e = np.exp(s - top)
            lse[i] = top + np.log(e.sum())
            p = e / e.sum()
            out[i] = (p[:, None] * v[:n]).sum(0)
            ds = p * ((v[:n] * do[i]).sum(1) - (do[i] * out[i]).sum())
            dq[i] = (ds[:, None] * k[:n]).sum(0) / np.sqrt(d)
            dk[:n] += ds[:, None] * q[i] / np.sqrt(d)
            dv[:n] += p[:, None] * do[i]
    return out, lse, dq, dk, dv


def call(q, k, v, do, off, how):
    out, dq = torch.full_like(q, 9.0), torch.full_like(q, 9.0)
    lse = torch.full(q.shape[:3], 9.0, device="cuda")
    if how == "plain":
        s1f.seg_attn_fwd(q, k, v, off, out, lse)
    else:
        n = s1f.fwd_workspace_bytes(q, k, off)
        s1f.seg_attn_fwd_ws(q, k, v, off, out, lse, torch.empty(n, dtype=torch.uint8, device="cuda") if n else None)
    dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    ws = torch.empty(s1f.bwd_workspace_bytes(q, k, off), dtype=torch.uint8, device="cuda")
    if how == "plain":
        s1f.seg_attn_bwd_dq(do, q, k, v, out, lse, off, dq, ws)
        s1f.seg_attn_bwd_dkdv(do, q, k, v, lse, off, dk, dv, ws)
    else:
        s1f.seg_attn_bwd(do, q, k, v, out, lse, off, dq, dk, dv, ws)
    return dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv)


def kind(x):
    return np.where(np.isnan(x), 3, np.where(x == INF, 1, np.where(x == -INF, 2, 0)))


@pytest.mark.parametrize("how", ["plain", "workspace"])
@pytest.mark.parametrize("which,value", [("v", INF), ("k", -INF), ("q", INF), ("do", INF), ("do", NAN), ("q", NAN), ("k", NAN), ("v", NAN), ("v", 1e37), ("v", -1e37)])
@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("hq,hkv,off,m,heads", SHAPES)
def test_elements_that_are_not_finite(hq, hkv, off, m, heads, d, which, value, how):
    g = torch.Generator(device="cuda")
    g.manual_seed(off + m + d)
    rnd = lambda h, n: torch.empty((1, h, n, d), device="cuda").normal_(generator=g)
    x = dict(q=rnd(hq, m), do=rnd(hq, m), k=rnd(hkv, off + m), v=rnd(hkv, off + m))
    clean = call(x["q"], x["k"], x["v"], x["do"], off, how)
    group, rows = hq // hkv, x[which].shape[2]
    for h in heads:
        x[which][0, h if which in ("q", "do") else h // group, rows * 2 // 3, 3] = value
    got = call(x["q"], x["k"], x["v"], x["do"], off, how)
    host = {n: t[0].double().cpu().numpy() for n, t in x.items()}
    touched = {h // group for h in heads}
    for g0 in touched:
        hs = range(g0 * group, (g0 + 1) * group)
        res = [exact(host["q"][h], host["k"][g0], host["v"][g0], host["do"][h], off) for h in hs]
        with np.errstate(all="ignore"):
            want = {"dk": sum(r[3] for r in res), "dv": sum(r[4] for r in res)}
        for i, name in enumerate(("out", "lse", "dq")):
            want[name] = np.stack([r[i] for r in res])
        for name, w in want.items():
            y = got[name][0, g0 if name in ("dk", "dv") else slice(hs[0], hs[-1] + 1)].double().cpu().numpy()
            assert (kind(y) == kind(w)).all(), (name, g0, int((kind(y) != kind(w)).sum()))
            fine = kind(w) == 0
            # fp32 sums of up to m * group or off + m terms: a rounding (2^-24) times the square root of their number of the largest
            # term, which may exceed the result by as much again
            assert np.linalg.norm(y[fine] - w[fine]) <= 2.0 ** -16 * max(np.linalg.norm(w[fine]), 1.0), name
    for name in got:
        per = 1 if name in ("dk", "dv") else group
        others = [h for h in range(got[name].shape[1]) if h // per not in touched]
        assert torch.equal(got[name][:, others], clean[name][:, others]), name

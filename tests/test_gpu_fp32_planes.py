"""fp32 operands travel as three bf16 planes: operands of all magnitudes (each head_dim column of V, dO and K has a power of two of its
own, so that a plane lost or shifted shows in the small ones too), walks of one to eight key tiles through the three-stage
ring, waves that end at different tiles, rows and keys past the end; the largest floats; infinities."""
import numpy as np
import pytest
import torch

import paper_2406_03488_amd as s1f
from oracle import attention as A

pytestmark = pytest.mark.gpu

# (query heads, K/V heads, offset, rows): last tiles of one key, walks of 1 to 8 tiles; enough heads for the wide tiles
SHAPES = [(2, 1, 0, 1), (2, 2, 0, 33), (4, 2, 31, 66), (2, 1, 96, 129), (2, 2, 64, 192), (264, 264, 127, 97)]


def _call(q, k, v, do, off):
    out, dq = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    lse = torch.full(q.shape[:3], float("nan"), device="cuda")
    s1f.seg_attn_fwd(q, k, v, off, out, lse)
    dk, dv = (torch.zeros(k.shape, device="cuda") for _ in range(2))
    ws = torch.empty(s1f.bwd_workspace_bytes(q, k, off), dtype=torch.uint8, device="cuda")
    s1f.seg_attn_bwd(do, q, k, v, out, lse, off, dq, dk, dv, ws)
    return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("hq,hkv,off,m", SHAPES)
def test_operands_of_all_magnitudes(d, hq, hkv, off, m):
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * off + m + d)
    rnd = lambda h, n: torch.empty((1, h, n, d), device="cuda").normal_(generator=g)
    q, do, k, v = rnd(hq, m), rnd(hq, m), rnd(hkv, off + m), rnd(hkv, off + m)
    up = torch.exp2(torch.arange(d, device="cuda") % 41 - 20.0)   # 2^-20 .. 2^20 along head_dim
    v, do = v * up, do / up                                       # dP = dO V^T stays of order one
    k, q = k * up, q / up
    got = _call(q, k, v, do, off)
    host = lambda x: x[0].double().cpu().numpy()
    for h in sorted({0, hq // 2, hq - 1}):
        kv = h // (hq // hkv)
        hs = slice(kv * (hq // hkv), (kv + 1) * (hq // hkv))
        qh, doh, kh, vh = host(q)[hs], host(do)[hs], host(k)[kv:kv + 1], host(v)[kv:kv + 1]
        out, lse = A.segment_forward(qh, kh, vh, off)
        dq, dk, dv = A.segment_backward(doh, qh, kh, vh, off)
        want = {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
        # Column by column.  dS = P (dP - delta) carries the rounding of dP and delta, which may cancel (a row that sees one key
        # has dQ = 0): an error of eps (|dP| + |delta|) in dS, times the other operand's column, summed over keys with sum P = 1
        # (dQ) or over at most m rows (dK).  The probabilities are off by the scores' own rounding: |S| < 64, so 2^6 eps.
        # eps: 2^-24 times the square root of the terms of a sum (up to 400), hence 2^-18; with the scores' 2^6 of it, 2^-13.
        dp = np.abs(doh @ vh[0].T).max() + np.abs((doh * out).sum(-1)).max()
        col = lambda x: np.abs(x).reshape(-1, d).max(0)
        size = {"out": col(vh), "lse": 64.0, "dq": dp * col(kh) / np.sqrt(d), "dk": m * len(qh) * dp * col(qh) / np.sqrt(d),
                "dv": m * len(qh) * col(doh)}
        for name, x in want.items():
            y = host(got[name])[hs if name in ("out", "lse", "dq") else slice(kv, kv + 1)]
            err = np.abs(y - x).max() if name == "lse" else col(y - x)
            assert np.isfinite(y).all() and (err <= 2.0 ** (-18 if name == "lse" else -13) * size[name]).all(), (name, h, (err / size[name]).max())


@pytest.mark.parametrize("d", [64, 80, 128])
def test_largest_floats_and_infinities(d):
    big = torch.finfo(torch.float32).max
    q, do, k, v = (torch.randn((1, 2, 70, d), device="cuda", generator=torch.Generator("cuda").manual_seed(d + i)) for i in range(4))
    v[:, 0, :, 5] = big       # a probability-weighted mean of the largest float is the largest float
    v[:, 1, :, 7] = -big
    out, lse = torch.empty_like(q), torch.empty((1, 2, 70), device="cuda")
    s1f.seg_attn_fwd(q, k, v, 0, out, lse)
    ratio = torch.stack([out[0, 0, :, 5] / big, out[0, 1, :, 7] / -big])
    near = torch.isfinite(ratio)   # (a mean that rounds up past the largest float is infinite)
    assert near.sum() > 0 and (ratio[near] - 1).abs().max() <= 2.0 ** -18
    keep = torch.ones(d, dtype=torch.bool, device="cuda")
    keep[[5, 7]] = False
    assert torch.isfinite(out[..., keep]).all()
    v[:, 0, 69] = float("inf")   # seen by the last row only; rows whose block ends before its tile stay as they are
    again = torch.empty_like(out)
    s1f.seg_attn_fwd(q, k, v, 0, again, lse)
    assert torch.equal(again[:, :, :64], out[:, :, :64]) and not torch.isfinite(again[0, 0, 69]).any()


@pytest.mark.parametrize("d", [64, 80, 128])
def test_products_left_out_do_not_add_up(d):
    """Scores of one product each, of operands just below a step of the second plane.  With planes cut off, a1 * b2 + a2 * b1 of
    all of them is 2^-22 of the product and of one sign; rounded to nearest, what is left out is at most 2^-24 (each of the first two
    planes leaves 2^-8, then 2^-9 of itself), of either sign here.  Read from lse = s of rows that see one key."""
    heads = 4096
    up = 1 + 2.0 ** -7 - 2.0 ** -16 + torch.arange(64, device="cuda", dtype=torch.float64) * 2.0 ** -23
    x, y = up.repeat(64), up.repeat_interleave(64)
    q, k = torch.zeros((1, heads, 1, d), device="cuda"), torch.zeros((1, heads, 1, d), device="cuda")
    q[0, :, 0, 5], k[0, :, 0, 5] = x.float(), y.float()
    out, lse = torch.empty_like(q), torch.empty((1, heads, 1), device="cuda")
    s1f.seg_attn_fwd(q, k, torch.ones_like(k), 0, out, lse)
    f = lambda v: float(np.float32(v))
    unit = f(f(f(1 / d ** 0.5) * f(1.4426950408889634)) * 1.0) * f(0.6931471805599453)   # lse of a score of one, in the kernel's constants
    err = lse[0, :, 0].double() / (x * y * unit) - 1
    assert abs(err.mean().item()) <= 2.0 ** -24 and err.abs().max().item() <= 2.0 ** -21   # (single ones: three roundings as well)


@pytest.mark.parametrize("d", [64, 80, 128])
def test_every_bit_of_an_operand_counts(d):
    """A row that sees one key: out = v and dv = dout, all 24 bits of them (the last plane alone is 2^-17 of a value and less)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    q, k = (torch.zeros((3, 50, 1, d), device="cuda") for _ in range(2))
    v, do = (torch.empty_like(q).normal_(generator=g) for _ in range(2))
    got = _call(q, k, v, do, 0)
    assert torch.equal(got["out"], v) and torch.equal(got["dv"], do) and not got["lse"].any()


@pytest.mark.parametrize("d", [64, 80, 128])
def test_every_product_of_planes_counts(d):
    """Heads of one row that sees two keys, with so few elements that are not zero that every result is one product, of scores, dP or
    dS among its factors: p1 = P(key 1), dS = p1 p2 (dO . v1), dQ = dS k1, dK = dS q, dV = p dO.  Relative errors are a few times 2^-24,
    with one of the six products or the last plane of one operand missing 2e-6 and more (tests/test_host_fp32_planes.py)."""
    heads = 2048
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    q, do = (torch.zeros((1, heads, 1, d), device="cuda") for _ in range(2))
    k, v = (torch.zeros((1, heads, 2, d), device="cuda") for _ in range(2))
    rnd = lambda: torch.empty((1, heads), device="cuda").normal_(generator=g)
    do[:, :, 0, 3], v[:, :, 0, 3], k[:, :, 0, 7], k[:, :, 0, d - 1], q[:, :, 0, d - 1] = (rnd() for _ in range(5))
    got = _call(q, k, v, do, 1)
    host = lambda x: x[0].double().cpu().numpy()
    out, lse = A.segment_forward(host(q), host(k), host(v), 1)
    dq, dk, dv = A.segment_backward(host(do), host(q), host(k), host(v), 1)
    for name, x in {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}.items():
        assert np.linalg.norm(host(got[name]) - x) <= 1e-6 * np.linalg.norm(x), (name, np.linalg.norm(host(got[name]) - x) / np.linalg.norm(x))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("power", [-125, -115, 60, 100])
@pytest.mark.parametrize("small", ["v", "do", "q", "k"])
def test_operands_at_the_ends_of_the_range(d, power, small):
    """One operand 2^power times as large (of large queries or keys the other as much smaller): the same relative errors of what is
    linear in it.  At 2^-125 one value in three is a subnormal number, with the bits that it has."""
    g = torch.Generator(device="cuda")
    g.manual_seed(d + power)
    x = {n: torch.empty((1, 2, 150, d), device="cuda").normal_(generator=g) for n in ("q", "k", "v", "do")}
    x[small] = x[small] * 2.0 ** power
    if small in ("q", "k") and power > 0:
        other = "k" if small == "q" else "q"
        x[other] = x[other] * 2.0 ** -power
    got = _call(x["q"], x["k"], x["v"], x["do"], 0)
    names = {"v": ("out",), "do": ("dv",), "q": ("dk", "out", "lse"), "k": ("dq", "out", "lse")}[small]
    _relative_errors_of(names, got, x)


def _relative_errors_of(names, got, x):
    host = lambda t: t[0].double().cpu().numpy()
    out, lse = A.segment_forward(host(x["q"]), host(x["k"]), host(x["v"]), 0)
    dq, dk, dv = A.segment_backward(host(x["do"]), host(x["q"]), host(x["k"]), host(x["v"]), 0)
    want = {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    for name in names:
        y = host(got[name])
        top = np.abs(want[name]).max()
        assert np.linalg.norm(y / top - want[name] / top) <= 2e-6 * np.linalg.norm(want[name] / top), name   # (a last plane lost: 1e-3, 1e-6 at 2^-115)

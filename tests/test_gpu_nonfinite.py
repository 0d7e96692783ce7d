"""A key or value that is not finite must not reach rows that come before it, further than the tile it lies in: a hidden
key has probability zero, but zero times infinity is NaN, so a kernel must not multiply tiles that a row does not see.
Rows whose own 32 rows end before the key's 32-key tile begins keep the result they have with finite data, whatever tile
width a launch takes."""
import pytest
import torch

import paper_2406_03488_amd as s1f

pytestmark = pytest.mark.gpu

# (batch, query heads, K/V heads, offset, rows): a few workgroups of the narrowest tiles; enough (batch, head) pairs that
# the wide ones are chosen, in one and in several rounds; a prefix long enough that the launches are cut along the keys
SHAPES = [(1, 4, 2, 45, 200), (3, 112, 112, 0, 193), (3, 64, 8, 0, 385), (1, 112, 112, 333, 770), (1, 2, 1, 2100, 333)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("nb,hq,hkv,off,m", SHAPES)
def test_later_keys_that_are_not_finite_do_not_reach_earlier_rows(dtype, d, nb, hq, hkv, off, m):
    g = torch.Generator(device="cuda")
    g.manual_seed(off + m + d)
    rnd = lambda h, n: torch.empty((nb, h, n, d), device="cuda", dtype=dtype).normal_(generator=g)
    q, do, k, v = rnd(hq, m), rnd(hq, m), rnd(hkv, off + m), rnd(hkv, off + m)

    def results(k, v, workspace):
        out, dq = torch.zeros_like(q), torch.zeros_like(q)
        lse = torch.zeros(q.shape[:3], device="cuda")
        if workspace:
            nbytes = s1f.fwd_workspace_bytes(q, k, off)
            s1f.seg_attn_fwd_ws(q, k, v, off, out, lse, torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None)
        else:
            s1f.seg_attn_fwd(q, k, v, off, out, lse)
        dk, dv = (torch.zeros(k.shape, device="cuda") for _ in range(2))
        ws = torch.empty(s1f.bwd_workspace_bytes(q, k, off), dtype=torch.uint8, device="cuda")
        s1f.seg_attn_bwd(do, q, k, v, out, lse, off, dq, dk, dv, ws)
        return {"out": out, "lse": lse, "dq": dq}

    rows = torch.arange(m, device="cuda")
    for workspace in (True, False):
        clean = results(k, v, workspace)
        for bad, poisoned, value in ((off + m - 1, "v", float("inf")), (off + m // 2, "k", float("nan")),
                                     (off + m // 2 + 40, "v", float("nan"))):
            kk, vv = k.clone(), v.clone()
            (kk if poisoned == "k" else vv)[:, :, bad] = value
            before = (off + rows // 32 * 32 + 31) // 32 < bad // 32
            assert before.sum() > 30
            got = results(kk, vv, workspace)
            for name in clean:
                x, y = got[name][:, :, before].float(), clean[name][:, :, before].float()
                assert torch.isfinite(x).all(), f"{name}: {poisoned} row {bad} reaches earlier rows"
                # rows next to it may be rescaled at another tile: one rounding of the probabilities and of the result
                bound = (2.0 ** -6 if dtype == torch.bfloat16 else 2.0 ** -18) * max(1.0, y.abs().max().item())
                assert (x - y).abs().max().item() <= bound, name

"""Forward without a workspace whose second launch takes the last, partly filled unit of every head: that it does is asked of the
library; every row against the call that leaves the units whole or cuts them along the keys, and rows of each kind of tile against the
oracle."""
import numpy as np
import pytest
import torch

import paper_2406_03488_amd as s1f
from oracle import attention as A

pytestmark = pytest.mark.gpu


# (batch, heads, offset, rows), 64-row tiles of each last unit in the second launch: 192-row units, as many of them left over as there
# are heads and more; last units of 1, 30, 45, 64, 65, 72, 120 and 128 rows
@pytest.mark.parametrize("d,shape,tiles,layout", [
    (128, (1, 56, 39549, 3678), 1, "bhsd"), (128, (1, 128, 21141, 1537), 1, "bshd"), (128, (1, 128, 27876, 1608), 2, "bhsd"),
    (128, (2, 48, 20000, 2150), 1, "bhsd"), (80, (2, 64, 9370, 1537), 1, "bhsd"), (80, (1, 130, 8808, 1600), 1, "bshd"),
    (80, (2, 40, 12616, 2541), 1, "bshd"), (80, (2, 64, 9825, 1601), 2, "bhsd"), (80, (2, 64, 9825, 1664), 2, "bshd"),
    (80, (2, 40, 12719, 2616), 2, "bhsd")])
def test_rows_of_every_tile(d, shape, tiles, layout):
    nb, h, off, m = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(off + m + d)

    def rnd(n):
        if layout == "bshd":
            return torch.empty((nb, n, h, d), device="cuda", dtype=torch.bfloat16).normal_(generator=g).permute(0, 2, 1, 3)
        return torch.empty((nb, h, n, d), device="cuda", dtype=torch.bfloat16).normal_(generator=g)

    q, k, v = rnd(m), rnd(off + m), rnd(off + m)
    rows, whole, cut, _, second = s1f.launch_plan(q, k, off, s1f.PLAN_FWD)
    assert rows == 192 and cut == 0 and whole > 0 and second >= nb * h, "the shape no longer takes the path it is here for"
    assert s1f.launch_paths(q, k, off)[4] == tiles == -(-(m % 192) // 64)
    out, lse = torch.full_like(q, float("nan")), torch.full((nb, h, m), float("nan"), device="cuda")
    s1f.seg_attn_fwd(q, k, v, off, out, lse)
    want, want_lse = torch.empty_like(q), torch.empty_like(lse)
    nbytes = s1f.fwd_workspace_bytes(q, k, off)
    s1f.seg_attn_fwd_ws(q, k, v, off, want, want_lse, torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None)
    # the calls differ in the order of fp32 sums and raise running maxima at other keys: one bf16 rounding of the largest result
    top = want.float().abs().max().item()
    assert (out.float() - want.float()).abs().max().item() <= 2.0 ** -7 * top
    assert (lse - want_lse).abs().max().item() <= 1e-5
    # the first whole unit, the last one (left over for the last heads) and the partly filled one
    host = lambda x: x.double().cpu().numpy()
    last = m // 192 * 192
    for b, i in ((0, 0), (nb - 1, h // 2), (nb - 1, h - 1)):
        for r0, r1 in ((0, 4), (last - 4, last), (last, min(last + 4, m)), (m - 1, m)):
            x, y = A.segment_forward(host(q[b, i:i + 1, r0:r1]), host(k[b, i:i + 1]), host(v[b, i:i + 1]), off + r0)
            got = host(out[b, i:i + 1, r0:r1])
            # bf16: a rounding of each probability and of the result
            assert np.abs(got - x).max() <= 2.0 ** -7 * max(np.abs(x).max(), 2.0 ** -3), (b, i, r0)
            assert np.abs(host(lse[b, i:i + 1, r0:r1]) - y).max() <= 1e-5, (b, i, r0)

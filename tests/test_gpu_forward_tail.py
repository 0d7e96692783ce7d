"""Forward without a workspace whose second launch takes the last, partly filled unit of every head."""
import pytest
import torch

import paper_2406_03488_amd as s1f

pytestmark = pytest.mark.gpu


# (batch, heads, offset, rows): 192-row units, more of them left over than there are heads; last units of 1, 30 and 64 rows (one
# 64-row tile each) and of 65 (two), whose tiles and those of the whole units left over then fit one to a compute unit
@pytest.mark.parametrize("d,shape,layout", [(128, (1, 56, 39549, 3678), "bhsd"), (128, (1, 56, 9001, 3649), "bshd"),
                                            (128, (2, 28, 9001, 3712), "bshd"), (80, (1, 56, 9001, 3678), "bhsd"),
                                            (128, (1, 112, 9000, 1770), "bhsd"), (80, (1, 64, 12000, 3329), "bhsd")])
def test_rows_of_every_tile(d, shape, layout):
    nb, h, off, m = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(off + m + d)

    def rnd(n):
        if layout == "bshd":
            return torch.empty((nb, n, h, d), device="cuda", dtype=torch.bfloat16).normal_(generator=g).permute(0, 2, 1, 3)
        return torch.empty((nb, h, n, d), device="cuda", dtype=torch.bfloat16).normal_(generator=g)

    q, k, v = rnd(m), rnd(off + m), rnd(off + m)
    out, lse = torch.full_like(q, float("nan")), torch.full((nb, h, m), float("nan"), device="cuda")
    s1f.seg_attn_fwd(q, k, v, off, out, lse)
    want, want_lse = torch.empty_like(q), torch.empty_like(lse)
    nbytes = s1f.fwd_workspace_bytes(q, k, off)
    s1f.seg_attn_fwd_ws(q, k, v, off, want, want_lse, torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None)
    # the calls differ in the order of fp32 sums and raise running maxima at other keys: one bf16 rounding of the largest result
    top = want.float().abs().max().item()
    assert (out.float() - want.float()).abs().max().item() <= 2.0 ** -7 * top
    assert (lse - want_lse).abs().max().item() <= 1e-5

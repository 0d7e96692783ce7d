"""Calls of so many (batch, head) pairs that one launch would hold 2^32 threads or more, which the runtime accepts and cuts short: one row
per sequence that sees its own key only, so that out = v, lse = q.k / sqrt(d), dq = dk = 0 and dv = dout."""
import math

import pytest
import torch

import paper_2406_03488_amd as s1f

pytestmark = pytest.mark.gpu


# workgroups of the dQ and the dK/dV half together: more than 2^24 of 256 threads, or (fp32 above head_dim 64) than 2^23 of 512;
# of the dK/dV half alone more than 2^23 of 512; of every kernel alone more than 2^24 of 256
@pytest.mark.parametrize("dtype,d,batch", [(torch.bfloat16, 64, 129), (torch.float32, 128, 65), (torch.float32, 80, 129),
                                           (torch.bfloat16, 64, 257)])
def test_all_entries_are_computed(dtype, d, batch):
    heads = 65535
    g = torch.Generator(device="cuda")
    g.manual_seed(batch)
    q, k, v, do = (torch.empty((batch, heads, 1, d), device="cuda", dtype=dtype).normal_(generator=g) for _ in range(4))
    out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
    s1f.seg_attn_fwd(q, k, v, 0, out, lse)
    eps = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -20   # a rounding of p = 1; fp32: the sums of up to 128 terms in lse
    assert ((out - v).abs() <= eps * v.abs()).all()
    for b in (0, batch // 2, batch - 1):
        s = (q[b].double() * k[b].double()).sum(-1) / math.sqrt(d)
        assert (lse[b].double() - s).abs().max().item() <= 1e-4
    dk, dv = (torch.zeros_like(k, dtype=torch.float32) for _ in range(2))
    dq = torch.full_like(q, float("nan"))
    ws = torch.empty(s1f.bwd_workspace_bytes(q, k, 0), dtype=torch.uint8, device="cuda")
    for how in ("one call", "halves"):
        if how == "one call":
            s1f.seg_attn_bwd(do, q, k, v, out, lse, 0, dq, dk, dv, ws)
        else:
            s1f.seg_attn_bwd_dq(do, q, k, v, out, lse, 0, dq, ws)
            s1f.seg_attn_bwd_dkdv(do, q, k, v, lse, 0, dk, dv, ws)
        # p = exp(s - lse) is off by the rounding of |s| < 2^7 (dv), dP - delta by that of its sums of d terms
        assert ((dv - do.float()).abs() <= 2 * max(eps, 2.0 ** -16) * do.float().abs()).all(), how
        assert torch.isfinite(dq).all() and dq.abs().max().item() <= 2.0 ** -10 and dk.abs().max().item() <= 2.0 ** -10, how
        dq.fill_(float("nan"))
        dk.zero_()
        dv.zero_()

"""The backward's two halves in one launch: the same bits as one after the other, nothing written outside its workspace."""
import pytest
import torch

import paper_2406_03488_amd as s1f
from test_host_launches import PAIRS

pytestmark = pytest.mark.gpu

# dtype, head_dim, batch, query heads, K/V heads, offset, rows, storage, rows per unit of the dQ half in the one launch (0: there is none
# for this width) and whether its units come first: each width whole and cut, next to a whole and a cut dK/dV half, either of them
# first; one row, ends of tiles and one past them; several workgroups of statistics
SHAPES = [
    ("bf16", 64, 1, 1, 1, 0, 1, "bhsd", 64, 0), ("bf16", 64, 2, 8, 2, 1000, 357, "bshd", 64, 1), ("bf16", 64, 1, 32, 8, 4600, 1882, "bhsd", 128, 0),
    ("bf16", 64, 3, 32, 32, 2585, 129, "bhsd", 64, 1), ("bf16", 64, 1, 56, 56, 4772, 65, "bshd", 128, 1), ("bf16", 64, 3, 56, 56, 196, 554, "bhsd", 0, 0),
    ("bf16", 80, 3, 3, 3, 31, 65, "bshd", 64, 0), ("bf16", 80, 1, 32, 32, 2406, 513, "bhsd", 192, 1), ("bf16", 80, 1, 32, 32, 4522, 1913, "bhsd", 128, 1),
    ("bf16", 80, 3, 64, 8, 0, 129, "bshd", 192, 0), ("bf16", 80, 1, 32, 32, 1500, 577, "bhsd", 128, 0),
    ("bf16", 128, 1, 2, 1, 63, 64, "bhsd", 64, 0), ("bf16", 128, 1, 64, 8, 2901, 561, "bshd", 64, 0), ("bf16", 128, 1, 32, 32, 0, 1500, "bhsd", 64, 0),
    ("bf16", 128, 1, 112, 112, 1500, 769, "bhsd", 64, 1), ("bf16", 128, 1, 32, 32, 1500, 577, "bshd", 128, 0),
    ("f32", 64, 1, 4, 4, 768, 256, "bhsd", 64, 0), ("f32", 64, 2, 3, 1, 5, 129, "bshd", 64, 0), ("f32", 64, 3, 56, 56, 333, 65, "bhsd", 128, 0),
    ("f32", 80, 1, 4, 4, 300, 193, "bshd", 0, 0), ("f32", 80, 1, 64, 8, 300, 200, "bhsd", 128, 1), ("f32", 80, 1, 32, 32, 700, 321, "bshd", 128, 0),
    ("f32", 128, 1, 8, 2, 1240, 1060, "bhsd", 128, 0), ("f32", 128, 1, 2, 1, 0, 33, "bhsd", 128, 0), ("f32", 128, 1, 32, 32, 700, 321, "bhsd", 0, 0),
    ("f32", 128, 1, 64, 8, 300, 200, "bshd", 128, 1),
]


def _data(seed, dtype, d, nb, hq, hk, off, m, layout):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32

    def rnd(h, n):
        if layout == "bshd":
            return torch.empty((nb, n, h, d), device="cuda").normal_(generator=g).to(t).permute(0, 2, 1, 3)
        return torch.empty((nb, h, n, d), device="cuda").normal_(generator=g).to(t)

    return rnd(hq, m), rnd(hq, m), rnd(hk, off + m), rnd(hk, off + m)


def _apart_bytes(q, k, off, e=4):
    """Of the workspace that the halves share one after the other: statistics, then the partial results of either."""
    rows, _, units, chunks, _ = s1f.launch_plan(q, k, off, s1f.PLAN_DQ)
    _, _, k_units, k_chunks, _ = s1f.launch_plan(q, k, off, s1f.PLAN_DKDV)
    d = q.shape[3]
    stats = -(-2 * e * q.shape[0] * q.shape[1] * q.shape[2] // 256) * 256
    return stats + max(units * chunks * rows * d * e, k_units * (k_chunks - 1) * 2 * 128 * d * e)


@pytest.mark.parametrize("dtype,d,nb,hq,hk,off,m,layout,rows,dq_first", SHAPES)
def test_one_launch_equals_two(dtype, d, nb, hq, hk, off, m, layout, rows, dq_first):
    q, do, k, v = _data(70 + off + m, dtype, d, nb, hq, hk, off, m, layout)
    out, lse = torch.empty_like(q), torch.empty((nb, hq, m), device="cuda")
    s1f.seg_attn_fwd(q, k, v, off, out, lse)
    like_k = torch.empty_like(k, dtype=torch.float32)
    assert like_k.stride() == k.stride()
    need, apart = s1f.bwd_workspace_bytes(q, k, off), _apart_bytes(q, k, off)
    both, dq_rows, first, _, _ = s1f.launch_paths(q, k, off)
    assert (both * dq_rows, first) == (rows, dq_first), "the shape no longer takes the path it is here for"
    # a workspace for one half's partial results only, which "one call, smaller workspace" brings, makes a difference where both are cut
    cut = [s1f.launch_plan(q, k, off, i)[2] > 0 for i in (s1f.PLAN_DQ, s1f.PLAN_DKDV)]
    assert (need > apart) == (both and all(cut))
    got = {}
    for how, size in (("one call", need), ("one call, smaller workspace", apart), ("halves", need), ("no workspace", 0)):
        dq = torch.full_like(q, float("nan"))
        dk, dv = like_k.clone().fill_(0.25), like_k.clone().fill_(-0.5)
        room = torch.full((size + 4096,), 0xff, dtype=torch.uint8, device="cuda")   # (statistics read before they are written: NaN)
        ws = room[:size]
        if how == "halves":
            s1f.seg_attn_bwd_dq(do, q, k, v, out, lse, off, dq, ws)
            s1f.seg_attn_bwd_dkdv(do, q, k, v, lse, off, dk, dv, ws)
        elif how == "no workspace":
            s1f.seg_attn_bwd_noalloc(do, q, k, v, out, lse, off, dq, dk, dv)
        else:
            s1f.seg_attn_bwd(do, q, k, v, out, lse, off, dq, dk, dv, ws)
        torch.cuda.synchronize()
        assert (room[size:] == 0xff).all(), how
        got[how] = dict(dq=dq, dk=dk, dv=dv)
    for how, r in got.items():
        for name, x in r.items():
            assert torch.isfinite(x).all(), (how, name)
            if how == "no workspace" and name == "dq":   # its dQ half may be cut less: sums in another order
                want = got["halves"]["dq"].double()
                bound = 2.0 ** -8 if dtype == "bf16" else 1e-5   # a rounding of the result; fp32 sums
                assert (x.double() - want).norm() <= bound * want.norm()   # (one row that sees one key: zero)
            else:
                assert torch.equal(x, got["halves"][name]), (how, name)


@pytest.mark.parametrize("layout", ["bhsd", "bshd"])
@pytest.mark.parametrize("d", [80, 128])
@pytest.mark.parametrize("nb,hq,hk,off,m", PAIRS)
def test_units_in_pairs_of_tiles_equal_the_one_launch(nb, hq, hk, off, m, d, layout):
    """The dQ half by itself in two 64-row tiles for each unit of 128 rows: the bits of the one launch, whose units are 128 rows."""
    q, do, k, v = _data(90 + off + m, "f32", d, nb, hq, hk, off, m, layout)
    out, lse = torch.empty_like(q), torch.empty((nb, hq, m), device="cuda")
    s1f.seg_attn_fwd(q, k, v, off, out, lse)
    assert s1f.launch_paths(q, k, off)[:2] == (1, 128), "the one call no longer takes the path it is here for"
    like_k, need = torch.empty_like(k, dtype=torch.float32), s1f.bwd_workspace_bytes(q, k, off)
    dqs = []
    for halves in (True, False):
        room = torch.full((need + 4096,), 0xff, dtype=torch.uint8, device="cuda")   # (a chunk that is not written: NaN)
        dq, dk, dv = torch.full_like(q, float("nan")), like_k.clone().zero_(), like_k.clone().zero_()
        if halves:
            s1f.seg_attn_bwd_dq(do, q, k, v, out, lse, off, dq, room[:need])
        else:
            s1f.seg_attn_bwd(do, q, k, v, out, lse, off, dq, dk, dv, room[:need])
        assert (room[need:] == 0xff).all()
        dqs.append(dq)
    assert torch.isfinite(dqs[0]).all() and torch.equal(*dqs)

"""The compiled tensor calls against their Python forms: same results, same refusals."""
import numpy as np
import pytest
import torch

import paper_2406_03488_amd as s1f
from paper_2406_03488_amd import binding

pytestmark = pytest.mark.gpu


class Sub(torch.Tensor):
    pass


def _sequence(dtype, form):
    """A step of two segments through every tensor call; `form` turns an offset into what the call is given."""
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    nb, hq, hk, n, d, cut = 2, 4, 2, 150, 64, 90
    rnd = lambda h: torch.empty((nb, n, h, d), device="cuda").normal_(generator=g).to(dtype).permute(0, 2, 1, 3)
    q, do, k, v = rnd(hq), rnd(hq), rnd(hk), rnd(hk)
    kc, vc = torch.zeros_like(k), torch.zeros_like(v)
    out, dq, dks, dvs = torch.empty_like(q), torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    dk, dv = (torch.zeros_like(k, dtype=torch.float32) for _ in range(2))
    segs, lse = [(0, cut), (cut, n)], []
    for i, (a, b) in enumerate(segs):
        x = slice(a, b)
        s1f.kv_append(k[:, :, x], v[:, :, x], form(a), kc, vc)
        lse.append(torch.empty((nb, hq, b - a), device="cuda"))
        if i == 0:
            s1f.seg_attn_fwd(q[:, :, x], kc, vc, form(a), out[:, :, x], lse[i])
        else:
            size = s1f.fwd_workspace_bytes(q[:, :, x], kc, a)
            ws = torch.empty(size, dtype=torch.uint8, device="cuda") if size else None
            s1f.seg_attn_fwd_ws(q[:, :, x], kc, vc, form(a), out[:, :, x], lse[i], ws)
    for i, (a, b) in reversed(list(enumerate(segs))):
        x = slice(a, b)
        args = (do[:, :, x], q[:, :, x], kc, vc, out[:, :, x], lse[i], form(a), dq[:, :, x], dk, dv)
        if i == 0:
            s1f.seg_attn_bwd_noalloc(*args)
        else:
            s1f.seg_attn_bwd(*args, torch.empty(s1f.bwd_workspace_bytes(q[:, :, x], kc, a), dtype=torch.uint8, device="cuda"))
        s1f.kv_grad_emit(dk, dv, form(a), dks[:, :, x], dvs[:, :, x])
    return [kc, vc, out, *lse, dq, dk, dv, dks, dvs]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_results(dtype):
    native = binding._native()
    t = torch.empty((1, 1, 8, 64), device="cuda", dtype=dtype)
    assert native.append(t, t, np.int64(0), t, t) == -1   # a numpy offset takes the Python form
    for a, b in zip(_sequence(dtype, int), _sequence(dtype, np.int64)):
        assert torch.equal(a, b)


def test_on_the_current_stream():
    want = _sequence(torch.bfloat16, int)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = _sequence(torch.bfloat16, int)
    side.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, got))


def test_same_refusals():
    e = lambda *shape, t=torch.bfloat16, dev="cuda": torch.zeros(shape, dtype=t, device=dev)
    q, k, lse = e(1, 2, 32, 64), e(1, 2, 64, 64), e(1, 2, 32, t=torch.float32)
    with pytest.raises(s1f.S1FError) as err:
        s1f.seg_attn_fwd(q, k, k, 33, q, lse)
    assert "segment out of range" in str(err.value)
    with pytest.raises(s1f.S1FError):
        s1f.seg_attn_fwd(q, k, k, -1, q, lse)
    with pytest.raises(ValueError):
        s1f.seg_attn_fwd(q, k, e(1, 2, 63, 64), 0, q, lse)
    with pytest.raises(ValueError):
        s1f.seg_attn_fwd_ws(q, k, k, 0, q, e(1, 2, 31, t=torch.float32), None)
    with pytest.raises(TypeError):
        s1f.seg_attn_fwd_ws(q, k, k, 0, q, lse.half(), None)
    with pytest.raises(TypeError):
        s1f.seg_attn_fwd(q.half(), k.half(), k.half(), 0, q.half(), lse)
    with pytest.raises(ValueError):
        s1f.seg_attn_fwd(q.transpose(2, 3), k, k, 0, q.transpose(2, 3), lse)
    with pytest.raises(TypeError):
        s1f.seg_attn_bwd(q, q, k, k, q, lse, 0, q, k, k, k)
    with pytest.raises(AttributeError):
        s1f.seg_attn_bwd(q, q, k, k, q, lse, 0, q, k.float(), k.float(), None)
    with pytest.raises(ValueError):
        s1f.kv_append(q, q, 0, k.float(), k.float())
    with pytest.raises(ValueError):
        s1f.kv_grad_emit(k, k, 0, q, q)
    out = q.as_subclass(Sub)   # a subclass goes through its own methods
    s1f.seg_attn_fwd(out, k, k, 0, out, lse)
    torch.cuda.synchronize()


def test_compiled_forms_leave_mismatched_tensors_to_the_python_forms():
    """-1: nothing has been launched (tests/test_host_tensor_calls.py: the Python forms refuse them)."""
    native = binding._native()
    e = lambda *shape, t=torch.bfloat16: torch.zeros(shape, dtype=t, device="cuda")
    q, lse, ws = e(2, 2, 32, 64), e(2, 2, 32, t=torch.float32), e(1 << 16, t=torch.uint8)
    for k in (e(1, 2, 32, 64), e(2, 2, 32, 32), e(2, 2, 32, 64, t=torch.float32)):
        acc = torch.zeros_like(k, dtype=torch.float32)
        assert native.fwd(q, k, k, 0, q, lse) == -1 and native.fwd_ws(q, k, k, 0, q, lse, ws) == -1
        assert native.bwd(q, q, k, k, q, lse, 0, q, acc, acc, ws) == -1
        assert native.bwd_noalloc(q, q, k, k, q, lse, 0, q, acc, acc) == -1
    assert native.fwd(q, q, q, 0, q, lse.bfloat16()) == -1
    cache, acc = e(2, 2, 64, 64), e(2, 2, 64, 64, t=torch.float32)
    for seg in (e(1, 2, 8, 64), e(2, 1, 8, 64), e(2, 2, 8, 32)):
        assert native.append(seg, seg, 0, cache, cache) == -1 and native.emit(acc, acc, 0, seg, seg) == -1
    wide = e(3, 4, 8, 128)   # more than the cache takes: read in part, as ever
    assert native.append(wide, wide, 0, cache, cache) == 0 and native.emit(acc, acc, 0, wide, wide) == 0
    torch.cuda.synchronize()

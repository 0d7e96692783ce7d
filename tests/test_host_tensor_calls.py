"""What the Python forms of the tensor calls refuse before the library is called: tensors that its kernels would read or write past.  The
library is replaced by one that only counts its calls, so that nothing reaches a device."""
import sys
import types

import pytest
import torch

import paper_2406_03488_amd as s1f
from paper_2406_03488_amd import binding

NAMES = ("fwd", "fwd_ws", "bwd", "bwd_noalloc", "append", "emit")


class Library:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        return lambda *args: self.calls.append(name) or 0


@pytest.fixture
def library(monkeypatch):
    lib = Library()
    monkeypatch.setattr(binding, "_native", lambda: types.SimpleNamespace(**{n: lambda *a: -1 for n in NAMES}))
    monkeypatch.setattr(binding, "load_library", lambda: lib)
    monkeypatch.setattr(binding, "_stream_ptr", lambda: 0)
    return lib


def attention_calls(q, k, lse):
    """Every attention call over tensors shaped like q and k."""
    acc = torch.zeros_like(k, dtype=torch.float32)
    ws = torch.empty(64, dtype=torch.uint8)
    return [lambda: s1f.seg_attn_fwd(q, k, k, 0, q, lse), lambda: s1f.seg_attn_fwd_ws(q, k, k, 0, q, lse, ws),
            lambda: s1f.seg_attn_bwd(q, q, k, k, q, lse, 0, q, acc, acc, ws),
            lambda: s1f.seg_attn_bwd_noalloc(q, q, k, k, q, lse, 0, q, acc, acc),
            lambda: binding.seg_attn_bwd_dq(q, q, k, k, q, lse, 0, q, ws),
            lambda: binding.seg_attn_bwd_dkdv(q, q, k, k, lse, 0, acc, acc, ws)]


def bf16(*shape):
    return torch.zeros(shape, dtype=torch.bfloat16)


@pytest.mark.parametrize("k_shape", [(1, 2, 32, 64), (2, 2, 32, 32)])
def test_prefix_smaller_than_the_queries_is_refused(library, k_shape):
    for call in attention_calls(bf16(2, 2, 32, 64), bf16(*k_shape), torch.zeros(2, 2, 32)):
        with pytest.raises(ValueError):
            call()
    assert library.calls == []


@pytest.mark.parametrize("dtypes", [(torch.float32, torch.bfloat16), (torch.bfloat16, torch.float32)])
def test_prefix_of_another_type_is_refused(library, dtypes):
    q, k = (torch.zeros(2, 2, 32, 64, dtype=t) for t in dtypes)
    for call in attention_calls(q, k, torch.zeros(2, 2, 32)):
        with pytest.raises(TypeError):
            call()
    assert library.calls == []


@pytest.mark.parametrize("k_shape", [(2, 2, 32, 64), (3, 1, 64, 64), (2, 2, 32, 128)])
def test_prefix_that_covers_the_queries_is_taken(library, k_shape):
    calls = attention_calls(bf16(2, 2, 32, 64), bf16(*k_shape), torch.zeros(2, 2, 32))
    for call in calls:
        call()
    assert len(library.calls) == len(calls)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float64])
def test_lse_of_another_type_is_refused(library, dtype):
    for call in attention_calls(bf16(2, 2, 32, 64), bf16(2, 2, 32, 64), torch.zeros(2, 2, 32, dtype=dtype)):
        with pytest.raises(TypeError):
            call()
    assert library.calls == []


@pytest.mark.parametrize("seg_shape,taken", [((1, 2, 8, 64), False), ((2, 1, 8, 64), False), ((2, 2, 8, 32), False),
                                             ((2, 2, 8, 64), True), ((3, 4, 8, 128), True)])
def test_segment_smaller_than_the_cache_is_refused(library, seg_shape, taken):
    seg, cache, acc = bf16(*seg_shape), bf16(2, 2, 16, 64), torch.zeros(2, 2, 16, 64)
    for call in (lambda: s1f.kv_append(seg, seg, 0, cache, cache), lambda: s1f.kv_grad_emit(acc, acc, 0, seg, seg)):
        if taken:
            call()
        else:
            with pytest.raises(ValueError):
                call()
    assert len(library.calls) == (2 if taken else 0)


@pytest.mark.parametrize("broken", ["missing", "of another torch"])
def test_without_the_compiled_forms_the_python_forms_serve(monkeypatch, broken):
    """Only libs1f.so is needed: a module of the compiled forms that is missing, or was built against another torch, costs a warning."""
    name = "paper_2406_03488_amd._torch_calls"
    module = None if broken == "missing" else types.SimpleNamespace(torch_version="1.0.0")
    monkeypatch.setitem(sys.modules, name, module)
    if module is None:
        monkeypatch.delattr(s1f, "_torch_calls", raising=False)
    else:
        monkeypatch.setattr(s1f, "_torch_calls", module, raising=False)
    monkeypatch.setattr(binding, "_calls_of", None)
    monkeypatch.setattr(binding, "_calls", None)
    with pytest.warns(RuntimeWarning, match="Python forms"):
        native = binding._native()
    assert all(getattr(native, n)(None) == -1 for n in NAMES)
    lib = Library()
    monkeypatch.setattr(binding, "load_library", lambda: lib)
    monkeypatch.setattr(binding, "_stream_ptr", lambda: 0)
    q, lse = bf16(2, 2, 32, 64), torch.zeros(2, 2, 32)
    s1f.seg_attn_fwd(q, q, q, 0, q, lse)   # (and no second warning)
    assert lib.calls == ["s1f_seg_attn_fwd"]

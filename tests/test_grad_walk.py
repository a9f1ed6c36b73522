"""The native walk over gradients (host code, no GPU needed): it says PLAIN only where a fill of the buffer is all that an
in-place operation on the gradient would do; everything else is left to the general path."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2203_13085_amd import _grad_walk

PLAIN, OTHER, MISSING = 0, 1, 2
P = torch.nn.Parameter


def _params(dtype=torch.float32):
    ps = [P(torch.zeros(s, dtype=dtype)) for s in ((3, 4), (5,), (2, 3, 4, 5), (1,))]
    for p in ps:
        p.grad = torch.ones_like(p)
    return ps


def _addr(ps):
    return (ctypes.c_void_p * len(ps))(*[p.grad.data_ptr() for p in ps])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_plain_gradients_and_their_versions(dtype):
    ps = _params(dtype)
    a = _addr(ps)
    before = [p.grad._version for p in ps]
    assert _grad_walk.state(ps, P, b"".join([a]), False) == PLAIN and [p.grad._version for p in ps] == before
    assert _grad_walk.state(ps, P, a, True) == PLAIN
    assert [p.grad._version for p in ps] == [v + 1 for v in before]
    assert _grad_walk.state(ps, P, None, False) == PLAIN and _grad_walk.state([], P, None, True) == PLAIN


def test_a_missing_gradient_is_told_from_a_replaced_one():
    ps = _params()
    a = _addr(ps)
    ps[1].grad = torch.ones(5)                       # elsewhere
    versions = [p.grad._version for p in ps]
    assert _grad_walk.state(ps, P, a, True) == OTHER and [p.grad._version for p in ps] == versions
    assert _grad_walk.state(ps, P, None, False) == PLAIN
    ps[3].grad = None
    assert _grad_walk.state(ps, P, a, True) == MISSING and _grad_walk.state(ps, P, None, False) == MISSING


def _strided():
    p = P(torch.zeros(4, 3))
    p.grad = torch.ones(3, 4).t()
    return p


def _with_history():
    p = P(torch.ones(4))
    (p * p).sum().backward(create_graph=True)
    return p


def _inference():
    p = P(torch.ones(4))
    with torch.inference_mode():
        g = torch.ones(4)
    p.grad = g
    return p


def _sparse():
    e = torch.nn.Embedding(6, 2, sparse=True)
    e(torch.tensor([1, 3])).sum().backward()
    return e.weight


def _swapped_data():
    p = P(torch.zeros(6))
    p.grad = torch.ones(6)
    p.grad.data = torch.ones(6)[2:]                   # a shorter tensor under the same object
    return p


def _negative():
    p = P(torch.zeros(4))
    p.grad = torch._neg_view(torch.ones(4))
    return p


def _other_type():
    class Q(P):
        pass
    q = Q(torch.zeros(4))
    q.grad = torch.ones(4)
    return q


def _forward_mode():
    import torch.autograd.forward_ad as fwAD
    p = P(torch.zeros(4))
    ctx = fwAD.dual_level()
    ctx.__enter__()
    p.grad = fwAD.make_dual(torch.ones(4), torch.ones(4))
    p._level = ctx                                     # closed by the test
    return p


def _lazy_clone():
    p = P(torch.zeros(4))
    p.grad = torch.ones(4)
    p._at = p.grad.data_ptr()                         # asked for later, it would un-share the buffer
    p._other = torch._lazy_clone(p.grad)              # one buffer until somebody writes
    return p


def _torch_function_subclass():
    class G(torch.Tensor):                            # no dispatcher of its own: only Python's __torch_function__
        @classmethod
        def __torch_function__(cls, func, types, args=(), kwargs=None):
            return super().__torch_function__(func, types, args, kwargs or {})
    p = P(torch.zeros(4))
    p.grad = torch.ones(4).as_subclass(G)
    return p


@pytest.mark.parametrize("make", [_lazy_clone, _torch_function_subclass, _strided, _with_history, _inference, _sparse, _swapped_data, _negative, _other_type, _forward_mode])
def test_anything_but_a_plain_gradient_goes_the_general_way(make):
    p = make()
    try:
        at = p._at if hasattr(p, "_at") else 0 if p.grad.layout != torch.strided else p.grad.data_ptr()
        a = np.array([at], dtype=np.uint64)
        if not p.grad.is_inference():
            v = p.grad._version
        assert _grad_walk.state([p], P, a, True) == OTHER
        if not p.grad.is_inference():
            assert p.grad._version == v
    finally:
        if hasattr(p, "_level"):
            p._level.__exit__(None, None, None)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_a_gradient_of_another_length_than_was_bound(dtype):
    ps = _params(dtype)
    a, sizes = _addr(ps), np.array([p.numel() * p.element_size() for p in ps], dtype=np.uint64)
    assert _grad_walk.state(ps, P, a, True, sizes) == PLAIN
    ps[2].data = ps[2].data[:1]                       # parameter and gradient shortened in step, at the bound address
    ps[2].grad = ps[2].grad[:1]
    assert ps[2].grad.data_ptr() == a[2] and ps[2].grad.shape == ps[2].shape
    versions = [p.grad._version for p in ps]
    assert _grad_walk.state(ps, P, a, True, sizes) == OTHER and [p.grad._version for p in ps] == versions
    ps[0].data, ps[0].grad = ps[0].data.to(torch.float64), None      # the same number of elements, of another width
    ps[0].grad = torch.ones(3, 4, dtype=torch.float64)
    wide = np.array([ps[0].grad.data_ptr()], dtype=np.uint64)
    assert _grad_walk.state(ps[:1], P, wide, True, sizes[:1].copy()) == OTHER


def test_bad_arguments_are_refused():
    ps = _params()
    with pytest.raises(ValueError):
        _grad_walk.state(ps, P, b"12345678", True)
    with pytest.raises(ValueError):
        _grad_walk.state(ps, P, _addr(ps), True, b"12345678")
    with pytest.raises(TypeError):
        _grad_walk.state(tuple(ps), P, None, True)
    assert _grad_walk.state([1, 2], P, None, True) == OTHER


@pytest.mark.parametrize("missing", [True, False])
def test_the_torch_class_works_without_the_walk(monkeypatch, missing):
    """Not built, or built for another torch: the module imports, says so, and walks in Python."""
    import importlib
    import sys
    import paper_2203_13085_amd
    from paper_2203_13085_amd import torch_api
    if missing:
        monkeypatch.delattr(paper_2203_13085_amd, "_grad_walk", raising=False)
        monkeypatch.setitem(sys.modules, "paper_2203_13085_amd._grad_walk", None)      # import fails
    else:
        monkeypatch.setattr(_grad_walk, "torch_version", "0.0.0")
    try:
        with pytest.warns(RuntimeWarning, match="native walk"):
            api = importlib.reload(torch_api)
        opt = api.LASGD.__new__(api.LASGD)
        opt._flat = _params()
        opt._check_bound()
        opt.zero_grad()
        assert not any(p.grad.any() for p in opt._flat)
        opt._flat[1].grad = None
        with pytest.raises(AssertionError):
            opt._check_bound()
    finally:
        monkeypatch.undo()
        importlib.reload(torch_api)
    assert torch_api._walk is _grad_walk

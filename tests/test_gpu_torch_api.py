"""End to end with real autograd gradients: K small torch models trained with the
LASGD wrapper on the GPU; the oracle is fed the very gradients autograd
produced (copied to the host each step) and must land on the same parameters."""
import copy

import numpy as np
import pytest
import torch

from oracle import lasgd_oracle as O32
from paper_2203_13085_amd import binding as B
from tests.parity_util import assert_close

pytestmark = pytest.mark.gpu


def _flat(tensors):
    return np.concatenate([t.detach().float().cpu().numpy().ravel() for t in tensors])


@pytest.mark.parametrize("m", [1, 3])
def test_k_models_with_autograd_gradients(m):
    from paper_2203_13085_amd.torch_api import LASGD
    torch.manual_seed(0)
    dev = torch.device("cuda:0")
    K, steps, lr, mu, wd = 3, 9, 0.05, 0.9, 1e-3
    base = torch.nn.Sequential(torch.nn.Linear(20, 33), torch.nn.ReLU(), torch.nn.Linear(33, 5)).to(dev)
    replicas = [copy.deepcopy(base) for _ in range(K)]
    opt = LASGD(replicas, lr=lr, momentum=mu, nesterov=True, weight_decay=wd, m=m, no_decay_1d=True)
    params0 = [p for p in base.parameters()]
    numels = [p.numel() for p in params0]
    wds = [0.0 if p.dim() <= 1 else wd for p in params0]
    orc = O32.Oracle(K, numels, mu, True, wds)
    orc.set_model(_flat(params0))
    try:
        started, tau = False, 0
        for step in range(steps):
            opt.zero_grad()
            for k, model in enumerate(replicas):
                g = torch.Generator(device=dev); g.manual_seed(1000 * step + k)
                x = torch.randn(16, 20, generator=g, device=dev)
                y = torch.randn(16, 5, generator=g, device=dev)
                torch.nn.functional.mse_loss(model(x), y).backward()
            torch.cuda.synchronize()
            grads = [_flat([p.grad for p in model.parameters()]) for model in replicas]
            fired = opt.step()
            orc.local_step(grads, lr)
            if not started:
                orc.snapshot(); orc.average(); started = True
                assert not fired
            else:
                tau += 1
                if tau == m:
                    orc.merge(True); orc.average(); tau = 0
                    assert fired
                else:
                    assert not fired
            torch.cuda.synchronize()
            for k, model in enumerate(replicas):
                assert_close(_flat(list(model.parameters())), orc.x[k], f"step {step} replica {k}")
        assert_close(opt.center().numpy(), orc.z, "centre")
        # replicas have moved apart and back: they differ, but not by much
        a, b = _flat(list(replicas[0].parameters())), _flat(list(replicas[1].parameters()))
        assert 0 < np.abs(a - b).max() < 0.5
    finally:
        opt.close()


def test_zero_grad_clears_every_gradient_in_place():
    """All buffers, also one that the caller replaced, at unchanged addresses; saved-tensor checks still see the write;
    a dropped gradient is refused as before."""
    from paper_2203_13085_amd.torch_api import LASGD
    dev = torch.device("cuda:0")
    replicas = [torch.nn.ParameterList([torch.nn.Parameter(torch.ones(n, device=dev)) for n in (5, 1, 4097)]) for _ in range(3)]
    opt = LASGD(replicas, lr=0.1)
    try:
        ps = [p for r in replicas for p in r]
        ps[2].grad = torch.ones(4097, device=dev)
        for p in ps:
            p.grad.fill_(2.0)
        at = [(p.grad.data_ptr(), p.grad._version) for p in ps]
        opt.zero_grad()
        torch.cuda.synchronize()
        for p, (ptr, version) in zip(ps, at):
            assert p.grad.data_ptr() == ptr and p.grad._version > version and not p.grad.any()
        ps[1].grad = None
        with pytest.raises(AttributeError):
            opt.zero_grad()
    finally:
        opt.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("hint", [3, 4])
def test_zero_grad_clears_every_bound_gradient_and_nothing_else(dtype, hint):
    """One launch over the records: tensors around a tile's 256 elements and a lane's four, several tensors in a block of
    tiles; what lies behind a gradient's end stays."""
    from paper_2203_13085_amd.torch_api import LASGD
    numels = [1, 3, 4, 5, 255, 256, 257, 1030, 2, 70001]
    dev, guard = torch.device("cuda:0"), 8
    nets, slabs = [], []
    for k in range(3):
        net = torch.nn.Module()
        net.ps = torch.nn.ParameterList([torch.nn.Parameter(torch.zeros(n, device=dev, dtype=dtype)) for n in numels])
        for p in net.ps:
            slab = torch.full((p.numel() + guard,), 7.0, device=dev, dtype=dtype)
            p.grad = slab[:p.numel()]
            slabs.append(slab)
        nets.append(net)
    opt = LASGD(nets, lr=0.1)
    try:
        opt.ctx.set_tuning(nontemporal=hint)
        before = [p.grad._version for p in opt._flat]
        for _ in range(2):
            opt.zero_grad()
            torch.cuda.synchronize()
            for slab, p in zip(slabs, opt._flat):
                assert not p.grad.any() and bool((slab[p.numel():] == 7.0).all())
            for slab in slabs:
                slab.fill_(7.0)
        assert all(p.grad._version > v for p, v in zip(opt._flat, before))
        # a gradient elsewhere: cleared where it is now, as before; the bound buffer is not touched
        moved = torch.full_like(opt._flat[5], 3.0)
        opt._flat[5].grad = moved
        opt.zero_grad()
        torch.cuda.synchronize()
        assert not moved.any() and bool((slabs[5] == 7.0).all()) and not opt._flat[4].grad.any()
        opt._flat[5].grad = None
        with pytest.raises(AttributeError):
            opt.zero_grad()
        with pytest.raises(AssertionError):
            opt.step()
    finally:
        opt.close()


def test_zero_grad_is_seen_by_a_graph_that_saved_the_gradient():
    from paper_2203_13085_amd.torch_api import LASGD
    net = torch.nn.Linear(8, 8, device="cuda:0")
    opt = LASGD([net], lr=0.1)
    try:
        w = torch.ones(8, device="cuda:0", requires_grad=True)
        y = (net.bias.grad * w).sum()                       # saves the gradient for w's backward
        opt.zero_grad()
        with pytest.raises(RuntimeError, match="modified by an inplace operation"):
            y.backward()
    finally:
        opt.close()


def test_zero_grad_after_close():
    """The gradients are the modules' own and outlive the library's tables."""
    from paper_2203_13085_amd.torch_api import LASGD
    net = torch.nn.Linear(8, 8, device="cuda:0")
    opt = LASGD([net], lr=0.1)
    for p in net.parameters():
        p.grad.fill_(2.0)
    opt.close()
    opt.zero_grad()
    torch.cuda.synchronize()
    assert not any(p.grad.any() for p in net.parameters())

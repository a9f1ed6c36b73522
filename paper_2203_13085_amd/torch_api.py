"""LASGD for K torch models that live on one GPU.

A thin convenience over the binding for callers who already have K replicas of a
torch module (the paper's P workers, Sec. 4): it binds every replica's parameter
and gradient tensors to a LASGD context once and then runs one iteration of
Algorithm 1 per `step()` -- a local update of all replicas, and every m-th
call the fused global update followed by the launch of the next mean on the
side stream.  All arithmetic happens in the library's kernels; torch supplies
the tensors, the autograd gradients and the streams.

Gradient tensors are allocated here once and attached to the parameters
(`p.grad`), so that autograd accumulates into buffers whose addresses never
change; clear them with `zero_grad()` of this class (or
`module.zero_grad(set_to_none=False)`), never by dropping them.
"""
from __future__ import annotations

import warnings
from typing import List, Optional, Sequence

import numpy as np
import torch

from . import binding as B


def _load_walk():
    """The native walk over gradients, or None (and a warning) where it was not built for this very torch: it reads torch's
    objects through the headers it was compiled against.  Everything works without it, with walks in Python."""
    try:
        from . import _grad_walk
        if _grad_walk.torch_version == torch.__version__:
            return _grad_walk
        why = f"it was built for torch {_grad_walk.torch_version}, this is {torch.__version__}"
    except (ImportError, AttributeError) as e:
        why = str(e)
    warnings.warn(f"the native walk over gradients is left out, zero_grad() and step() take longer: {why} "
                  "(build it with `python -m paper_2203_13085_amd.build`)", RuntimeWarning, stacklevel=2)
    return None


_walk = _load_walk()


class LASGD:
    def __init__(self, replicas: Sequence[torch.nn.Module], lr: float, momentum: float = 0.9,
                 nesterov: bool = True, weight_decay: float = 0.0, m: int = 1,
                 no_decay_1d: bool = False, side_stream: bool = True):
        """replicas: K modules with identical parameter lists on the same GPU, already
        holding the same initial weights (every node starts from the same model).
        m: local steps per global update (tau_max with the early exit disabled).
        no_decay_1d: apply no weight decay to 1-D tensors (norm scales, biases)."""
        assert len(replicas) >= 1 and m >= 1
        self.replicas = list(replicas)
        self.params: List[List[torch.nn.Parameter]] = [[p for p in r.parameters() if p.requires_grad] for r in self.replicas]
        first = self.params[0]
        assert first, "no trainable parameters"
        dev = first[0].device
        assert dev.type == "cuda", "the LASGD path runs only on the GPU"
        dtype = first[0].dtype
        assert dtype in (torch.float32, torch.bfloat16)
        for ps in self.params:
            assert len(ps) == len(first)
            for p, q in zip(ps, first):
                assert p.shape == q.shape and p.dtype == dtype and p.device == dev and p.is_contiguous()
        self._flat = [p for ps in self.params for p in ps]
        self._bytes = np.array([p.numel() * p.element_size() for p in self._flat], dtype=np.uint64)    # what the library clears
        self.lr, self.m, self.tau, self.t = float(lr), int(m), 0, 0
        self.device = dev
        self.main = torch.cuda.Stream(device=dev)
        self.side = torch.cuda.Stream(device=dev) if side_stream else self.main
        wd = [0.0 if (no_decay_1d and p.dim() <= 1) else float(weight_decay) for p in first]
        with torch.cuda.device(dev):
            self.ctx = B.Context(len(self.replicas), [p.numel() for p in first],
                                 storage=B.BF16 if dtype == torch.bfloat16 else B.F32,
                                 momentum=momentum, nesterov=nesterov, weight_decay=wd,
                                 main_stream=self.main.cuda_stream, side_stream=self.side.cuda_stream)
            for k, ps in enumerate(self.params):
                for p in ps:
                    if p.grad is None or not p.grad.is_contiguous():
                        p.grad = torch.zeros_like(p, memory_format=torch.contiguous_format)
                self.ctx.bind(k, [p.data_ptr() for p in ps], [p.grad.data_ptr() for p in ps])
            torch.cuda.synchronize(dev)
            if dtype == torch.bfloat16:
                self.ctx.init_master()
        self._started = False

    def zero_grad(self) -> None:
        # The gradients sit where the library reads them, so the library clears them, in one launch, once a native walk has
        # seen that every one is there, at its address and plain.  A list of 632 tensors (MobileNetV2, K = 4) took
        # _foreach_zero_ eight launches and, with the list and the version counters, 170 us of host time; this takes 20.
        if _walk and self._eager() and _walk.state(self._flat, torch.nn.Parameter, b"".join(self.ctx.bound_grads), True,
                                                   self._bytes) == 0:
            self.ctx.zero_grads(torch.cuda.current_stream(self.device).cuda_stream)
            return
        grads = [p.grad for p in self._flat]
        try:
            torch._foreach_zero_(grads)
            torch.autograd.graph.increment_version(grads)   # a graph that saved one of them has to notice, as after zero_()
        except TypeError:                           # a gradient was dropped: fail where the first one is missing
            for g in grads:
                g.zero_()

    def _eager(self) -> bool:
        # the library's tables are there, nobody watches torch's operations, and no graph is recorded that could outlive the tables
        return (torch._C._len_torch_dispatch_stack() == 0 and torch._C._len_torch_function_stack() == 0
                and torch._C._functorch.peek_interpreter_stack() is None and not torch.compiler.is_compiling()
                and self.ctx.is_open and torch.cuda.current_device() == self.device.index
                and not torch.cuda.is_current_stream_capturing())

    def _check_bound(self) -> None:
        # a dropped or replaced .grad would leave the library reading a stale buffer
        if _walk and _walk.state(self._flat, torch.nn.Parameter, None, False) == 0:
            return
        for p in self._flat:
            assert p.grad is not None, "a gradient buffer was dropped (use zero_grad(set_to_none=False))"

    @torch.no_grad()
    def step(self, lr: Optional[float] = None) -> bool:
        """One iteration of Algorithm 1 for all replicas, after their backward passes.
        Returns True if a global update happened in this call."""
        self._check_bound()
        lr = self.lr if lr is None else float(lr)
        cur = torch.cuda.current_stream(self.device)
        self.main.wait_stream(cur)                  # gradients are complete before the update reads them
        fired = False
        if not self._started:                       # steps 2-5: first update, send, start the All-Reduce
            self.ctx.local_step(lr)
            self.ctx.snapshot()
            self.ctx.average()
            self._started = True
            self.tau = 0
        else:                                       # steps 6-9
            self.tau += 1
            if self.tau >= self.m:
                self.ctx.step_merge(lr, True)
                self.ctx.average()
                self.tau, self.t, fired = 0, self.t + 1, True
            else:
                self.ctx.local_step(lr)
        cur.wait_stream(self.main)                  # the next forward sees the new parameters
        return fired

    def center(self) -> torch.Tensor:
        """The current mean model z (flat, fp32), e.g. for evaluation."""
        return torch.from_numpy(np.ascontiguousarray(self.ctx.read_state(B.STATE_Z)))

    def close(self) -> None:
        self.ctx.close()

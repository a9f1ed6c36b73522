"""The work a user of this framework has it do, as timed cases.

A case is a model's parameter list, a replica count, a cadence, a storage type and the way the framework is called.
One pass is what a training loop issues between two global updates (or for one step of a comparator), on state that
stays on the GPU; its outputs are the replicas' parameters, whole, and whatever else the caller can see.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2203_13085_amd import binding as B
from paper_2203_13085_amd import workloads as W

DEV = "cuda:0"
ROW = 256                      # elements: every tensor of a flat parameter buffer starts on such a boundary
MU, WD = 0.9, 1e-4             # momentum and weight decay of the workloads in use


# ---- parameter lists ---------------------------------------------------------------------------------------------
def _numels(c):
    if c["list"] == "flat":                                 # one vector: a flattened model
        return [int(c["n"])]
    if c["list"] == "small":                                # the framework's own ragged little list
        return W.small().numels
    if c["list"] == "ragged":                               # `tensors` tensors of very unlike, odd sizes, about n elements
        r = random.Random(int(c["lseed"]))
        w = [math.exp(r.uniform(0.0, 8.0)) for _ in range(int(c["tensors"]))]
        return [max(1, int(c["n"] * a / sum(w))) for a in w]
    shapes = W.mobilenet_v2_shapes() if c["list"] == "mobilenetv2" else W.resnet_shapes(int(c["list"][6:]))
    return [W.numel(s) for _, s in shapes]


def _stds(c):
    """Per tensor: the standard deviation of its initial draw, or None and its constant (norm scales 1, shifts 0)."""
    if c["list"] in ("flat", "small", "ragged"):
        return [(0.01, 0.0)] * len(_numels(c))
    shapes = W.mobilenet_v2_shapes() if c["list"] == "mobilenetv2" else W.resnet_shapes(int(c["list"][6:]))
    return [(W.init_std(kind, s, "he"), 1.0 if kind == "bn_gamma" else 0.0) for kind, s in shapes]


def _offsets(numels):
    off = [0]
    for n in numels:
        off.append(off[-1] + (n + ROW - 1) // ROW * ROW)
    return off


# ---- the cases ---------------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest calls: a handful of short, odd tensors, launch after launch (a head or an adapter being tuned)
        dict(name="small-list-k3", call="cycle", list="small", K=3, m=2, storage="f32", streams=2),
        # a flattened model of a million parameters, the small benchmark workload
        dict(name="flat-1m-k4", call="cycle", list="flat", n=1 << 20, K=4, m=2, storage="f32", streams=1),
        # many small tensors and a global update every step
        dict(name="mobilenetv2-k16", call="cycle", list="mobilenetv2", K=16, m=1, storage="f32", streams=1),
        # the ordinary size
        dict(name="resnet18-k8", call="cycle", list="resnet18", K=8, m=4, storage="f32", streams=1),
        # the headline workload: global update every four steps, the mean on a second stream
        dict(name="resnet50-k8", call="cycle", list="resnet50", K=8, m=4, storage="f32", streams=2),
        # the largest: bf16 parameters and gradients with fp32 masters, 32 replicas, update every eight steps
        dict(name="resnet50-bf16-k32", call="cycle", list="resnet50", K=32, m=8, storage="bf16", streams=2),
        # global update and next mean in one pass, every step
        dict(name="resnet18-bf16-k12-fused", call="fused", list="resnet18", K=12, m=1, storage="bf16", streams=1),
        # the synchronous comparator: all-reduced gradients, one shared step
        dict(name="resnet50-k8-sgd-ar", call="sgd_ar", list="resnet50", K=8, storage="f32", streams=1),
        # replicas at their own pace: masked steps with a step size each, one global update at the round's end
        dict(name="resnet18-k8-adaptive", call="adaptive", list="resnet18", K=8, storage="f32", streams=2, rseed=3),
        # partial All-Reduce with elastic coefficients: some replicas sit the round out
        dict(name="mobilenetv2-k16-partial", call="partial", list="mobilenetv2", K=16, m=2, storage="f32", streams=2, rseed=5,
             alpha=0.5, beta=0.5),
        # the call that needs no context and allocates nothing, on vectors of ResNet-50's size
        dict(name="static-k8", call="static", list="flat", n=25557032, K=8, storage="f32"),
        # torch modules through the optimizer class: clear the gradients, backward, step
        dict(name="torch-mobilenetv2-k4", call="torch", list="mobilenetv2", K=4, m=2, storage="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["cycle", "cycle", "cycle", "fused", "sgd_ar", "adaptive", "partial", "static", "torch"])
    c = dict(call=call, list=rng.choice(["flat", "ragged", "ragged", "mobilenetv2", "resnet18", "resnet50"]))
    if call == "static":
        c["list"] = "flat"
    if c["list"] in ("flat", "ragged"):
        c["n"] = _log(rng, 1000, 3.0e7)
    if c["list"] == "ragged":
        c["tensors"] = _log(rng, 2, 250)
        c["lseed"] = rng.randrange(1 << 20)
    n = sum(_numels(c))
    c["K"] = _log(rng, 1, max(1, min(64, int(4.0e8 / n))))
    c["storage"] = "f32" if call == "static" else rng.choice(["f32", "f32", "bf16"])
    if call == "torch":
        c["K"] = min(c["K"], 8)
    if call in ("cycle", "fused", "partial", "torch"):
        c["m"] = rng.choice([1, 2, 3, 4, 8]) if call == "cycle" else rng.choice([1, 2, 3])
    if call not in ("static", "torch"):
        c["streams"] = rng.choice([1, 2])
    if call == "cycle":
        c["nesterov"] = rng.random() < 0.8
        c["separate"] = rng.random() < 0.25          # local step and global update as two calls
    if call in ("adaptive", "partial"):
        c["rseed"] = rng.randrange(1 << 20)
    if call == "partial":
        c["alpha"], c["beta"] = rng.choice([(1.0, 1.0), (0.5, 0.5), (0.25, 1.0)])
    return c


def _lr(c):
    return {"flat": 0.1, "small": 0.05, "ragged": 0.1, "mobilenetv2": 0.4, "resnet18": 0.4, "resnet50": 0.8}[c["list"]]


def _counts(c):
    """Local steps of each replica in one adaptive round, 1..5 as in the paper's histogram (most nodes take two)."""
    r = random.Random(int(c["rseed"]))
    return [r.choices([1, 2, 3, 4, 5], [0.15, 0.6, 0.15, 0.05, 0.05])[0] for _ in range(c["K"])]


def _lrs(c):
    """A step size per replica: each node's schedule follows its own clock."""
    return [_lr(c) * (1.0 - 0.01 * (k % 5)) for k in range(c["K"])]


def _members(c):
    """Bit mask of a partial round's participants: about two thirds, at least one."""
    r = random.Random(int(c["rseed"]))
    return sum(1 << k for k in range(c["K"]) if r.random() < 0.67) or 1


# ---- inputs ------------------------------------------------------------------------------------------------------
def _inputs(c, seed):
    """(x0 [total], g [K, total]) on the GPU in the storage type; gaps between tensors hold zeros."""
    numels = _numels(c)
    off = _offsets(numels)
    dt = torch.bfloat16 if c["storage"] == "bf16" else torch.float32
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    x0 = torch.randn(off[-1], generator=gen, device=DEV)
    gap = torch.ones(off[-1], device=DEV)
    for n, o, (std, const) in zip(numels, off, _stds(c)):
        if std is None:
            x0[o:o + n] = const
        else:
            x0[o:o + n] *= std
        x0[o + n:o + (n + ROW - 1) // ROW * ROW] = 0.0
        gap[o + n:o + (n + ROW - 1) // ROW * ROW] = 0.0
    g = torch.empty(c["K"], off[-1], dtype=dt, device=DEV)
    for k in range(c["K"]):                                            # gradients differ from replica to replica
        g[k] = torch.randn(off[-1], generator=gen, device=DEV) * 1e-3 * gap
    return x0.to(dt), g


def _static_inputs(c, seed):
    """Sent models that have drifted apart, and local models a step further on."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    K, n = c["K"], int(c["n"])
    rows = (n + ROW - 1) // ROW * ROW
    x, sent = torch.zeros(K, rows, device=DEV), torch.zeros(K, rows, device=DEV)
    base = torch.randn(n, generator=gen, device=DEV) * 0.01
    for k in range(K):
        sent[k, :n] = base + torch.randn(n, generator=gen, device=DEV) * 1e-3
        x[k, :n] = sent[k, :n] + torch.randn(n, generator=gen, device=DEV) * 1e-3
    return x, sent


_made = []


def _streams():
    """The program's two streams: one that trains and one for the All-Reduce, whatever contexts it holds."""
    if not _made:
        _made.extend(torch.cuda.Stream(device=DEV) for _ in range(2))
    return _made


class _State:
    pass


class _Net(torch.nn.Module):
    """A module with the given list of parameters, which are views of one flat buffer."""

    def __init__(self, flat, grad, numels, off):
        super().__init__()
        self.ps = torch.nn.ParameterList([torch.nn.Parameter(flat[o:o + n]) for n, o in zip(numels, off)])
        for p, n, o in zip(self.ps, numels, off):
            p.grad = grad[o:o + n]


def prepare(case, seed):
    c, st = case, _State()
    st.c = c
    K = c["K"]
    if c["call"] == "static":
        st.x, st.sent = _static_inputs(c, seed)
        st.xp, st.sp = [t.data_ptr() for t in st.x], [t.data_ptr() for t in st.sent]
        return st
    numels = _numels(c)
    off = _offsets(numels)
    x0, st.g = _inputs(c, seed)
    st.x = x0.repeat(K, 1)                                                # every replica starts from the same model
    st.lr = _lr(c)
    if c["call"] == "torch":
        from paper_2203_13085_amd.torch_api import LASGD
        st.back = st.g.clone()                                             # what the backward pass adds to the gradients
        nets = [_Net(st.x[k], st.g[k], numels, off) for k in range(K)]
        st.opt = LASGD(nets, lr=st.lr, momentum=MU, nesterov=True, weight_decay=WD, m=c["m"])
        st.opt.step()                                                      # first update, send, first All-Reduce
        return st
    main, side = _streams()
    if c["streams"] == 1:
        side = main
    bf16 = c["storage"] == "bf16"
    esize = 2 if bf16 else 4
    torch.cuda.synchronize()
    st.ctx = B.Context(K, numels, storage=B.BF16 if bf16 else B.F32, momentum=MU, nesterov=c.get("nesterov", True),
                       wd_scalar=WD, main_stream=main.cuda_stream, side_stream=side.cuda_stream)
    for k in range(K):
        st.ctx.bind(k, [st.x[k].data_ptr() + o * esize for o in off[:-1]], [st.g[k].data_ptr() + o * esize for o in off[:-1]])
    if bf16:
        st.ctx.init_master()
    if c["call"] == "sgd_ar":
        return st
    st.ctx.local_step(st.lr)                                               # the algorithm's prologue: first update, send
    st.ctx.snapshot()
    if c["call"] == "fused":
        st.ctx.average()
    if c["call"] == "adaptive":
        st.lrs = _lrs(c)
        counts = _counts(c)
        st.ticks = [sum(1 << k for k in range(K) if counts[k] > j) for j in range(max(counts))]
    if c["call"] == "partial":
        st.mask = _members(c)
        st.ctx.average()                                                   # the first mean sets the centre
        st.ctx.merge(True)
        st.ctx.set_elastic(c["alpha"], c["beta"])
    return st


# ---- one pass ----------------------------------------------------------------------------------------------------
def run(state):
    st, c = state, state.c
    call = c["call"]
    if call == "static":
        B.global_update_static(st.xp, st.sp, int(c["n"]), True, torch.cuda.current_stream().cuda_stream)
        return {"x": st.x, "sent": st.sent}
    if call == "torch":
        for _ in range(c["m"]):
            st.opt.zero_grad()
            st.g.add_(st.back)                                             # the backward pass accumulates
            st.opt.step()
        return {"x": st.x, "grad": st.g}
    ctx, lr = st.ctx, st.lr
    if call == "cycle":
        ctx.average()
        for _ in range(c["m"] - 1):
            ctx.local_step(lr)
        if c.get("separate"):
            ctx.local_step(lr)
            ctx.merge(True)
        else:
            ctx.step_merge(lr, True)
    elif call == "fused":
        for _ in range(2):                                                 # the second update uses the first one's mean
            for _ in range(c["m"] - 1):
                ctx.local_step(lr)
            ctx.step_merge_average(lr)
    elif call == "sgd_ar":
        ctx.sgd_ar_step(lr)
    elif call == "adaptive":
        ctx.average()
        for mask in st.ticks[:-1]:
            ctx.local_step_ex(st.lrs, mask)
        ctx.step_merge_ex(st.lrs, st.ticks[-1], (1 << c["K"]) - 1, True)
    else:
        ctx.average_ex(st.mask)
        for _ in range(c["m"] - 1):
            ctx.local_step(lr)
        ctx.step_merge_ex([lr] * c["K"], (1 << c["K"]) - 1, st.mask, True)
    return {"x": st.x}


# ---- what a pass cannot do without ---------------------------------------------------------------------------------
def work(case):
    """Each call's inputs read once and its outputs written once.  A local step of one replica moves 20 bytes a parameter
    in either storage type (f32: g, x, v in, x, v out; bf16: 2 + 4 + 4 in, 4 + 4 + 2 out) and does 8 operations; a global
    update adds s in and out and z once; a mean reads the P sent models and writes z."""
    c = case
    K, n = c["K"], float(sum(_numels(c)))
    step, step_f = 20.0 * n, 8.0 * n
    upd, upd_f = 8.0 * n, 2.0 * n

    def mean(p):
        return 4.0 * (p + 1) * n

    call, m = c["call"], c.get("m", 1)
    if call == "static":                       # x, sent in and out; z need not leave the chip
        return {"bytes": 16.0 * K * n, "flops": 3.0 * K * n}
    if call == "cycle":
        extra = (8.0 * K * n) if c.get("separate") else 0.0                # x goes out and comes in again between the two
        return {"bytes": m * K * step + K * upd + 4 * n + mean(K) + extra, "flops": m * K * step_f + K * (upd_f + n)}
    if call == "torch":                        # clear, accumulate (two in, one out), step
        return {"bytes": m * (4.0 + 12.0) * K * n * (0.5 if c["storage"] == "bf16" else 1.0)
                + m * K * step + K * upd + 4 * n + mean(K), "flops": m * K * (step_f + n) + K * (upd_f + n)}
    if call == "fused":
        return {"bytes": 2 * (m * K * step + K * upd + 8 * n), "flops": 2 * (m * K * step_f + K * (upd_f + n))}
    if call == "sgd_ar":
        return {"bytes": K * step, "flops": K * (step_f + n)}
    if call == "adaptive":
        a = sum(_counts(c))
        return {"bytes": a * step + K * upd + 4 * n + mean(K) + _idle(c) * 8.0 * n, "flops": a * step_f + K * (upd_f + n)}
    p = bin(_members(c)).count("1")
    blend = 4.0 * n if c["beta"] != 1.0 else 0.0
    return {"bytes": m * K * step + p * upd + 4 * n + mean(p) + blend, "flops": m * K * step_f + p * (upd_f + n)}


def _idle(c):
    """Replicas that take the round's global update without a local step in that call (x in and out)."""
    counts = _counts(c)
    return sum(1 for k in counts if k < max(counts))


def tolerance(case):
    """Four times the distance from the 64-bit result.  fp32 (6e-8): a pass is a dozen roundings of values of one size,
    2^-24 each.  bf16 (1.7e-3): the parameters come back with 8 bits, and a last bit of the master can turn one over."""
    if case["storage"] == "bf16":
        return {"rel": 7e-3, "max": 8e-3}
    return {"rel": 2.5e-7, "max": 4e-6}


# ---- the same in 64 bits ---------------------------------------------------------------------------------------------
class _Ref:
    def __init__(self, c, seed):
        f = lambda a: float(np.float32(a))  # noqa: E731  (the entry points take 32-bit coefficients)
        x0, g = _inputs(c, seed)
        self.x = x0.double().repeat(c["K"], 1)
        self.g = g
        self.v = torch.zeros_like(self.x)
        self.s = torch.zeros_like(self.x)
        self.z = None
        self.mu, self.wd, self.f = f(MU), f(WD), f
        self.nesterov = c.get("nesterov", True)
        self.K = c["K"]

    def step(self, lr, mask=-1, g=None):
        for k in range(self.K):
            if not (mask >> k) & 1:
                continue
            g1 = (self.g[k].double() if g is None else g) + self.wd * self.x[k]
            self.v[k] = self.mu * self.v[k] + g1
            d = g1 + self.mu * self.v[k] if self.nesterov else self.v[k]
            self.x[k] -= self.f(lr[k] if isinstance(lr, list) else lr) * d

    def send(self, mask=-1):
        for k in range(self.K):
            if (mask >> k) & 1:
                self.s[k] = self.x[k]

    def mean(self, mask=-1, beta=1.0):
        ks = [k for k in range(self.K) if (mask >> k) & 1]
        z = sum(self.s[k] for k in ks) / len(ks)
        self.z = z if self.z is None or beta == 1.0 else (1.0 - beta) * self.z + beta * z

    def merge(self, mask=-1, alpha=1.0):
        for k in range(self.K):
            if (mask >> k) & 1:
                self.x[k] += alpha * (self.z - self.s[k])
        self.send(mask)


def exact(case, seed):
    c = case
    if c["call"] == "static":
        x, sent = _static_inputs(c, seed)
        out = sent.double().mean(0) + (x.double() - sent.double())
        return {"x": out, "sent": out}
    r, lr = _Ref(c, seed), _lr(c)
    call, m = c["call"], c.get("m", 1)
    if call == "sgd_ar":
        r.step(lr, g=sum(r.g[k].double() for k in range(r.K)) / r.K)
        return {"x": r.x}
    r.step(lr)
    r.send()
    if call in ("cycle", "torch"):
        r.mean()
        for _ in range(m):
            r.step(lr)
        r.merge()
    elif call == "fused":
        for _ in range(2):
            r.mean()
            for _ in range(m):
                r.step(lr)
            r.merge()
    elif call == "adaptive":
        r.mean()
        counts = _counts(c)
        for j in range(max(counts)):
            r.step(_lrs(c), sum(1 << k for k in range(r.K) if counts[k] > j))
        r.merge()
    else:
        r.mean()
        r.merge()
        members = _members(c)
        r.mean(members, c["beta"])
        for _ in range(m):
            r.step(lr)
        r.merge(members, c["alpha"])
    if call == "torch":
        return {"x": r.x, "grad": r.g.double()}
    return {"x": r.x}

"""GPU parity at the benchmark's full sizes and launch configuration.

configs[1], [2], [3] (ResNet-18 K=8, ResNet-50 K=8, MobileNetV2 K=16): Algorithm 1
runs on the whole workload on both sides -- default launch shape, the mean on the
stream bench.py times it on -- and EVERY element of the parameters, momentum,
sent models and mean is compared after the prologue and after every loop
iteration.  configs[4] (ResNet-50, bf16 storage, K=32; 13 GB of state): the
oracle also follows the whole workload; a sample of columns (tensor edges, tile
boundaries, random) is compared after every step and every element of every
array after each global update and at the end.

Gradients are drawn on the device with a seeded generator (an input recipe, not
part of the method) and copied to the host, so both sides consume the same bits.
"""
import os

import numpy as np
import pytest
import torch

from oracle import lasgd_oracle as O32
from paper_2203_13085_amd import binding as B
from paper_2203_13085_amd import workloads as W
from tests.parity_util import ATOL, RTOL, assert_close, say

pytestmark = pytest.mark.gpu

HOST_THREADS = max(1, min(16, len(os.sched_getaffinity(0))))


def assert_same(got: np.ndarray, ref: np.ndarray, what: str, max_bit_diffs: int = 0) -> int:
    """Whole-array comparison that is cheap when the arrays agree: bit patterns first;
    only the elements that differ are then held against the tolerance (+0 == -0)."""
    assert got.shape == ref.shape, f"{what}: shape {got.shape} vs {ref.shape}"
    if got.dtype == np.uint16:
        bad = np.flatnonzero(got != ref)
        assert bad.size == 0, f"{what}: {bad.size} of {got.size} bf16 patterns differ, first at {bad[:5]}"
        return 0
    gb, rb = got.view(np.uint32), ref.view(np.uint32)
    if np.array_equal(gb, rb):
        return 0
    idx = np.flatnonzero(gb != rb)
    g64, r64 = got[idx].astype(np.float64), ref[idx].astype(np.float64)
    ok = np.abs(g64 - r64) <= ATOL + RTOL * np.abs(r64)
    assert ok.all(), (f"{what}: {int((~ok).sum())} of {got.size} outside 1e-6 rel / 1e-7 abs, first at "
                      f"{idx[~ok][:5]}, max |d| = {np.abs(g64 - r64).max():.3e}")
    nbits = int(np.sum(~((g64 == 0) & (r64 == 0))))
    assert nbits <= max_bit_diffs, f"{what}: within tolerance but {nbits} of {got.size} differ in bits, first at {idx[:5]}"
    return nbits


def _sample_columns(numels, rng, n_random):
    off = np.concatenate([[0], np.cumsum(numels)]).astype(np.int64)
    picks = []
    for t, n in enumerate(numels):
        edge = np.unique(np.clip(np.concatenate([np.arange(0, 9), np.arange(n - 9, n)]), 0, n - 1))
        picks.append(off[t] + edge)
    order = np.argsort(numels)
    for t in list(order[:3]) + list(order[-3:]):          # smallest and largest tensors: tile boundaries
        n = numels[t]
        b = np.arange(256, n, 256)
        if b.size > 64:
            b = b[rng.choice(b.size, 64, replace=False)]
        band = (b[:, None] + np.arange(-4, 5)[None, :]).ravel()
        picks.append(off[t] + np.clip(band, 0, n - 1))
    picks.append(rng.integers(0, off[-1], n_random))
    cols = np.unique(np.concatenate(picks))
    tensor_of = np.searchsorted(off, cols, side="right") - 1
    counts = np.bincount(tensor_of, minlength=len(numels))
    assert counts.min() >= 1
    return cols, counts


def _device_gradients(dev, w, gen, step):
    """Draw this step's K gradients on the device; return them packed on the host."""
    dev.ctx.sync()
    out = []
    for k in range(w.K):
        gen.manual_seed(1_000_003 * w.seed + 7919 * step + k)
        g = torch.randn(dev.g[k].numel(), generator=gen, device=dev.dev) * 1e-3
        dev.g[k].copy_(g.to(dev.g[k].dtype))
        out.append(dev._get(dev.g[k]))
    torch.cuda.synchronize()
    return out


def _compare_everything(dev, orc, step, z_ties):
    w = dev.w
    bf16 = w.storage == "bf16"
    for k in range(w.K):
        tag = f"step {step} replica {k}"
        if bf16:
            assert_same(dev.params(k), orc.x16[k], f"bf16 params {tag}")
            assert_same(dev.ctx.read_state(B.STATE_X, k), orc.x[k], f"master {tag}")
        else:
            assert_same(dev.params(k), orc.x[k], f"x {tag}")
        assert_same(dev.ctx.read_state(B.STATE_V, k), orc.v[k], f"v {tag}")
        assert_same(dev.ctx.read_state(B.STATE_S, k), orc.s[k], f"s {tag}")
    return assert_same(dev.ctx.read_state(B.STATE_Z), orc.z, f"z step {step}", max_bit_diffs=z_ties)


def _full_size_run(cfg, fused_mean=False, full_every_step=True, sample=None, T=None, **changes):
    import dataclasses
    from paper_2203_13085_amd.driver import DeviceReplicas
    w = W.config(cfg)
    if T is not None:
        w = dataclasses.replace(w, T=T)
    w = dataclasses.replace(w, **changes)
    bf16 = w.storage == "bf16"
    nt = len(w.numels)
    wd = [w.weight_decay] * nt
    x0 = np.concatenate([W.initial_tensor(w, t) for t in range(nt)])
    if bf16:
        x0 = W.to_bf16_bits(x0)
    dev = DeviceReplicas(w, weight_decay=wd, side_stream=w.side_stream)
    try:
        tuning = dev.ctx.get_tuning()
        # the in-order mean (and the fused call) reproduce the oracle's sum bit for bit; the split
        # mean adds replica ranges separately and may differ at fp64 double-rounding ties
        z_ties = 0 if (fused_mean or tuning["avg_split"] == 1) else 5
        say(f"[full] configs[{cfg}] {w.name}: K={w.K} N={w.N} T={w.T} m={w.m} fused_mean={fused_mean} "
            f"side_stream={w.side_stream} host threads={HOST_THREADS} launch shape {tuning}")
        orc = O32.Oracle(w.K, w.numels, w.momentum, w.nesterov, wd, storage=w.storage, threads=HOST_THREADS)
        orc.set_model(x0)
        dev.load_model(x0)
        gen = torch.Generator(device=dev.dev)
        dcols = None
        if sample is not None:
            dcols = dev._idx[torch.from_numpy(sample).to(dev.dev)]

        def check(step, fired):
            if full_every_step or fired:
                nz = _compare_everything(dev, orc, step, z_ties)
                say(f"[full] configs[{cfg}] step {step}: every element of x, v, s, z agrees (z ties: {nz})")
                return
            dev.ctx.sync()
            for k in range(w.K):
                got = dev.x[k][dcols]
                if bf16:
                    assert_same(got.view(torch.int16).cpu().numpy().view(np.uint16), orc.x16[k][sample],
                                f"bf16 params (sample) step {step} replica {k}")
                else:
                    assert_same(got.cpu().numpy(), orc.x[k][sample], f"x (sample) step {step} replica {k}")

        g = _device_gradients(dev, w, gen, 0)
        orc.prologue(g, w.lr)
        dev.prologue(w.lr)
        check(0, True)
        tau = 0
        for i in range(1, w.T + 1):
            g = _device_gradients(dev, w, gen, i)
            fired = orc.iteration(g, w.lr, w.m)
            tau = dev.iteration(w.lr, tau, w.m, fused_mean=fused_mean)
            check(i, fired or i == w.T)
        say(f"[full] configs[{cfg}] ok")
    finally:
        dev.close()
        del dev
        torch.cuda.empty_cache()


@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_full_size_every_element_every_step(cfg):
    _full_size_run(cfg)


def test_full_size_fused_mean_every_element_every_step():
    # configs[3] (a global update every step) through lasgd_step_merge_average
    _full_size_run(3, fused_mean=True)


@pytest.mark.parametrize("K,storage", [(8, "f32"), (12, "f32"), (12, "bf16")])
def test_full_size_fused_mean_in_one_kernel(K, storage):
    """The ResNet-18 list, which streams, through lasgd_step_merge_average at replica counts that stay in one kernel: whole
    loads and two workgroups a CU at K = 8, two replicas a wave with staged loads at K = 12 (MobileNetV2 with its sixteen
    replicas, above, takes two kernels)."""
    _full_size_run(1, fused_mean=True, T=2, m=1, K=K, storage=storage)


def test_full_size_hundred_steps():
    """configs[2] for 100 loop iterations (25 global updates) with a fresh gradient every step: a column sample
    after every step, every element of every array after every global update.  Rounding differences would
    have a hundred steps to surface and grow; there must be none."""
    w = W.config(2)
    cols, _ = _sample_columns(w.numels, np.random.default_rng(102), 60000)
    _full_size_run(2, full_every_step=False, sample=cols, T=100)


def test_full_size_bf16_k32():
    w = W.config(4)
    cols, _ = _sample_columns(w.numels, np.random.default_rng(104), 60000)
    _full_size_run(4, full_every_step=False, sample=cols)


def test_one_huge_tensor_64bit_offsets():
    """A single tensor of 2^30 + 3 elements (4 GiB per array), K = 2: element offsets inside a
    tensor, arena offsets and replica strides all exceed 32 bits' worth of bytes; the tail is
    ragged.  Inputs are drawn on the device; the oracle follows a sample of columns."""
    import dataclasses
    from paper_2203_13085_amd.driver import DeviceReplicas
    n = (1 << 30) + 3
    w = dataclasses.replace(W.small(K=2, numels=(n,), m=2, T=3), name="huge")
    rng = np.random.default_rng(9)
    cols = np.unique(np.concatenate([np.arange(0, 16), np.arange(n - 16, n), rng.integers(0, n, 50000),
                                     (1 << 29) + np.arange(-8, 8), (1 << 30) + np.arange(-8, 3)]))
    wd = [w.weight_decay]
    dev = DeviceReplicas(w, weight_decay=wd)
    try:
        say(f"[huge] N={n} K={w.K} sample={cols.size}")
        dcols = torch.from_numpy(cols).to(dev.dev)
        gen = torch.Generator(device=dev.dev)
        gen.manual_seed(77)
        x0 = torch.randn(n, generator=gen, device=dev.dev) * 0.01
        for k in range(w.K):
            dev.x[k][:n].copy_(x0)
        torch.cuda.synchronize()
        orc = O32.Oracle(w.K, [cols.size], w.momentum, w.nesterov, wd)
        orc.set_model(x0[dcols].cpu().numpy())
        del x0

        def new_grads(step):
            dev.ctx.sync()
            out = []
            for k in range(w.K):
                gen.manual_seed(1000 * step + k)
                dev.g[k][:n].normal_(0.0, 1e-3, generator=gen)
                out.append(dev.g[k][dcols].cpu().numpy())
            torch.cuda.synchronize()
            return out

        def check(step):
            for k in range(w.K):
                dev.ctx.sync()
                assert_close(dev.x[k][dcols].cpu().numpy(), orc.x[k], f"x step {step} replica {k}")
                assert_close(dev.ctx.read_state(B.STATE_V, k)[cols], orc.v[k], f"v step {step} replica {k}")
                assert_close(dev.ctx.read_state(B.STATE_S, k)[cols], orc.s[k], f"s step {step} replica {k}")
            assert_close(dev.ctx.read_state(B.STATE_Z)[cols], orc.z, f"z step {step}")

        g = new_grads(0)
        orc.prologue(g, w.lr); dev.prologue(w.lr)
        check(0)
        tau = 0
        for i in range(1, w.T + 1):
            g = new_grads(i)
            orc.iteration(g, w.lr, w.m)
            tau = dev.iteration(w.lr, tau, w.m)
        check(w.T)
    finally:
        dev.close()
        del dev
        torch.cuda.empty_cache()

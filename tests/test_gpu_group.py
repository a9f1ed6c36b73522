"""GPU parity of the replica-group kernels (one workgroup per tile, one wave per
replica, the K values of an element meeting in LDS): lasgd_step_merge_average
against the oracle's global update + mean, and lasgd_sgd_ar_step against the
oracle's mean-gradient step, for every replica count that changes the group's
shape (1 wave, up to 16 waves, two replicas per wave, two passes)."""
import dataclasses

import numpy as np
import pytest

from paper_2203_13085_amd import binding as B
from paper_2203_13085_amd import workloads as W
from tests.parity_util import assert_close, compare_state, packed_inputs, run_parity, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 3, 8, 16, 17, 31, 32, 33, 64])
def test_fused_mean_every_group_shape(K):
    # ragged list: full rows, a scalar tail, a one-element tensor, several tiles
    w = W.small(K=K, numels=(1030, 1, 4, 257, 768), m=2, T=5)
    wd = [0.0, 1e-3, 1e-2, 1e-4, 5e-4]
    assert run_parity(w, weight_decay=wd, fused_mean=True) == 0        # z bit-exact: the sum runs in replica order


@pytest.mark.parametrize("vec", [1, 2, 4])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_fused_mean_tile_sizes_and_storage(vec, storage):
    w = W.small(K=5, numels=(3000, 7, 513, 256, 1025, 2), storage=storage, m=1, T=5)
    assert run_parity(w, tuning=dict(vec=vec), fused_mean=True) == 0


def test_fused_mean_bf16_two_passes_heavy_ball():
    w = W.small(K=40, numels=(2048, 12, 999), storage="bf16", m=3, T=6, nesterov=False)
    assert run_parity(w, fused_mean=True, tuning=dict(nontemporal=3)) == 0


def test_fused_mean_grid_cap_and_same_stream():
    w = W.small(K=8, numels=(20000, 33, 4096), m=1, T=4)
    assert run_parity(w, tuning=dict(max_blocks=3), fused_mean=True, side_stream=False) == 0


def test_fused_mean_mobilenet_list_every_step():
    # the workload this call is meant for: K = 16, a global update every step (reduced T)
    w = dataclasses.replace(W.config(3), T=2)
    assert run_parity(w, fused_mean=True) == 0


@pytest.mark.parametrize("n", [5000, 650_003])
def test_fused_mean_mixes_with_the_two_stream_calls(n):
    """Cycles alternate between step_merge + average (650,003 elements, a mean of 17 MiB: on
    the side stream; 5000: on the main stream) and the fused call;
    average_done works after either; the protocol errors are the documented ones."""
    from oracle import lasgd_oracle as O32
    from paper_2203_13085_amd.driver import DeviceReplicas
    w = W.small(K=6, numels=(n, 3, 700), m=1, T=8)
    wd = [w.weight_decay] * len(w.numels)
    x0, grads = packed_inputs(w)
    orc = O32.Oracle(w.K, w.numels, w.momentum, w.nesterov, wd)
    dev = DeviceReplicas(w, weight_decay=wd, side_stream=True)
    c = dev.ctx
    try:
        c.set_tuning(avg_split=1)
        orc.set_model(x0); dev.load_model(x0)
        dev.load_grads(grads(0))
        c.local_step(w.lr)
        with pytest.raises(B.LasgdError) as e:           # nothing sent, no mean pending
            c.step_merge_average(w.lr)
        assert e.value.status == B.ERR_STATE
        c.snapshot(); c.average()
        orc.prologue(grads(0), w.lr)
        compare_state(dev, orc, 0)
        for i in range(1, w.T + 1):
            g = grads(i)
            dev.load_grads(g)
            orc.iteration(g, w.lr, 1)
            if i % 2:
                c.step_merge_average(w.lr)
            else:
                c.step_merge(w.lr, True); c.average()
            c.sync()
            assert c.average_done()
            with pytest.raises(B.LasgdError) as e:       # a mean is pending: s may not be overwritten
                c.snapshot()
            assert e.value.status == B.ERR_STATE
            compare_state(dev, orc, i)
        # partly merged pending mean: the fused call must refuse
        c.merge_ex(0b000111, True)
        with pytest.raises(B.LasgdError) as e:
            c.step_merge_average(w.lr)
        assert e.value.status == B.ERR_STATE
        c.merge_ex(0b111000, True)
        c.average()
        c.set_elastic(0.5, 1.0)
        with pytest.raises(B.LasgdError) as e:
            c.step_merge_average(w.lr)
        assert e.value.status == B.ERR_STATE
    finally:
        dev.close()


def _graph_replay_equals_eager(w, m, tuning=None):
    """m-1 local steps + the fused call captured as one graph and replayed several times, with
    eager library work and host synchronisation between the replays: every replay must give the
    oracle's state (z included: the graph writes it in place)."""
    import torch
    from oracle import lasgd_oracle as O32
    from paper_2203_13085_amd.driver import DeviceReplicas
    x0, grads = packed_inputs(w)
    wd = [w.weight_decay] * len(w.numels)
    dev = DeviceReplicas(w, weight_decay=wd)
    o = O32.Oracle(w.K, w.numels, w.momentum, w.nesterov, wd)
    try:
        if tuning:
            dev.ctx.set_tuning(**tuning)
        g = grads(1)
        o.set_model(x0); dev.load_model(x0); dev.load_grads(g)
        o.prologue(g, w.lr); dev.prologue(w.lr)
        # one eager cycle through the fused call: from here on z is made on the main stream
        for _ in range(m):
            o.iteration(g, w.lr, m)
        for _ in range(m - 1):
            dev.ctx.local_step(w.lr)
        dev.ctx.step_merge_average(w.lr)
        graph = dev.capture_fused_cycle(w.lr, m)
        with pytest.raises(B.LasgdError) as e:           # recorded, not launched: nothing to poll
            dev.ctx.average_done()
        assert e.value.status == B.ERR_STATE
        for rep in range(5):
            with torch.cuda.stream(dev.main):
                graph.replay()
            for _ in range(m):
                o.iteration(g, w.lr, m)
            compare_state(dev, o, rep)
            if rep % 2 == 0:                             # an eager cycle in between, two-stream calls
                for _ in range(m - 1):
                    dev.ctx.local_step(w.lr)
                dev.ctx.step_merge(w.lr, True)
                dev.ctx.average()
                for _ in range(m):
                    o.iteration(g, w.lr, m)
                dev.ctx.sync()
                assert dev.ctx.average_done()
                # back to "z made on the main stream" before the next replay
                for _ in range(m - 1):
                    dev.ctx.local_step(w.lr)
                dev.ctx.step_merge_average(w.lr)
                for _ in range(m):
                    o.iteration(g, w.lr, m)
        with torch.cuda.stream(dev.main):                # back to back, no host synchronisation
            graph.replay()
            graph.replay()
        for _ in range(2 * m):
            o.iteration(g, w.lr, m)
        compare_state(dev, o, 99)
    finally:
        dev.close()


@pytest.mark.parametrize("m", [1, 3])
def test_fused_mean_graph_replay_equals_eager(m):
    _graph_replay_equals_eager(W.small(K=4, numels=(70000, 5, 1024, 4099), m=m), m)


@pytest.mark.parametrize("K", [12, 13])
def test_streaming_fused_call_replays_from_a_graph(K):
    """The streaming forms under capture: one kernel with staged loads, and from K = 13 on update + in-order mean, two
    nodes of the graph.  The split mean of the eager cycles in between is set to one part, so that z is bit-exact."""
    _graph_replay_equals_eager(W.small(K=K, numels=(9000, 5, 1024, 513), m=2), 2, tuning=dict(nontemporal=3, avg_split=1))


@pytest.mark.parametrize("storage,K", [("f32", 1), ("f32", 3), ("f32", 8), ("bf16", 16), ("f32", 17), ("bf16", 33),
                                       ("f32", 64)])
def test_sgd_ar_every_group_shape(storage, K):
    from oracle import lasgd_oracle as O32
    from paper_2203_13085_amd.driver import DeviceReplicas
    w = W.small(K=K, numels=(1030, 1, 4, 257, 768), storage=storage)
    wd = [1e-3, 0.0, 1e-2, 1e-4, 0.0]
    x0, grads = packed_inputs(w)
    orc = O32.Oracle(K, w.numels, w.momentum, w.nesterov, wd, storage=storage)
    dev = DeviceReplicas(w, weight_decay=wd)
    try:
        say(f"[sgd-ar] K={K} storage={storage}")
        orc.set_model(x0); dev.load_model(x0)
        for i in range(4):
            g = grads(i)
            dev.load_grads(g)
            orc.sgd_ar_step(g, w.lr)
            dev.ctx.sgd_ar_step(w.lr)
            for k in range(K):
                assert_close(dev.ctx.read_state(B.STATE_X, k), orc.x[k], f"x step {i} replica {k}")
                assert_close(dev.ctx.read_state(B.STATE_V, k), orc.v[k], f"v step {i} replica {k}")
                if storage == "bf16":
                    np.testing.assert_array_equal(dev.params(k), orc.x16[k])
    finally:
        dev.close()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("K", [4, 9, 11, 12, 13, 25])
def test_streaming_shapes_of_the_group_calls(K, storage):
    """The shapes taken once the state no longer fits the memory-side cache (here asked for by the streaming hint):
    one or two replicas a wave, paced workgroups, and from K = 13 on update + in-order mean.  z stays bit-exact.
    From K = 16 on the first of the two SGD-AR steps is one kernel and the second two."""
    w = W.small(K=K, numels=(1030, 1, 4, 257, 768, 2051), storage=storage, m=1, T=4)
    assert run_parity(w, tuning=dict(nontemporal=3), fused_mean=True) == 0
    from oracle import lasgd_oracle as O32
    from paper_2203_13085_amd.driver import DeviceReplicas
    x0, grads = packed_inputs(w)
    wd = [w.weight_decay] * len(w.numels)
    orc = O32.Oracle(K, w.numels, w.momentum, w.nesterov, wd, storage=storage)
    dev = DeviceReplicas(w, weight_decay=wd)
    try:
        dev.ctx.set_tuning(nontemporal=3)
        orc.set_model(x0); dev.load_model(x0)
        for i in range(2):
            g = grads(i)
            dev.load_grads(g)
            orc.sgd_ar_step(g, w.lr)
            dev.ctx.sgd_ar_step(w.lr)
        for k in range(K):
            assert_close(dev.ctx.read_state(B.STATE_X, k), orc.x[k], f"x replica {k}")
            assert_close(dev.ctx.read_state(B.STATE_V, k), orc.v[k], f"v replica {k}")
    finally:
        dev.close()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("K", [1, 8, 10, 14, 15, 16, 24])
def test_streaming_shapes_at_the_rules_edges(K, storage):
    """Both sides of each line of the shape rules that the test above leaves out."""
    test_streaming_shapes_of_the_group_calls(K, storage)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("K", [16, 17, 24, 25, 33])
def test_streaming_sgd_ar_in_one_kernel_with_many_replicas(K, storage):
    """What every call takes where there is no memory for the mean gradient's array: one replica a wave at K = 16, two up to 24,
    then four, and several passes.  Tiles of 512 elements take it too, and go by the same rule."""
    from oracle import lasgd_oracle as O32
    from paper_2203_13085_amd.driver import DeviceReplicas
    w = W.small(K=K, numels=(1030, 1, 4, 257, 768, 2051), storage=storage)
    x0, grads = packed_inputs(w)
    orc = O32.Oracle(K, w.numels, w.momentum, w.nesterov, [w.weight_decay] * len(w.numels), storage=storage)
    dev = DeviceReplicas(w, weight_decay=[w.weight_decay] * len(w.numels))
    try:
        dev.ctx.set_tuning(nontemporal=3, vec=2)
        orc.set_model(x0); dev.load_model(x0)
        for i in range(3):
            g = grads(i)
            dev.load_grads(g)
            orc.sgd_ar_step(g, w.lr)
            dev.ctx.sgd_ar_step(w.lr)
        for k in range(K):
            assert_close(dev.ctx.read_state(B.STATE_X, k), orc.x[k], f"x replica {k}")
            assert_close(dev.ctx.read_state(B.STATE_V, k), orc.v[k], f"v replica {k}")
    finally:
        dev.close()


@pytest.mark.parametrize("storage,K,R,hint", [("bf16", 40, 1, 3), ("f32", 40, 2, 3), ("bf16", 33, 1, 4), ("f32", 64, 2, 4),
                                              ("f32", 17, 4, 3), ("f32", 12, 1, 3)])
def test_replicas_a_wave_as_asked_for(storage, K, R, hint):
    """group_r: one kernel whatever K, and a second and third pass of a wave where K exceeds 16 R."""
    w = W.small(K=K, numels=(2048, 12, 999, 1, 514), storage=storage, m=2, T=4, nesterov=False)
    assert run_parity(w, fused_mean=True, tuning=dict(nontemporal=hint, group_r=R)) == 0
    from oracle import lasgd_oracle as O32
    from paper_2203_13085_amd.driver import DeviceReplicas
    x0, grads = packed_inputs(w)
    wd = [w.weight_decay] * len(w.numels)
    orc = O32.Oracle(K, w.numels, w.momentum, w.nesterov, wd, storage=storage)
    dev = DeviceReplicas(w, weight_decay=wd)
    try:
        dev.ctx.set_tuning(nontemporal=hint, group_r=R)
        orc.set_model(x0); dev.load_model(x0)
        for i in range(3):
            g = grads(i)
            dev.load_grads(g)
            orc.sgd_ar_step(g, w.lr)
            dev.ctx.sgd_ar_step(w.lr)
        for k in range(K):
            assert_close(dev.ctx.read_state(B.STATE_X, k), orc.x[k], f"x replica {k}")
            assert_close(dev.ctx.read_state(B.STATE_V, k), orc.v[k], f"v replica {k}")
            if storage == "bf16":
                np.testing.assert_array_equal(dev.params(k), orc.x16[k])
    finally:
        dev.close()


@pytest.mark.parametrize("K", [3, 4, 8, 16])
def test_sgd_ar_in_cache_with_more_waves_than_the_chip_holds(K):
    """Beyond 8192 waves the in-cache shape takes two replicas a wave from K = 4 on; below, one (the list above is small)."""
    from oracle import lasgd_oracle as O32
    from paper_2203_13085_amd.driver import DeviceReplicas
    w = W.small(K=K, numels=(8193 * 256 // K + 3, 5))
    x0, grads = packed_inputs(w)
    wd = [1e-3, 0.0]
    orc = O32.Oracle(K, w.numels, w.momentum, w.nesterov, wd)
    dev = DeviceReplicas(w, weight_decay=wd)
    try:
        orc.set_model(x0); dev.load_model(x0)
        g = grads(0)
        dev.load_grads(g)
        for _ in range(2):
            orc.sgd_ar_step(g, w.lr)
            dev.ctx.sgd_ar_step(w.lr)
        for k in range(K):
            assert_close(dev.ctx.read_state(B.STATE_X, k), orc.x[k], f"x replica {k}")
            assert_close(dev.ctx.read_state(B.STATE_V, k), orc.v[k], f"v replica {k}")
    finally:
        dev.close()

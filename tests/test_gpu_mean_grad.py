"""lasgd_sgd_ar_step in two kernels (the mean gradient, then the step): bit for bit what the oracle's in-order sum gives, over
the replica counts that change a wave's batches of loads, ragged tiles, and replays of graphs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2203_13085_amd import binding as B              # noqa: E402
from paper_2203_13085_amd import workloads as W            # noqa: E402
from tests.parity_util import assert_close                 # noqa: E402
from tests.test_gpu_ext import _pair                       # noqa: E402

pytestmark = pytest.mark.gpu


def _same(dev, orc, what):
    for k in range(dev.w.K):
        assert_close(dev.ctx.read_state(B.STATE_X, k), orc.x[k], f"x replica {k} {what}")
        assert_close(dev.ctx.read_state(B.STATE_V, k), orc.v[k], f"v replica {k} {what}")
        if dev.w.storage == "bf16":
            np.testing.assert_array_equal(dev.params(k), orc.x16[k])


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("K", [15, 16, 17, 23, 28, 30, 64])
@pytest.mark.parametrize("blocks", [-1, 3])
def test_batches_and_ragged_tiles(K, storage, blocks):
    """K = 15 is the one kernel; from 16 on batches of eight, four, two and one replicas' rows."""
    w = W.small(K=K, numels=(1030, 1, 4, 257, 768, 2), storage=storage)
    orc, dev, grads = _pair(w, wd=[1e-3, 0.0, 1e-2, 1e-4, 0.0, 0.0])
    try:
        dev.ctx.set_tuning(nontemporal=3, max_blocks=blocks)
        for i in range(3):
            g = grads(i)
            dev.load_grads(g)
            orc.sgd_ar_step(g, w.lr)
            dev.ctx.sgd_ar_step(w.lr)
            _same(dev, orc, f"step {i}")
    finally:
        dev.close()


@pytest.mark.parametrize("storage,K,n", [("f32", 8, 3_670_017), ("f32", 8, 3_669_000), ("bf16", 8, 3_670_017), ("bf16", 12, 1_223_400),
                                         ("f32", 12, 1_223_400), ("f32", 12, 1_222_001), ("f32", 7, 4_194_305)])
def test_both_sides_of_the_line_of_few_replicas(storage, K, n):
    """56 and 112 MiB an array, from which on twelve and eight replicas take two kernels."""
    w = W.small(K=K, numels=(n, 3), storage=storage)
    orc, dev, grads = _pair(w)
    try:
        g = grads(0)
        dev.load_grads(g)
        for _ in range(2):
            orc.sgd_ar_step(g, w.lr)
            dev.ctx.sgd_ar_step(w.lr)
        _same(dev, orc, "")
    finally:
        dev.close()


def test_graph_replays_mix_with_calls():
    w = W.small(K=18, numels=(1030, 257, 3))
    orc, dev, grads = _pair(w)
    try:
        dev.ctx.set_tuning(nontemporal=3)
        g = grads(0)
        dev.load_grads(g)
        graph = torch.cuda.CUDAGraph()
        dev.ctx.sync()
        with torch.cuda.graph(graph, stream=dev.main):
            dev.ctx.sgd_ar_step(w.lr)
        for rep in range(4):
            with torch.cuda.stream(dev.main):
                graph.replay()
            orc.sgd_ar_step(g, w.lr)
            _same(dev, orc, f"replay {rep}")
            dev.ctx.sgd_ar_step(w.lr)
            orc.sgd_ar_step(g, w.lr)
        _same(dev, orc, "at the end")
    finally:
        dev.close()


@pytest.mark.parametrize("K,n,growth", [(16, 1 << 22, 1),        # 256 MiB an array: two kernels
                                        (7, 1 << 23, 0),         # 224 MiB, too few replicas: always one
                                        (32, 1 << 17, 0)])       # 16 MiB: below the hint's size
def test_memory_is_for_callers_of_the_call(K, n, growth):
    """A context holds v, s and z; the array for the mean gradient comes with the first call that takes two kernels, once."""
    x, g = (torch.zeros(K, n, device="cuda") for _ in range(2))
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        torch.zeros(8, device="cuda").add_(1.0)              # a stream's first launch creates its queue
    torch.cuda.synchronize()

    def used():
        torch.cuda.synchronize()
        free, total = torch.cuda.mem_get_info()
        return total - free

    def made():
        return B.Context(K, [n], storage=B.F32, momentum=0.9, nesterov=True, wd_scalar=0.0, main_stream=st.cuda_stream, side_stream=st.cuda_stream)

    made().close()                                           # whatever the runtime sets up with a first context
    u0 = used()
    c = made()
    try:
        row = (n + 256) * 4
        assert used() - u0 <= (2 * K + 1) * row + (6 << 20)              # pages and tables: a few MiB
        for k in range(K):
            c.bind(k, [x[k].data_ptr()], [g[k].data_ptr()])
        u1 = used()
        c.sgd_ar_step(0.1)
        assert growth * n * 4 <= used() - u1 <= growth * (row + (2 << 20))
        u2 = used()
        for _ in range(3):
            c.sgd_ar_step(0.1)
        assert used() == u2
    finally:
        c.close()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_first_call_and_those_after_it(storage):
    """The first call takes one kernel, the others two: the same bits."""
    w = W.small(K=19, numels=(1030, 1, 257, 3), storage=storage)
    orc, dev, grads = _pair(w)
    try:
        dev.ctx.set_tuning(nontemporal=3)
        for i in range(3):
            g = grads(i)
            dev.load_grads(g)
            orc.sgd_ar_step(g, w.lr)
            dev.ctx.sgd_ar_step(w.lr)
            _same(dev, orc, f"call {i}")
    finally:
        dev.close()

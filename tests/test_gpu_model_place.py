"""bf16 storage, from 8 MiB an array on: after a global update that re-sends, the fp32 model is kept once, in s, and the next
call that needs it reads it there.  Whatever calls follow one another, and whatever graphs are recorded and replayed between them, the state has to be
the oracle's, to the bit."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

from paper_2203_13085_amd import workloads as W            # noqa: E402
from tests.parity_util import compare_state, run_parity    # noqa: E402
from tests.test_gpu_ext import _pair                       # noqa: E402

pytestmark = pytest.mark.gpu


def _calls(orc, c, g, w):
    """The calls by name: each does the same on both sides."""
    full = (1 << w.K) - 1
    lrs = [w.lr * (1 - 0.01 * k) for k in range(w.K)]

    def both(o, d):
        def f(mask=full):
            o(mask)
            d(mask)
        return f

    return {
        "step": both(lambda m: orc.local_step(g, lrs, mask=m), lambda m: c.local_step_ex(lrs, m)),
        "plain_step": both(lambda m: orc.local_step(g, w.lr), lambda m: c.local_step(w.lr)),
        "send": both(lambda m: orc.snapshot(mask=m), lambda m: c.snapshot_ex(m)),
        "mean": both(lambda m: orc.average(mask=m), lambda m: c.average_ex(m)),
        "merge": both(lambda m: orc.merge(True, mask=m), lambda m: c.merge_ex(m, True)),
        "merge_keep": both(lambda m: orc.merge(False, mask=m), lambda m: c.merge_ex(m, False)),
        "update": both(lambda m: (orc.local_step(g, w.lr), orc.merge(True, mask=m)),
                       lambda m: c.step_merge(w.lr, True) if m == full else c.step_merge_ex([w.lr] * w.K, full, m, True)),
        "update_keep": both(lambda m: (orc.local_step(g, w.lr), orc.merge(False)), lambda m: c.step_merge(w.lr, False)),
        "fused": both(lambda m: (orc.local_step(g, w.lr), orc.merge(True), orc.average()), lambda m: c.step_merge_average(w.lr)),
        "sgd_ar": both(lambda m: orc.sgd_ar_step(g, w.lr), lambda m: c.sgd_ar_step(w.lr)),
    }


SEQUENCES = [
    "mean update mean update plain_step mean plain_step update",                 # an update right after an update, and steps between
    "mean merge mean merge plain_step send mean merge_keep plain_step send mean update_keep send mean update",
    "mean update sgd_ar mean merge sgd_ar plain_step send mean update",          # the comparator reads the model too
    "mean fused fused plain_step fused update mean fused merge plain_step",      # one pass after another, and out again
    "mean:odd update:odd step:odd mean:odd merge:odd step:even mean:odd update:odd send:even mean update",   # some in s, some not
    "mean merge:even step:odd merge:odd step:low mean fused step:odd update step:even send",
    "sgd_ar mean:odd update:odd sgd_ar step:low send:even mean merge:even sgd_ar merge:odd sgd_ar sgd_ar",      # the same with some of the models in s
]


SHAPES = [(1, (2_097_001, 3), 4), (5, (700, 3, 256, 420_001), 4), (5, (700, 3, 256, 420_001), 3), (12, (175_003, 64), 3),
          (13, (161_515, 64), 3), (13, (161_515, 64), 4), (4, (523_265, 500), 4),        # the last: one row short of 8 MiB
          (17, (125_003, 64), 3)]        # sgd_ar in two kernels, from a sequence's second one on


@pytest.mark.parametrize("K,numels,hint,sequence", [s + (q,) for s in SHAPES for q in SEQUENCES if s[0] > 1 or ":" not in q])
def test_sequences_of_calls(K, numels, hint, sequence):
    w = W.small(K=K, numels=numels, storage="bf16")
    orc, dev, grads = _pair(w)
    full = (1 << K) - 1
    masks = {"odd": 0xaaaaaaaaaaaaaaaa & full, "even": 0x5555555555555555 & full, "low": 1}
    try:
        dev.ctx.set_tuning(nontemporal=hint, avg_split=1)
        g = grads(0)
        dev.load_grads(g)
        calls = _calls(orc, dev.ctx, g, w)
        calls["plain_step"]()
        calls["send"]()
        for word in sequence.split():
            name, _, mask = word.partition(":")
            calls[name](masks.get(mask, full))
        compare_state(dev, orc, 0)
    finally:
        dev.close()


@pytest.mark.parametrize("first", ["replay", "call"])
@pytest.mark.parametrize("sent", ["all", "some"])
@pytest.mark.parametrize("fused,K,hint", [(False, 5, 4), (True, 5, 4), (True, 13, 3)])
def test_graphs_recorded_while_the_models_are_in_s(fused, K, hint, sent, first):
    """Two graphs, a cycle and a lone local step, recorded when all or some of the models are in s only, then replayed and
    mixed with ordinary calls in either order: a replay has to find the model wherever the last call left it."""
    w = W.small(K=K, numels=(700, 3, 256, 2_100_001 // K), storage="bf16")
    orc, dev, grads = _pair(w)
    full = (1 << w.K) - 1
    try:
        dev.ctx.set_tuning(avg_split=1, nontemporal=hint)
        g = grads(0)
        dev.load_grads(g)
        calls = _calls(orc, dev.ctx, g, w)
        for name in ("plain_step", "send", "mean", "update"):
            calls[name]()
        if fused:
            calls["mean"]()
            calls["fused"]()
        if sent == "some":
            calls["step"](0b00110)
        cycle = dev.capture_fused_cycle(w.lr, 2) if fused else dev.capture_cycle(w.lr, 2)
        step = torch.cuda.CUDAGraph()
        with torch.cuda.graph(step, stream=dev.main):
            dev.ctx.local_step(w.lr)

        def replay(graph):
            with torch.cuda.stream(dev.main):
                graph.replay()
            if graph is step:
                orc.local_step(g, w.lr)
            elif fused:
                orc.local_step(g, w.lr); orc.local_step(g, w.lr); orc.merge(True); orc.average()
            else:
                orc.average(); orc.local_step(g, w.lr); orc.local_step(g, w.lr); orc.merge(True)

        def eager():
            if fused:
                calls["plain_step"]()
                calls["fused"]()
            else:
                calls["mean"]()
                calls["plain_step"]()
                calls["update"]()

        for i, what in enumerate([first, "replay", "call", "step", "replay", "replay", "call", "step", "step", "call", "replay"]):
            eager() if what == "call" else replay(step if what == "step" else cycle)
            if i % 3 == 0:
                compare_state(dev, orc, i)
        compare_state(dev, orc, 99)
    finally:
        dev.close()


@pytest.mark.parametrize("K,n,hint", [(3, 700_001, -1), (17, 125_003, 3)])          # 17: recorded as two kernels
def test_a_model_in_s_is_read_after_recording_before_any_replay(K, n, hint):
    w = W.small(K=K, numels=(n, 3), storage="bf16")
    orc, dev, grads = _pair(w)
    try:
        dev.ctx.set_tuning(nontemporal=hint, avg_split=1)
        g = grads(0)
        dev.load_grads(g)
        calls = _calls(orc, dev.ctx, g, w)
        for name in ("plain_step", "send", "mean", "update"):
            calls[name]()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=dev.main):
            dev.ctx.sgd_ar_step(w.lr)
        compare_state(dev, orc, 0)
        for rep in range(3):
            with torch.cuda.stream(dev.main):
                graph.replay()
            orc.sgd_ar_step(g, w.lr)
            compare_state(dev, orc, rep + 1)
    finally:
        dev.close()


@pytest.mark.parametrize("m", [1, 2])
@pytest.mark.parametrize("K", [6, 7, 9, 12, 13, 18, 19, 24, 25])
def test_streaming_fused_update_at_the_rules_edges(K, m):
    """One replica a wave, two, the gradients at once or later, and two kernels from K = 25 on; with every model in s (m = 1) and
    with a step between.  z is the in-order mean to the bit."""
    w = W.small(K=K, numels=(1030, 1, 257, 2_097_152 // K + 77), storage="bf16", m=m, T=2 * m + 1)
    assert run_parity(w, tuning=dict(nontemporal=3), fused_mean=True) == 0


@pytest.mark.parametrize("K,R,hint", [(40, 1, 3), (40, 2, 4), (64, -1, 4), (33, -1, 3), (17, 4, 3)])
def test_fused_update_in_several_passes(K, R, hint):
    """A wave's second and third turn, replicas that do not fill the last one, and four replicas a wave, with every model in s."""
    w = W.small(K=K, numels=(1030, 1, 257, 2_097_152 // K + 77), storage="bf16", m=1, T=3)
    assert run_parity(w, tuning=dict(nontemporal=hint, group_r=R), fused_mean=True) == 0


class _Graph:
    """A recorded graph by the runtime's own calls, which tell how many nodes it has."""

    hip = ctypes.CDLL("libamdhip64.so")

    def __init__(self, stream, record):
        self.stream, self.graph, self.run, n = stream, ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_size_t()
        torch.cuda.synchronize()
        self._do("hipStreamBeginCapture", ctypes.c_void_p(stream.cuda_stream), 2)          # relaxed
        try:
            record()
        finally:
            self._do("hipStreamEndCapture", ctypes.c_void_p(stream.cuda_stream), ctypes.byref(self.graph))
        self._do("hipGraphGetNodes", self.graph, None, ctypes.byref(n))
        self.nodes = n.value
        self._do("hipGraphInstantiate", ctypes.byref(self.run), self.graph, None, None, ctypes.c_size_t(0))

    def _do(self, name, *args):
        st = getattr(self.hip, name)(*args)
        assert st == 0, (name, st)

    def replay(self):
        self._do("hipGraphLaunch", self.run, ctypes.c_void_p(self.stream.cuda_stream))

    def close(self):
        torch.cuda.synchronize()
        self._do("hipGraphExecDestroy", self.run)
        self._do("hipGraphDestroy", self.graph)


class _Nobody:
    def __getattr__(self, name):
        return lambda *a, **k: None


# what is recorded -> how many kernels that is, and how many with one that copies the models back in front
RECORDED = {"plain_step": (1, 0), "step:odd": (1, 1), "step": (1, 0), "sgd_ar": (1, 0), "mean update": (2, 0), "mean merge plain_step": (3, 0),
            "send mean merge": (3, 0), "send:even mean:even update:even": (3, 0), "step:odd plain_step": (2, 1), "fused": (1, 0)}


@pytest.mark.parametrize("shape", [dict(), dict(waves_per_block=4, max_blocks=37, kper_step=3, kper_merge=5), dict(vec=4), dict(vec=2, group_r=2)])
@pytest.mark.parametrize("what", list(RECORDED))
def test_a_recorded_graph_holds_its_own_kernels_alone(what, shape):
    """Recorded while the models are in s, and the same once more; replayed second one first, then with calls between.  The first kernel
    of the first replay brings the models back, without a kernel of its own, wherever that first kernel writes all of them."""
    K = 5
    w = W.small(K=K, numels=(700, 3, 256, 420_001), storage="bf16")
    orc, dev, grads = _pair(w)
    full = (1 << K) - 1
    masks = {"odd": 0b01010, "even": 0b10101}
    graphs = []
    try:
        dev.ctx.set_tuning(avg_split=1, **shape)
        g = grads(0)
        dev.load_grads(g)
        both, oracle, device = _calls(orc, dev.ctx, g, w), _calls(orc, _Nobody(), g, w), _calls(_Nobody(), dev.ctx, g, w)

        def do(calls, words):
            for word in words.split():
                name, _, mask = word.partition(":")
                calls[name](masks.get(mask, full))
        do(both, "plain_step send mean update" + (" mean" if what == "fused" else ""))
        graphs = [_Graph(dev.main, lambda: do(device, what)) for _ in range(2)]
        kernels, copies = RECORDED[what]
        assert [x.nodes for x in graphs] == [kernels + copies, kernels + copies]
        for i, which in enumerate([1, 0, 0, 1]):
            graphs[which].replay()
            do(oracle, what)
            compare_state(dev, orc, i)
        for i in range(2):
            do(both, "plain_step " + what)
            graphs[i].replay()
            do(oracle, what)
            compare_state(dev, orc, 10 + i)
    finally:
        for x in graphs:
            x.close()
        dev.close()


def test_a_recorded_mean_gradient_and_its_step_bring_the_models_back():
    """Two kernels are recorded, the second of which reads the models in s: no third that copies them.  The graph recorded last is
    replayed first."""
    w = W.small(K=17, numels=(125_003, 64), storage="bf16")
    orc, dev, grads = _pair(w)
    graphs = []
    try:
        dev.ctx.set_tuning(nontemporal=3, avg_split=1)
        g = grads(0)
        dev.load_grads(g)
        calls = _calls(orc, dev.ctx, g, w)
        for name in ("plain_step", "send", "mean", "update"):
            calls[name]()
        calls["step"](0b10010)
        graphs = [_Graph(dev.main, lambda: dev.ctx.sgd_ar_step(w.lr)) for _ in range(2)]
        assert [x.nodes for x in graphs] == [2, 2]
        for i, which in enumerate([1, 0, 1]):
            graphs[which].replay()
            orc.sgd_ar_step(g, w.lr)
            compare_state(dev, orc, i)
            calls["sgd_ar"]()
        compare_state(dev, orc, 99)
    finally:
        for x in graphs:
            x.close()
        dev.close()


@pytest.mark.parametrize("what", ["plain_step", "fused", "mean update"])
def test_a_call_before_the_first_replay_of_such_a_graph(what):
    """The call brings the models back; the graph's first kernel finds them in the master copies then, whatever was in s."""
    w = W.small(K=4, numels=(700, 3, 523_000), storage="bf16")
    orc, dev, grads = _pair(w)
    graph = None
    try:
        dev.ctx.set_tuning(avg_split=1)
        g = grads(0)
        dev.load_grads(g)
        both, oracle, device = _calls(orc, dev.ctx, g, w), _calls(orc, _Nobody(), g, w), _calls(_Nobody(), dev.ctx, g, w)
        for name in ("plain_step", "send", "mean", "update") + (("mean",) if what == "fused" else ()):
            both[name]()
        graph = _Graph(dev.main, lambda: [device[n]() for n in what.split()])
        both["plain_step"]()
        both["plain_step"]()
        for i in range(3):
            graph.replay()
            for n in what.split():
                oracle[n]()
            compare_state(dev, orc, i)
    finally:
        if graph:
            graph.close()
        dev.close()

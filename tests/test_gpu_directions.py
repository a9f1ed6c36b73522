"""Arrays of 8 to 64 MiB: every other launch takes its items from the last to the first, rows of items are padded to the eight
XCDs, and a replica's arrays are kept from lying a round number apart.  Tile counts that leave every kind of remainder, more
than one chunk of tiles, masks, both call families and all group calls: the oracle's state to the bit, whichever way the launches ran."""
import pytest

torch = pytest.importorskip("torch")

from paper_2203_13085_amd import workloads as W            # noqa: E402
from tests.parity_util import compare_state                # noqa: E402
from tests.test_gpu_ext import _pair                       # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("K,numels,blocks", [(3, (699_136, 1, 300), -1),        # 2731 + 1 + 2 tiles: remainder 6
                                             (3, (700_416,), -1),               # 2736 tiles: no remainder
                                             (3, (700_417, 255), -1),           # 2738 tiles
                                             (2, (1 << 20,), -1),               # replicas 4 MiB apart, but for one row
                                             (1, (2_100_001, 2_049), -1),       # more than one chunk of 8192 tiles
                                             (3, (699_136, 1, 300), 37),        # a capped grid
                                             (3, (670_000,), -1)])              # below 8 MiB: forward only
def test_both_directions(K, numels, blocks, storage):
    w = W.small(K=K, numels=numels, storage=storage)
    orc, dev, grads = _pair(w)
    c, full = dev.ctx, (1 << K) - 1
    try:
        c.set_tuning(avg_split=1, max_blocks=blocks)
        g = grads(0)
        dev.load_grads(g)
        orc.local_step(g, w.lr); c.local_step(w.lr)
        orc.snapshot(); c.snapshot()
        for m in (1, 2, 2):
            orc.average(); c.average()
            for _ in range(m - 1):
                orc.local_step(g, w.lr); c.local_step(w.lr)
            orc.local_step(g, w.lr); orc.merge(True); c.step_merge(w.lr, True)
        compare_state(dev, orc, 0)
        orc.sgd_ar_step(g, w.lr); c.sgd_ar_step(w.lr)
        orc.average(); c.average()
        for m in (1, 2, 3):
            for _ in range(m - 1):
                orc.local_step(g, w.lr); c.local_step(w.lr)
            orc.local_step(g, w.lr); orc.merge(True); orc.average(); c.step_merge_average(w.lr)
        orc.merge(False); c.merge(False)
        compare_state(dev, orc, 1)
        some = full & 0b101
        lrs = [w.lr * (1 - 0.1 * k) for k in range(K)]
        for _ in range(3):
            orc.local_step(g, lrs, mask=some); c.local_step_ex(lrs, some)
            orc.sgd_ar_step(g, w.lr); c.sgd_ar_step(w.lr)
        orc.snapshot(mask=some); c.snapshot_ex(some)
        orc.average(mask=some); c.average_ex(some)
        orc.local_step(g, lrs); orc.merge(True, mask=some); c.step_merge_ex(lrs, full, some, True)
        compare_state(dev, orc, 2)
    finally:
        dev.close()

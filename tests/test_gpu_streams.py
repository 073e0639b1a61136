"""GPU <-> oracle parity over every schedule a gather can take, with victim hits,
and over the changes from one to another: rows so wide that a few dozen misses
exceed what a gather on one stream is expected to fetch, in minibatches that
are mostly resident for a while and then mostly miss.  Each case checks that the
schedules it is for did run.  Every integer and byte output must match exactly
(tests/parity_driver.py).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2407_15264_amd import lsmgnn  # noqa: E402
from paper_2407_15264_amd.workload import CacheShape  # noqa: E402
from tests.parity_driver import (Store, log, run_async_parity, run_mixed_parity, run_parity,  # noqa: E402
                                 run_typed_async_parity)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lsmgnn.lib()


def _stream(n, lines, seed, count=60):
    """Minibatches over n nodes for a cache of `lines` lines: runs of mostly resident ones (a few strays), runs that
    mostly miss, runs of both in turn, and now and then an empty one or a lookup."""
    rng = np.random.default_rng(seed)
    hot = rng.permutation(n)[: lines // 2]
    batches = []
    while len(batches) < count:
        run = rng.integers(0, 3)
        for k in range(int(rng.integers(3, 7))):
            missing = run == 1 or (run == 2 and k % 2)
            if missing:
                ids = rng.integers(0, n, int(rng.integers(150, 400)))
            else:
                ids = np.concatenate([rng.choice(hot, int(rng.integers(100, 1500))), rng.integers(0, n, 4)])
            batches.append(rng.permutation(ids))
        if rng.random() < 0.3:
            batches.append(np.zeros(0, np.int64))
        if rng.random() < 0.3:
            batches.append(rng.choice(hot, 20))
        hot = np.where(rng.random(hot.size) < 0.1, rng.integers(0, n, hot.size), hot)
    return batches[:count]


@pytest.mark.parametrize("mode", ["blocking", "pipelined", "mixed", "pipelined, rejected calls", "mixed, rejected calls"])
@pytest.mark.parametrize("victim", [0, 9, 250])
@pytest.mark.parametrize("row_bytes", [16 << 10, 33_008])
def test_every_schedule(row_bytes, victim, mode):
    log(f"case: every schedule, {row_bytes} B rows, V={victim}, {mode}")
    n, sets = 2500, 60
    batches = _stream(n, 8 * sets, 31 * victim + row_bytes)
    store = Store.random_bytes(n, row_bytes, 8)
    stat = np.random.default_rng(9).integers(0, 9, n).astype(np.uint32)
    rejects = 5 if "rejected" in mode else None
    args = (store, stat, sets, victim, 3, batches)
    if mode == "blocking":
        res = run_parity(*args, rows="all", label=mode, per_gather_stats=False)
    elif mode.startswith("pipelined"):
        res = run_async_parity(*args, rows="all", label=mode, reject_seed=rejects)
    else:
        res = run_mixed_parity(*args, 6, label=mode, reject_seed=rejects)
    ways = res["routes"]
    log(f"  {ways} victim hits {res['total']['victim_hits']}")
    assert 0 < ways["one_block"] < ways["one_stream"] < len(batches) - 10
    if mode != "blocking":
        assert (ways["deferred"] if victim else ways["overlapped"]) > 5
    if victim > 9:
        assert res["total"]["victim_hits"] > 20


def test_every_schedule_of_several_caches():
    """Three caches on one device, which share its streams, two of them without a ring."""
    log("case: several caches, every schedule")
    n, sets = 2500, 60
    stores = [Store.random_bytes(n, rb, 10 + t) for t, rb in enumerate((16 << 10, 20_000, 2048))]
    stats = [np.random.default_rng(20 + t).integers(0, 9, n).astype(np.uint32) for t in range(3)]
    shapes = [CacheShape(sets, v, 3) for v in (0, 250, 0)]
    res = run_typed_async_parity(stores, stats, shapes, [_stream(n, 8 * sets, 40 + t) for t in range(3)], rows="all")
    for t, ways in enumerate(res["routes"]):
        log(f"  type {t}: {ways} victim hits {res['totals'][t]['victim_hits']}")
        assert ways["one_stream"] > 0
    assert res["routes"][0]["overlapped"] > 5 and res["routes"][1]["deferred"] > 5
    assert res["totals"][1]["victim_hits"] > 20

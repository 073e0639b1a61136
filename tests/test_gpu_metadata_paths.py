"""GPU <-> oracle parity at the sizes where the metadata kernels change path:
the number of a batch's IDs in one set (ordered by 8 lanes, by a wave, by a
block), sets that are settled by the probe beside sets that are walked, and
ring sizes on both sides of what one chunk, and a whole batch, enqueues.
Every integer and byte output must match exactly (tests/parity_driver.py).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2407_15264_amd import lsmgnn  # noqa: E402
from tests.parity_driver import Store, log, run_async_parity, run_parity  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lsmgnn.lib()


@pytest.mark.parametrize("policy", ["hybrid", "static", "dynamic", "round_robin"])
@pytest.mark.parametrize("k", [1, 7, 8, 9, 63, 64, 65, 511, 512, 513, 2049])
def test_ids_per_set(k, policy):
    """One set that receives exactly k unique IDs, in shuffled order with repeats."""
    log(f"case: {k} IDs in one set, {policy}")
    n = max(4 * k, 32)
    rng = np.random.default_rng(k)
    batches = []
    for _ in range(5):
        ids = rng.choice(n, k, replace=False)
        batches.append(rng.permutation(np.concatenate([ids, rng.choice(ids, k)])))
    store = Store.random_bytes(n, 32, k)
    stat = rng.integers(0, 6, n).astype(np.uint32)
    run_parity(store, stat, 1, max(1, k // 3), 3, batches, rows="all", label=f"k={k}", policy=policy)


@pytest.mark.parametrize("victim", [0, 40])
@pytest.mark.parametrize("sets", [64, 500])
def test_settled_and_walked_sets(sets, victim):
    """Batches that mostly repeat the one before, so that some touched sets hold all their IDs and others do not."""
    log(f"case: settled and walked sets, S={sets} V={victim}")
    n = sets * 12
    rng = np.random.default_rng(sets + victim)
    ids = rng.choice(n, sets * 4, replace=False)
    batches = []
    for b in range(12):
        batches.append(rng.permutation(ids))
        swap = rng.random(ids.size) < [0.0, 0.02, 0.3][b % 3]
        ids = np.where(swap, rng.integers(0, n, ids.size), ids)
    store = Store.random_bytes(n, 48, 1)
    stat = rng.integers(0, 9, n).astype(np.uint32)
    run_parity(store, stat, sets, victim, 4, batches, rows="all", label="settled")
    run_async_parity(store, stat, sets, victim, 4, batches, rows="all", label="settled pipelined")


@pytest.mark.parametrize("victim", [1, 100, 255, 256, 257, 700, 5000])
def test_ring_liveness_within_a_batch(victim):
    """Lines evicted to the ring and requested again later in the same batch, with rings that the batch's enqueues
    overrun before, at and after that request."""
    log(f"case: same-batch ring liveness, V={victim}")
    n, sets = 6000, 300
    rng = np.random.default_rng(victim)
    batches = [rng.choice(n, 4000) for _ in range(8)]
    store = Store.random_bytes(n, 16, 2)
    stat = rng.integers(0, 3, n).astype(np.uint32)
    run_parity(store, stat, sets, victim, 5, batches, rows="all", label=f"V={victim}")


@pytest.mark.parametrize("requests", [(1 << 20) - 255, (1 << 20) + 1])
def test_enqueue_scan_limit(requests):
    """Request lists on both sides of the size beyond which the chunks' enqueue counts are scanned by their own kernel."""
    log(f"case: {requests} requests")
    n = 700_000
    rng = np.random.default_rng(requests)
    batches = [rng.integers(0, n, requests) for _ in range(3)]
    store = Store.random_bytes(n, 16, 3)
    stat = rng.integers(0, 50, n).astype(np.uint32)
    run_parity(store, stat, 20_000, 30_000, 3, batches, rows="all", label="scan limit")

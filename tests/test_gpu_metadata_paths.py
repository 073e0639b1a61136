"""GPU <-> oracle parity at the sizes where the metadata kernels change path:
the number of a batch's IDs in one set (ordered by 8 lanes, by a wave, by a
block), and sets that are settled by the probe beside sets that are walked.
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

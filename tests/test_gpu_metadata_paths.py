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


@pytest.mark.parametrize("victim", [300, 4000, 20_000])
@pytest.mark.parametrize("nodes", [65_281, 65_536, 65_537, 131_073])
def test_ring_liveness_across_chunks(nodes, victim):
    """The same over hundreds of chunks of enqueue counts, at the sizes where a thread takes one more of them: every
    node in every batch, so that each line evicted before its turn is requested later."""
    log(f"case: same-batch ring liveness, {nodes} unique IDs, V={victim}")
    rng = np.random.default_rng(nodes + victim)
    batches = [rng.permutation(nodes) for _ in range(5)]
    store = Store.random_bytes(nodes, 16, 8)
    stat = rng.integers(0, 3, nodes).astype(np.uint32)
    run_parity(store, stat, nodes // 20, victim, 3, batches, rows="all", label=f"{nodes} IDs, V={victim}")


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


@pytest.mark.parametrize("policy", ["hybrid", "static", "dynamic", "round_robin"])
@pytest.mark.parametrize("victim,lookahead", [(0, 0), (0, 3), (37, 3), (2000, 16)])
@pytest.mark.parametrize("requests", [1, 63, 64, 65, 255, 257, 1023, 1024, 1025])
def test_small_gathers(requests, victim, lookahead, policy):
    """Request counts around those that one block takes, with mostly resident rows (the block's path), then a batch
    that misses everything and mostly resident ones again."""
    log(f"case: {requests} requests, V={victim} L={lookahead} {policy}")
    n, sets = 3 * max(requests, 40), max(requests, 40) // 4
    rng = np.random.default_rng(requests + victim)
    pool = rng.choice(n, max(1, sets * 4), replace=False)
    batches = []
    for b in range(14):
        if b == 7:
            batches.append(rng.integers(0, n, requests))
            pool = rng.choice(n, pool.size, replace=False)
            continue
        ids = rng.choice(pool, requests)
        stray = rng.random(requests) < 0.03
        batches.append(np.where(stray, rng.integers(0, n, requests), ids))
    store = Store.random_bytes(n, 48, 4)
    stat = rng.integers(0, 7, n).astype(np.uint32)
    run_parity(store, stat, sets, victim, lookahead, batches, rows="all", label="small", policy=policy)
    run_async_parity(store, stat, sets, victim, lookahead, batches, rows="all", label="small pipelined", policy=policy)


def test_small_gather_errors():
    """An ID out of range in a small gather's own or announced list leaves everything as it was."""
    log("case: small gather errors")
    n = 500
    store = Store.random_bytes(n, 32, 5)
    cache = lsmgnn.FeatureCache(n, 32, store.buf, np.arange(n, dtype=np.uint32), 80, 20, 2, 200)
    dev = torch.device("cuda")
    good = torch.arange(40, device=dev)
    for _ in range(3):
        cache.advance(good)
    for _ in range(3):
        r = cache.gather(good, outcome=True)
        cache.advance(good)
    before, stats = cache.export_state(), cache.stats()[1]
    out = torch.empty(200 * 32, dtype=torch.uint8, device=dev)
    uniq = torch.empty(200, dtype=torch.int64, device=dev)
    for bad in (n, -1, 1 << 40):
        wrong = good.clone()
        wrong[17] = bad
        with pytest.raises(lsmgnn.LsmgnnError) as e:
            cache.gather(wrong)
        assert e.value.code == lsmgnn.E_RANGE
        with pytest.raises(lsmgnn.LsmgnnError) as e:
            cache.gather_async(good, out, uniq, announce=wrong)
        assert e.value.code == lsmgnn.E_RANGE
        after = cache.export_state()
        for key in before:
            assert np.array_equal(before[key], after[key]), key
        assert cache.stats()[1] == stats
    r = cache.gather(good, outcome=True)
    assert r.n_unique == 40 and bool((r.outcome == lsmgnn.HIT).all())
    assert np.array_equal(r.out.cpu().numpy(), store.np[:40])
    cache.close()


@pytest.mark.parametrize("nodes", [4095, 4096, 4097, (1 << 22) - 1, 1 << 22, (1 << 22) + 1])
def test_dedup_chunks(nodes):
    """Node counts at the edges of the dedup map's chunks, and where the chunk size changes; the top IDs are requested."""
    log(f"case: {nodes} nodes")
    rng = np.random.default_rng(nodes)
    batches = [np.concatenate([rng.integers(0, nodes, 3000), [0, nodes - 1, nodes - 2], rng.integers(0, nodes, 40)])
               for _ in range(4)]
    store = Store.random_bytes(nodes, 16, 6)
    stat = rng.integers(0, 9, nodes).astype(np.uint32)
    run_parity(store, stat, 500, 300, 2, batches, rows="all", label=f"N={nodes}")


@pytest.mark.parametrize("victim", [0, 700])
@pytest.mark.parametrize("row_bytes", [16, 1008, 4096])
def test_more_host_rows_than_expected(row_bytes, victim):
    """Minibatches that miss everything after resident ones: they were expected to fetch little, and their host rows
    take more tiles than one launch has blocks for."""
    log(f"case: more host rows than expected, {row_bytes} B rows, V={victim}")
    n, sets, requests = 40_000, 1500, max(3000, (2 << 20) // row_bytes if row_bytes > 16 else 9000)
    rng = np.random.default_rng(row_bytes + victim)
    pool = rng.choice(n, requests // 2, replace=False)
    batches = []
    for b in range(12):
        if b % 4 == 3:
            batches.append(rng.permutation(n)[:requests])
            pool = rng.choice(n, requests // 2, replace=False)
        else:
            batches.append(rng.choice(pool, requests))
    store = Store.random_bytes(n, row_bytes, 7)
    stat = rng.integers(0, 7, n).astype(np.uint32)
    run_parity(store, stat, sets, victim, 2, batches, rows="all", label="unexpected misses")
    run_async_parity(store, stat, sets, victim, 2, batches, rows="all", label="unexpected misses pipelined")

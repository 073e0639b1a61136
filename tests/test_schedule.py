"""The host runtime's schedule (no GPU): which kernels and copies a call queues,
on which stream and behind what.  runtime.hip is compiled as host code against
tests/schedule/model.cc, which stands in for HIP and the kernels and reports
every pair of conflicting accesses that no stream order, event or host wait puts
in order."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

from paper_2407_15264_amd import build, lsmgnn

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2407_15264_amd", "csrc")
ROCM = os.path.dirname(os.path.dirname(os.path.realpath(shutil.which(build.HIPCC) or build.HIPCC)))
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")

pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="needs ROCm's clang++")

u64, vp = ctypes.c_uint64, ctypes.c_void_p


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("schedule") / "libschedule.so")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-g", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(CSRC, "runtime.hip"), os.path.join(HERE, "schedule", "model.cc"), "-lpthread",
                    "-Wl,-Bsymbolic", "-o", so], check=True, capture_output=True, timeout=300)
    L = ctypes.CDLL(so)
    L.lsmgnn_cache_create.argtypes = [ctypes.POINTER(lsmgnn.Config), ctypes.POINTER(vp)]
    L.lsmgnn_cache_destroy.argtypes = [vp]
    L.lsmgnn_advance.argtypes = [vp, vp, u64, vp]
    L.lsmgnn_gather.argtypes = [vp, vp, u64, vp, vp, vp, vp, ctypes.POINTER(u64), vp]
    L.lsmgnn_gather_async.argtypes = [vp, vp, u64, vp, u64, vp, vp, vp, vp, ctypes.POINTER(u64), ctypes.POINTER(u64),
                                      vp]
    L.lsmgnn_gather_wait.argtypes = [vp, u64, vp]
    L.lsmgnn_sync.argtypes = [vp]
    L.lsmgnn_set_profiling.argtypes = [vp, ctypes.c_int]
    L.model_plan.argtypes = [ctypes.c_uint32] * 4 + [ctypes.c_int]
    L.model_read_outputs.argtypes = [vp] * 4
    for f in (L.model_log, L.model_errors):
        f.restype = ctypes.c_char_p
    return L


class Cache:
    """A cache over the model; every gather gets output addresses of its own."""
    addr = 1 << 50

    def __init__(self, model, row_bytes=4096, victim=0, lookahead=2, max_batch=100_000, queues=False, pageable=False,
                 refresh=1):
        self.L, self.R, self.V, self.max_batch = model, row_bytes, victim, max_batch
        self.store = ctypes.create_string_buffer(64 * row_bytes + 64)
        self.static = (ctypes.c_uint32 * 64)()
        cfg = lsmgnn.Config(64, row_bytes, 100, victim, max_batch, lookahead, 0, 0, 1 if pageable else 0, 1, 0,
                            1 if queues else 0, refresh, (ctypes.addressof(self.store) + 63) // 64 * 64,
                            ctypes.addressof(self.static))
        self.h = vp()
        assert model.lsmgnn_cache_create(ctypes.byref(cfg), ctypes.byref(self.h)) == lsmgnn.OK
        self.t = 0

    def close(self):
        self.L.lsmgnn_cache_destroy(self.h)

    def _addrs(self):
        a = Cache.addr
        Cache.addr += 1 << 20
        return a, a + 65536, a + 2 * 65536, a + 3 * 65536

    def gather(self, n, unique=0, early=0, late=0, enq=0, err=False, pipelined=False, ann=None):
        """Returns (status, ticket, outputs, log of the operations the call queued)."""
        self.L.model_clear_log()
        self.L.model_plan(unique, early, late, enq, int(err))
        outs, nu, ticket = self._addrs(), u64(), u64()
        ids = (1 << 49) if n else None
        if pipelined:
            rc = self.L.lsmgnn_gather_async(self.h, ids, n, (1 << 49) if ann is not None else None, ann or 0, *outs,
                                            ctypes.byref(nu), ctypes.byref(ticket), None)
        else:
            rc = self.L.lsmgnn_gather(self.h, ids, n, *outs, ctypes.byref(nu), None)
        assert rc == (lsmgnn.E_RANGE if err else lsmgnn.OK)
        if rc == lsmgnn.OK:
            assert nu.value == unique
            self.t += 1
        return rc, ticket.value, outs, self.L.model_log().decode().split("\n")[:-1]

    def read(self, outs):
        self.L.model_read_outputs(*outs)


@pytest.fixture
def fresh(model):
    model.model_reset()
    model.model_caller_busy(0)
    return model


def check(model):
    errors = model.model_errors().decode()
    assert not errors, errors[:2000]


KINDS = {"no ring": dict(), "ring": dict(victim=5000), "queues": dict(victim=3000, queues=True),
         "pageable": dict(victim=5000, pageable=True, max_batch=3000, row_bytes=64)}


def random_calls(caches, rng, steps):
    """Blocking, pipelined, small, large, empty and rejected gathers, announcements, waits and syncs in any order."""
    pending = {c: [] for c in caches}
    for _ in range(steps):
        c = rng.choice(caches)
        waiting = pending[c]
        c.L.model_caller_busy(rng.randint(0, 1))
        kind = rng.random()
        if kind < 0.1:
            c.L.lsmgnn_advance(c.h, 1 << 49, 10, None)
        elif kind < 0.2 and waiting:
            ticket, outs = waiting.pop(rng.randrange(len(waiting)))
            assert c.L.lsmgnn_gather_wait(c.h, ticket, None) == lsmgnn.OK
            c.read(outs)
        elif kind < 0.25:
            assert c.L.lsmgnn_sync(c.h) == lsmgnn.OK
            for _, outs in waiting:
                c.read(outs)
            waiting.clear()
        else:
            n = rng.choice([0, 1, 250, 1024, 1025, 3000] + ([60_000] if c.max_batch > 60_000 else []))
            unique = n and rng.randint(1, n)
            miss = rng.choice([0, 1, min(unique, 120), unique // 2, unique])
            miss = min(miss, unique)
            early = rng.randint(0, miss)
            err = n > 0 and rng.random() < 0.2
            pipelined = rng.random() < 0.6
            enq = rng.choice([0, min(miss, 600)]) if c.V else 0
            rc, ticket, outs, _ = c.gather(n, unique, early, miss - early, enq, err, pipelined,
                                           ann=rng.choice([None, 0, 100]) if pipelined else None)
            if rc == lsmgnn.OK:
                if pipelined:
                    waiting.append((ticket, outs))
                else:
                    c.read(outs)


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("seed", range(8))
def test_no_unordered_accesses(fresh, kind, seed):
    c = Cache(fresh, **KINDS[kind])
    random_calls([c], random.Random(seed), 200)
    c.close()
    check(fresh)


@pytest.mark.parametrize("seed", range(8))
def test_no_unordered_accesses_between_caches(fresh, seed):
    """Several caches, which share their device's streams: with and without a ring, one with queues."""
    caches = [Cache(fresh, **KINDS[k]) for k in ("no ring", "ring", "no ring", "queues")]
    random_calls(caches, random.Random(seed), 400)
    for c in caches:
        c.close()
    check(fresh)


def test_retry_of_a_rejected_pipelined_gather(fresh):
    """A rejected gather's host fetch reads its gate; the retry, which resets the same gate, comes behind it."""
    c = Cache(fresh, victim=5000)
    for _ in range(3):
        c.gather(60_000, 50_000, 20_000, 5000, 3000, pipelined=True)
    c.gather(60_000, err=True, pipelined=True)
    c.gather(60_000, 50_000, 20_000, 5000, 3000, pipelined=True)
    c.close()
    check(fresh)


def moved(log):
    """How a gather's rows moved: by one launch on the meta stream, or over the three streams."""
    names = {line.split(" ")[-1] for line in log}
    assert ("move_rows@meta" in names) != ("host_late@host" in names), log
    return "one" if "move_rows@meta" in names else "three"


def tiny(log):
    return any(line.endswith("tiny@meta") for line in log)


def test_streams_of_a_steady_gather(fresh):
    """Up to 1 MiB expected over the link: one stream; above it, three.  Lists of about the same length scale."""
    rows = (1 << 20) // 4096
    c = Cache(fresh)
    assert moved(c.gather(1000, 900, 900)[3]) == "three"  # nothing known: every request may miss
    for n, host, want in [(1000, rows, "three"), (1000, rows, "three"), (1000, rows + 1, "one"), (1000, 0, "three"),
                          (1000, 0, "three"), (1000, 0, "one"), (4000, 0, "one"), (16003, 0, "one"),
                          (70_000, 0, "three")]:
        assert moved(c.gather(n, min(n, 900), host)[3]) == want, (n, host)
    c.close()
    check(fresh)


def test_an_empty_gather_predicts_nothing(fresh):
    c = Cache(fresh, victim=5000)
    for _ in range(3):
        c.gather(60_000, 50_000, 30_000, enq=100)
        c.gather(0)
        assert moved(c.gather(60_000, 50_000, 30_000, enq=100, pipelined=True)[3]) == "three"
        c.gather(0, pipelined=True)
    c.close()
    c = Cache(fresh, row_bytes=16)
    for _ in range(3):
        c.gather(1000, 900, 900)
        c.gather(0)
        log = c.gather(1000, 900, 900)[3]
        assert moved(log) == "one" and not tiny(log)
    c.close()
    check(fresh)


@pytest.mark.parametrize("pipelined", [False, True])
def test_a_lookup_predicts_no_large_gather(fresh, pipelined):
    c = Cache(fresh, row_bytes=1024)
    for _ in range(3):
        for _ in range(3):
            log = c.gather(250, 200, 0)[3]
        assert tiny(log)
        assert moved(c.gather(60_000, 50_000, 30_000, pipelined=pipelined)[3]) == "three"
    c.close()
    check(fresh)


def test_alternating_minibatches_take_three_streams(fresh):
    """Resident and missing minibatches in turn: the missing ones are never taken for resident ones."""
    c = Cache(fresh)
    for k in range(12):
        log = c.gather(5000, 4000, 3000 if k % 2 else 0, pipelined=k % 3 == 0)[3]
        assert moved(log) == "three", k
    c.close()
    check(fresh)

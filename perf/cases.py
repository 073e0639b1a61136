"""The work whose speed this repository looks after, as calls of its public
entry points: feature gathers through the cache (blocking and pipelined; small,
ordinary and large minibatches; a backing store that mostly hits, mostly
misses, is pageable; the victim ring and the per-iteration queues), the GPU
sampler, the split of a request list by node type, rows in request order, and
the reverse-PageRank static score.

Shapes follow the workloads of paper_2407_15264_amd/workload (row widths,
fanouts, seeds per minibatch, lookaheads, cache and ring shares); graphs are
R-MAT with the same (a, b, c, d), generated here on the GPU from the seed, with
fewer nodes where the feature store of the full shape would take minutes to
write.
"""
import functools

import numpy as np
import torch

from paper_2407_15264_amd import lsmgnn

DEV = torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")


# ------------------------------------------------------------------- cases
def _gather(name, nodes, edges, vectors, requests, seeds, fanout, sets, victim, lookahead, mode, minibatches, lists,
            **more):
    """vectors: 16-byte vectors per feature row; requests: length of every
    minibatch's request list, sampled from `seeds` seed nodes at a time; mode:
    "blocking" (one lsmgnn_gather, then lsmgnn_advance, a pass) or "pipelined"
    (`minibatches` lsmgnn_gather_async calls with their announcements, two in
    flight, a pass); lists: distinct minibatches the stream cycles through."""
    c = dict(name=name, kind="gather", nodes=nodes, edges=edges, vectors=vectors, requests=requests, seeds=seeds,
             fanout=fanout, sets=sets, victim=victim, lookahead=lookahead, mode=mode, minibatches=minibatches, lists=lists,
             policy="hybrid", victim_mode="fifo", refresh=1, pageable=False, resident=False)
    c.update(more)
    return c


def listed():
    return [
        # Serving: the neighbourhood of a few nodes looked up in a cache that
        # holds the whole feature table.  Only latency counts.
        _gather("lookup", 1 << 20, 1 << 22, 32, 250, 8, "10,5", 1 << 18, 0, 0, "blocking", 1, 16, resident=True),
        # The smallest training workload (2^14 nodes, fp32 x 128, 256 seeds,
        # ring, lookahead 2), one minibatch at a time.
        _gather("small blocking", 1 << 14, 1 << 18, 32, 9001, 256, "10,5", 2048, 1024, 2, "blocking", 1, 16),
        # The 1M-node training workload (fp32 x 256, cache of 10 % and ring of
        # 5 % of the nodes, lookahead 4), one minibatch at a time ...
        _gather("1M nodes blocking", 1 << 20, 1 << 24, 64, 123_457, 1024, "15,10,5", 13107, 52428, 4, "blocking", 1, 16),
        # ... and as the pipelined loop of a training run.
        _gather("1M nodes pipelined", 1 << 20, 1 << 24, 64, 123_457, 1024, "15,10,5", 13107, 52428, 4, "pipelined", 8, 16),
        # Large minibatches of fp16 x 1024 rows from a cache that holds the
        # whole table (288 GB of HBM hold many graphs' features): HBM-bound.
        _gather("resident pipelined", 1 << 21, 1 << 25, 128, 900_000, 8192, "15,10,5", 1 << 19, 0, 4, "pipelined", 4,
                8, resident=True),
        # fp16 x 1024 rows in ordinary host memory, copied by the library's
        # host threads; lookahead 16, about four of five rows hit.
        _gather("pageable pipelined", 1 << 19, 1 << 23, 128, 100_000, 1024, "15,10,5", 16384, 16384, 16, "pipelined", 4, 24,
                pageable=True),
        # The paper's own victim-buffer form (queues with prefetch) and update
        # period 4, fp32 x 768 rows (not a power of two), no pipelining.
        _gather("queues blocking", 300_000, 4_000_000, 192, 40_000, 512, "10,5,5", 5000, 15_000, 8, "blocking", 1, 16,
                victim_mode="queues", refresh=4),
        # A minibatch's request list sampled on the GPU: 1M nodes, waited for.
        dict(name="sample 1M nodes", kind="sample", nodes=1 << 20, edges=1 << 24, seeds=1024, fanout="15,10,5",
             wait=True),
        # The same on the 10M-node graph, 4096 seeds, queued ahead of its use.
        dict(name="sample 10M nodes", kind="sample", nodes=10_000_000, edges=120_000_000, seeds=4096,
             fanout="10,5,5", wait=False),
        # A typed minibatch's list split into its four node types (20M nodes).
        dict(name="split by type", kind="split", nodes=20_000_000, requests=389_123, types=4, own_work=True),
        # Rows in request order, fp32 x 1024, a minibatch of the 10M-node shape.
        dict(name="expand", kind="expand", nodes=10_000_000, requests=203_003, vectors=256),
        # The static score of the 1M-node graph, once before training.
        dict(name="pagerank", kind="pagerank", nodes=1 << 20, edges=1 << 24, iterations=20),
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm, odd ones among them."""
    return max(lo, min(hi, int(lo * (hi / lo) ** rng.random())))


def draw(rng):
    kind = rng.choice(["gather"] * 7 + ["sample"] * 2 + ["split", "expand", "pagerank"])
    if kind == "gather":
        nodes = _log(rng, 10_000, 1 << 20)
        vectors = _log(rng, 1, 128)
        fanout = rng.choice(["10,5", "10,5,5", "15,10,5", "25,10"])
        requests = _log(rng, 30, 150_000)
        seeds = max(4, requests // rng.randint(40, 150))
        resident = rng.random() < 0.35
        sets = nodes // 4 if resident else max(1, int(nodes * rng.uniform(0.05, 0.6)) // 8)
        lookahead = rng.choice([0, 2, 4, 8, 16])
        queues = rng.random() < 0.25 and lookahead > 0
        victim = rng.choice([0, max(lookahead + 1, int(nodes * rng.uniform(0.01, 0.1)))])
        mode = rng.choice(["blocking", "pipelined"])
        case = _gather("", nodes, int(nodes * rng.uniform(3, 16)), vectors, requests, seeds, fanout, sets, victim, lookahead,
                       mode, 1 if mode == "blocking" else rng.choice([4, 6]), lookahead + rng.choice([4, 8, 12]),
                       policy=rng.choice(["hybrid", "hybrid", "hybrid", "static", "dynamic", "round_robin"]),
                       victim_mode="queues" if queues else "fifo", refresh=rng.choice([1, 1, 4]),
                       pageable=rng.random() < 0.25, resident=resident)
        del case["name"]
        return case
    if kind == "sample":
        nodes = _log(rng, 1000, 10_000_000)
        return dict(kind=kind, nodes=nodes, edges=int(nodes * rng.uniform(2, 12)), seeds=_log(rng, 8, min(8192, nodes)),
                    fanout=rng.choice(["10,5", "10,5,5", "15,10,5", "25,10", "5,5,5,5", "64,3"]),
                    wait=rng.random() < 0.5)
    if kind == "split":
        return dict(kind=kind, nodes=_log(rng, 1000, 20_000_000), requests=_log(rng, 100, 1_000_000),
                    types=rng.randint(1, 16), own_work=rng.random() < 0.5)
    if kind == "expand":
        vectors = _log(rng, 1, 256)
        return dict(kind=kind, nodes=_log(rng, 1000, 10_000_000), vectors=vectors,
                    requests=_log(rng, 100, min(1_000_000, 50_000_000 // vectors)))
    nodes = _log(rng, 1000, 1 << 20)
    return dict(kind=kind, nodes=nodes, edges=int(nodes * rng.uniform(2, 16)), iterations=rng.choice([5, 10, 20]))


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _fanout(case):
    return [int(f) for f in case["fanout"].split(",")]


def _graph(nodes, edges, g):
    """R-MAT graph in CSR form by source: offsets int64, neighbours int32
    (self loops and repeated entries kept, neighbours sorted)."""
    scale = max(1, (nodes - 1).bit_length())
    src = torch.zeros(edges, dtype=torch.int64, device=DEV)
    dst = torch.zeros(edges, dtype=torch.int64, device=DEV)
    for _ in range(scale):
        r = torch.rand(edges, generator=g, device=DEV)
        src = (src << 1) + (r >= 0.76)
        dst = (dst << 1) + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    if nodes != 1 << scale:
        src, dst = (src * nodes) >> scale, (dst * nodes) >> scale
    key = torch.sort(src * nodes + dst)[0]
    src, dst = key // nodes, key % nodes
    off = torch.zeros(nodes + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.bincount(src, minlength=nodes), 0)
    return off, dst.to(torch.int32)


def _neighbour_list(off, adj, seeds, fanout, g):
    """The request list of some seeds: the seeds and, hop by hop, up to
    `fanout` random neighbours of every node reached so far (int64)."""
    parts, frontier = [seeds], torch.unique(seeds)
    for f in fanout:
        deg = off[frontier + 1] - off[frontier]
        pick = (torch.rand(frontier.numel(), f, generator=g, device=DEV) * deg[:, None]).long()
        pick = torch.minimum(pick, (deg - 1).clamp(min=0)[:, None]) + off[frontier][:, None]
        take = torch.arange(f, device=DEV)[None, :] < deg[:, None]
        part = adj[pick[take]].long()
        parts.append(part)
        frontier = torch.unique(part)
    return torch.cat(parts).contiguous()


def _request_list(case, off, adj, g):
    """A minibatch of exactly case["requests"] IDs: the lists of as many groups of seeds as it takes."""
    parts, n = [], 0
    while n < case["requests"]:
        seeds = torch.randint(0, case["nodes"], (case["seeds"],), generator=g, device=DEV)
        parts.append(_neighbour_list(off, adj, seeds, _fanout(case), g))
        n += parts[-1].numel()
    return torch.cat(parts)[: case["requests"]].contiguous()


def _skewed_ids(nodes, requests, g):
    """Request IDs as a power-law sampler gives them, without a graph."""
    u = torch.rand(requests, generator=g, device=DEV, dtype=torch.float64)
    return (u.pow(2.5) * nodes).long().clamp(max=nodes - 1)


def _result_words(n):
    """Pinned host memory for an asynchronous call's lengths and status."""
    return torch.zeros(n, dtype=torch.int64, pin_memory=True)


class _Stream:
    """A training (or serving) program's cache, store, request lists and
    output buffers, part way through its run."""

    def __init__(self, case, seed):
        g = _generator(seed)
        nodes, R = case["nodes"], 16 * case["vectors"]
        off, adj = _graph(nodes, case["edges"], g)
        self.lists = [_request_list(case, off, adj, g) for _ in range(case["lists"])]
        static = torch.bincount(adj.long(), minlength=nodes).cpu().numpy().astype(np.uint32)
        del off, adj
        rows = torch.empty(nodes * R // 2, dtype=torch.float16, device=DEV).normal_(generator=g).view(torch.uint8)
        if case["pageable"]:
            self.store = np.empty(nodes * R, np.uint8)
            torch.from_numpy(self.store).copy_(rows)
        else:
            self.store = lsmgnn.PinnedBuffer(nodes * R)
            torch.from_numpy(self.store.numpy()).copy_(rows)
        del rows
        fill = 1 << 16  # warm-up chunk of a resident table
        most = max(case["requests"], min(fill, nodes) if case["resident"] else 1)
        self.cache = lsmgnn.FeatureCache(nodes, R, self.store, static, case["sets"], case["victim"],
                                         case["lookahead"], most, pageable=case["pageable"],
                                         host_threads=16 if case["pageable"] else 0, policy=case["policy"],
                                         victim_mode=case["victim_mode"], refresh_period=case["refresh"])
        self.blocking, self.minibatches = case["mode"] == "blocking", case["minibatches"]
        self.lookahead = case["lookahead"]
        if case["resident"]:  # every row has been fetched once; the window is empty meanwhile
            buf = self._buffers(most, R)
            for a in range(0, nodes, fill):
                self.cache.gather(torch.arange(a, min(a + fill, nodes), device=DEV), *buf[:2], inverse=buf[2])
            del buf
        self.bufs = [self._buffers(case["requests"], R) for _ in range(self.minibatches)]
        self.t = 0
        # the k-th announcement is minibatch k: skip those of the warm-up gathers
        if self.lookahead:
            base = -(-nodes // fill) if case["resident"] else 0
            empty = torch.empty(0, dtype=torch.int64, device=DEV)
            for _ in range(base):
                self.cache.advance(empty)
            for j in range(self.lookahead + 1):
                self.cache.advance(self.lists[j % len(self.lists)])
        for _ in range(min(len(self.lists), 2 if case["resident"] else 16)):
            self._step_blocking(self.bufs[0])

    @staticmethod
    def _buffers(n, R):
        return (torch.zeros(n * R, dtype=torch.uint8, device=DEV), torch.zeros(n, dtype=torch.int64, device=DEV),
                torch.zeros(n, dtype=torch.int64, device=DEV))

    def _step_blocking(self, buf):
        K, t = len(self.lists), self.t
        r = self.cache.gather(self.lists[t % K], buf[0], buf[1], inverse=buf[2])
        if self.lookahead:
            self.cache.advance(self.lists[(t + self.lookahead + 1) % K])
        self.t = t + 1
        return r

    def step(self):
        if self.blocking:
            return [self._step_blocking(self.bufs[0])]
        K, done, last = len(self.lists), [], None
        for buf in self.bufs:
            t = self.t
            ahead = self.lists[(t + self.lookahead + 1) % K] if self.lookahead else None
            ticket, r = self.cache.gather_async(self.lists[t % K], buf[0], buf[1], inverse=buf[2], announce=ahead)
            if last is not None:
                self.cache.wait(last)  # the training step of the minibatch before follows here
            self.t, last = t + 1, ticket
            done.append(r)
        self.cache.wait(last)
        return done

    def __del__(self):
        if hasattr(self, "cache"):
            self.cache.close()
        if isinstance(getattr(self, "store", None), lsmgnn.PinnedBuffer):
            self.store.close()


def prepare(case, seed):
    kind, nodes = case["kind"], case["nodes"]
    if kind == "gather":
        return {"kind": kind, "stream": _Stream(case, seed)}
    g = _generator(seed)
    if kind == "sample":
        off, adj = _graph(nodes, case["edges"], g)
        fan = _fanout(case)
        most = reach = case["seeds"]
        for f in fan:
            reach = min(reach * f, case["edges"])
            most += reach
        count = 8
        seeds = torch.randint(0, nodes, (count, case["seeds"]), generator=g, device=DEV)
        out = torch.zeros(most, dtype=torch.int64, device=DEV)
        return {"kind": kind, "sampler": lsmgnn.GpuSampler(off, adj, fan, seed=seed & 0xffff), "seeds": seeds,
                "out": out, "result": _result_words(2), "wait": case["wait"], "b": 0}
    if kind == "split":
        T = case["types"]
        share = torch.rand(T, generator=g, device=DEV) + 0.1
        node_type = torch.multinomial(share, nodes, replacement=True, generator=g).to(torch.uint8)
        local = torch.empty(nodes, dtype=torch.int32, device=DEV)
        for t in range(T):
            mine = node_type == t
            local[mine] = torch.arange(int(mine.sum()), dtype=torch.int32, device=DEV)
        place = torch.randperm(nodes, generator=g, device=DEV)
        n = case["requests"]
        return {"kind": kind, "lists": [place[_skewed_ids(nodes, n, g)] for _ in range(4)], "node_type": node_type,
                "local": local, "outs": [torch.zeros(n, dtype=torch.int64, device=DEV) for _ in range(T)],
                "work": torch.zeros(lsmgnn.split_work_bytes(n, T), dtype=torch.uint8, device=DEV)
                if case["own_work"] else None, "result": _result_words(T + 1), "b": 0}
    if kind == "expand":
        uniq, inverse = torch.unique(_skewed_ids(nodes, case["requests"], g), return_inverse=True)
        R = 16 * case["vectors"]
        inverse = inverse[torch.randperm(inverse.numel(), generator=g, device=DEV)].contiguous()
        rows = torch.empty(uniq.numel() * R // 2, dtype=torch.float16, device=DEV).normal_(generator=g)
        return {"kind": kind, "rows": rows.view(torch.uint8), "inverse": inverse, "R": R,
                "out": torch.zeros(inverse.numel() * R, dtype=torch.uint8, device=DEV)}
    off, adj = _graph(nodes, case["edges"], g)
    return {"kind": kind, "off": off, "adj": adj, "iterations": case["iterations"]}


def run(state):
    kind = state["kind"]
    if kind == "gather":
        # the program's own buffers: rows, unique IDs and inverse index of each
        # minibatch (the first n_unique rows and unique IDs are this pass's)
        stream = state["stream"]
        return [(r.n_unique, *buf) for r, buf in zip(stream.step(), stream.bufs)]
    if kind == "expand":
        return lsmgnn.expand(state["rows"], state["inverse"], state["R"], out=state["out"])
    if kind == "pagerank":
        return lsmgnn.pagerank_scores(state["off"], state["adj"], iterations=state["iterations"], rank=True)
    b, state["b"] = state["b"], state["b"] + 1
    res = state["result"]
    if kind == "sample":
        seeds = state["seeds"][b % len(state["seeds"])]
        if state["wait"]:
            return state["sampler"].sample(seeds, b, state["out"]).numel(), state["out"]
        state["sampler"].sample_async(seeds, b, state["out"], res.data_ptr())
        return state["out"], res
    ids = state["lists"][b % len(state["lists"])]
    if state["work"] is not None:
        lsmgnn.split_by_type_async(ids, state["node_type"], state["local"], state["outs"], state["work"],
                                   res.data_ptr())
    else:
        lsmgnn.split_by_type_noalloc_async(ids, state["node_type"], state["local"], state["outs"],
                                          res.data_ptr())
    return list(state["outs"]), res


# ----------------------------------------------------------- what it takes
@functools.lru_cache(maxsize=None)
def _list_sizes(nodes, edges, seeds, fanout, requests=1):
    """(requests, unique IDs) of one minibatch of this shape; requests=1: of one group of seeds."""
    g = _generator(1)
    off, adj = _graph(nodes, edges, g)
    case = dict(nodes=nodes, seeds=seeds, fanout=fanout, requests=requests)
    if requests > 1:
        ids = _request_list(case, off, adj, g)
    else:
        ids = _neighbour_list(off, adj, torch.randint(0, nodes, (seeds,), generator=g, device=DEV), _fanout(case), g)
    return ids.numel(), torch.unique(ids).numel()


@functools.lru_cache(maxsize=None)
def _distinct(nodes, requests):
    """Expected distinct IDs among _skewed_ids(nodes, requests)."""
    edge = np.linspace(0.0, 1.0, nodes + 1) ** 0.4
    return float(-np.expm1(requests * np.log1p(-np.minimum(np.diff(edge), 1 - 1e-12))).sum())


def work(case):
    kind = case["kind"]
    if kind == "gather":
        # per minibatch: IDs in, unique IDs and inverse out, each unique row read and written once
        n, u = _list_sizes(case["nodes"], case["edges"], case["seeds"], case["fanout"], case["requests"])
        return {"bytes": case["minibatches"] * (16.0 * n + 8.0 * u + 32.0 * case["vectors"] * u), "flops": 0.0}
    if kind == "sample":
        # an adjacency entry read and an ID written per sample, two offsets per node expanded
        n, u = _list_sizes(case["nodes"], case["edges"], case["seeds"], case["fanout"])
        return {"bytes": 12.0 * n + 16.0 * u, "flops": 0.0}
    if kind == "split":
        return {"bytes": 21.0 * case["requests"], "flops": 0.0}  # ID, type, index in; index out
    if kind == "expand":
        # the inverse index, every output row written, every distinct row read once
        u = _distinct(case["nodes"], case["requests"])
        return {"bytes": case["requests"] * 8.0 + 16.0 * case["vectors"] * (case["requests"] + u), "flops": 0.0}
    # per iteration an index and a share per entry, a rank read and written per node
    it = case["iterations"]
    return {"bytes": it * (12.0 * case["edges"] + 24.0 * case["nodes"]) + 12.0 * case["nodes"],
            "flops": 2.0 * it * case["edges"]}


def tolerance(case):
    if case["kind"] == "pagerank":
        # 64-bit sums in another order (seen: 9e-15 against the sequential sums,
        # 4e-15 at most between two runs); a score whose rank lies within
        # rounding of a quantization step may differ by one
        return {"rel": 1e-13, "max": 1e-12, "differ": min(0.01, max(2e-5, 2.0 / case["nodes"]))}
    return "exact"


def exact(case, seed):
    """The ranks by a sequential power iteration in float64; every other
    output is moved, counted or listed, not computed."""
    if case["kind"] != "pagerank":
        return None
    nodes = case["nodes"]
    off, adj = _graph(nodes, case["edges"], _generator(seed))
    off, adj = off.cpu().numpy(), adj.cpu().numpy().astype(np.int64)
    deg = np.diff(off)
    rank = np.full(nodes, 1.0 / nodes)
    for _ in range(case["iterations"]):
        share = np.divide(rank, deg, out=np.zeros(nodes), where=deg > 0)
        pushed = np.bincount(adj, weights=np.repeat(share, deg), minlength=nodes)
        rank = 0.15 / nodes + 0.85 * (pushed + rank[deg == 0].sum() / nodes)
    return None, rank

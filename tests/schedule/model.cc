// A CPU model of what the host runtime of the feature-gather cache queues: the
// HIP calls it makes and the kernel launchers of internal.h, with no kernel run.
//
// Streams, events and host waits are vector clocks, so the model knows which
// queued operation is ordered behind which.  Every launcher declares the memory
// its kernels read and write (cache rows, staging rows, row lists, gate,
// outputs); two accesses of one resource, one of them a write, that no stream
// order, event or host wait puts in order are reported.  The victim ring's rows
// are checked by the slots' own rule: a host fetch reads rows written by the ring
// writes of gathers up to the second one before it, and a ring write overwrites
// rows that no later gather's fetch reads.
//
// What a batch would have found (unique IDs, host rows, enqueues, an ID out of
// range) is given by the test beforehand (model_plan).  Device addresses are
// numbers, never dereferenced.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "internal.h"
#include "lsmgnn.h"

struct ihipStream_t {
  int id;
};
struct ihipEvent_t {
  std::vector<uint32_t> clock;
};

namespace {

using Clock = std::vector<uint32_t>;
void join(Clock &a, const Clock &b) {
  if (a.size() < b.size()) a.resize(b.size());
  for (size_t i = 0; i < b.size(); ++i)
    if (a[i] < b[i]) a[i] = b[i];
}

// One queued operation: its stream, its position there, and what precedes it.
struct Op {
  int stream = 0;
  uint32_t seq = 0;
  Clock clock;
  std::string name;
};
bool before(const Op &a, const Op &b) {
  return (size_t)a.stream < b.clock.size() && a.seq <= b.clock[a.stream];
}

struct Plan {
  uint32_t unique = 0, early = 0, late = 0, enq = 0;
  bool err = false;
};

struct Batch {  // the gather that last reset a gate
  Plan p;
  uint64_t t = 0;
};

struct CacheState {
  std::vector<std::pair<uint64_t, Op>> fetches, writes, prefetches;  // by gather
  std::vector<uint64_t> enqueued;                                    // gathers with ring rows to write
};

struct Model {
  std::map<int, Clock> streams;  // 0: the caller's
  Clock host;
  int next_stream = 1;
  uintptr_t next_addr = (uintptr_t)1 << 44;
  std::map<std::pair<uintptr_t, int>, std::vector<std::pair<Op, bool>>> mem;
  Plan plan;
  std::map<const void *, Batch> batch;       // by gate
  std::map<const void *, uint64_t> staged;   // staging rows -> gather
  std::map<const void *, CacheState> cache;  // by DevState::sets
  std::map<const void *, const void *> cache_of;  // staging rows -> DevState::sets
  lsm::DedupResult *dd = nullptr;  // a dedup result not yet seen by the host
  uint64_t dd_word = 0;
  Op dd_op;
  bool caller_busy = false;
  std::string log, errors;
} M;

// the runtime creates its streams three at a time, in this order
const char *stream_name(int id) {
  static const char *names[] = {"meta", "host", "dma"};
  return id ? names[(id - 1) % 3] : "caller";
}

Op queue(hipStream_t s, const std::string &name) {
  Op op;
  op.stream = s ? s->id : 0;
  op.name = name + "@" + stream_name(op.stream);
  Clock &c = M.streams[op.stream];
  join(c, M.host);
  if (c.size() <= (size_t)op.stream) c.resize(op.stream + 1);
  op.seq = ++c[op.stream];
  op.clock = c;
  M.log += op.name + "\n";
  return op;
}

void error(const std::string &e) { M.errors += e + "\n"; }

void touch(const Op &op, const void *p, int part, bool write) {
  if (!p) return;
  auto &v = M.mem[{reinterpret_cast<uintptr_t>(p), part}];
  for (auto &a : v)
    if ((write || a.second) && !before(a.first, op))
      error((a.second ? "write " : "read ") + a.first.name + " not before " + (write ? "write " : "read ") + op.name +
            " (part " + std::to_string(part) + ")");
  if (write) v.clear();
  v.push_back({op, write});
}
void reads(const Op &op, const void *p, int part = 0) { touch(op, p, part, false); }
void writes(const Op &op, const void *p, int part = 0) { touch(op, p, part, true); }

// Parts of a gate that different kernels append to.
enum { kGateHead, kGateLists, kGateStage, kGateQueue };
// Parts of the output rows and of the host-fetch list.
enum { kOutHost, kOutHit };

const Batch &of(const lsm::Scratch &sc) { return M.batch[sc.gate]; }
std::string tag(const char *what, const lsm::Scratch &sc) {
  return std::to_string(of(sc).t) + (of(sc).p.err ? " rejected " : " ") + what;
}

// a gather's gate is reset: its lists are empty from here on
void reset_gate(const Op &op, const lsm::Scratch &sc) {
  for (int k = kGateHead; k <= kGateQueue; ++k) writes(op, sc.gate, k);
}

void publish(const Op &op, lsm::DedupResult *dd, uint32_t tag_, const Plan &p) {
  M.dd = dd;
  M.dd_word = lsm::dedup_word(tag_, p.err, p.err ? 0 : p.unique);
  M.dd_op = op;
}

void counters(const lsm::DevState &d, const Batch &b, lsm::Counters *hc) {
  std::memset(hc, 0, sizeof(*hc));
  hc->n_unique = b.p.unique;
  hc->n_host = b.p.early + b.p.late;
  hc->misses = hc->n_host;
  hc->hits = b.p.unique - hc->n_host;
  hc->enq_total = d.V ? b.p.enq : 0;
  if (d.qmode) hc->q_placed[(b.t + 1) % (d.L + 1)] = hc->enq_total;
  if (hc->enq_total) M.cache[d.sets].enqueued.push_back(b.t);
}

void fetch_early(const Op &op, const lsm::Scratch &sc, const void *out) {
  reads(op, sc.gate, kGateHead);
  if (of(sc).p.err) return;
  reads(op, sc.host_list, 0);
  writes(op, out, kOutHost);
}

// the host fetch's second part reads ring rows of gathers up to t - 2
void fetch_late(const Op &op, const lsm::DevState &d, const lsm::Scratch &sc, const void *out) {
  reads(op, sc.gate, kGateHead);
  reads(op, sc.gate, kGateLists);
  const Batch &b = of(sc);
  if (b.p.err) return;
  reads(op, sc.host_list, 1);
  writes(op, out, kOutHost);
  CacheState &c = M.cache[d.sets];
  if (!d.qmode)
    for (uint64_t s : c.enqueued) {
      if (s + 2 > b.t) continue;
      bool there = false;
      for (auto &w : c.writes)
        if (w.first == s) {
          there = true;
          if (!before(w.second, op)) error(w.second.name + " not before " + op.name);
        }
      if (!there) error("ring write of gather " + std::to_string(s) + " not queued before " + op.name);
    }
  c.fetches.push_back({b.t, op});
}

const uint8_t *staging_of(const lsm::DevState &d, uint64_t t) {
  return d.rows + (d.stage_row0 + (t & 1) * d.stage_rows) * d.R;
}

void hit(const Op &op, const lsm::DevState &d, const lsm::Scratch &sc, const void *out) {
  reads(op, sc.gate, kGateHead);
  const Batch &b = of(sc);
  if (b.p.err) return;
  reads(op, sc.hbm.src);
  reads(op, d.rows);
  if (d.V && !d.qmode && b.t) reads(op, staging_of(d, b.t + 1));
  if (d.V && d.qmode) reads(op, d.rows, 1 + (int)(b.t & 1));
  writes(op, out, kOutHit);
}

void stage(const Op &op, const lsm::DevState &d, const lsm::Scratch &sc) {
  reads(op, sc.gate, kGateHead);
  reads(op, sc.gate, kGateStage);
  if (of(sc).p.err) return;
  reads(op, sc.stage.src);
  reads(op, d.rows);
  writes(op, sc.staging);
  M.staged[sc.staging] = of(sc).t;
  M.cache_of[sc.staging] = d.sets;
}

void fill(const Op &op, const lsm::DevState &d, const lsm::Scratch &sc, const void *out) {
  reads(op, sc.gate, kGateHead);
  reads(op, sc.gate, kGateLists);
  if (of(sc).p.err) return;
  reads(op, sc.fill.src);
  reads(op, out, kOutHost);
  reads(op, out, kOutHit);
  writes(op, d.rows);
}

}  // namespace

// ------------------------------------------------------------- HIP calls
extern "C" {
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
  *p = reinterpret_cast<void *>(M.next_addr);
  M.next_addr += (n + 4095) / 4096 * 4096;
  return hipSuccess;
}
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  *p = std::aligned_alloc(64, (n + 63) / 64 * 64);
  if (*p) std::memset(*p, 0, n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { return *d = h, hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *, const void *) { return hipErrorInvalidValue; }
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  return *s = new ihipStream_t{M.next_stream++}, hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return delete s, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return join(M.host, M.streams[s ? s->id : 0]), hipSuccess; }
hipError_t hipStreamQuery(hipStream_t s) {
  if (!s) return M.caller_busy ? hipErrorNotReady : hipSuccess;
  if (M.dd) {  // the host polls: its dedup result arrives
    __atomic_store_n(&M.dd->word, M.dd_word, __ATOMIC_RELEASE);
    join(M.host, M.dd_op.clock);
    M.dd = nullptr;
  }
  return hipErrorNotReady;
}
hipError_t hipEventCreate(hipEvent_t *e) { return *e = new ihipEvent_t{}, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  Clock &c = M.streams[s ? s->id : 0];
  join(c, M.host);
  return e->clock = c, hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  return join(M.streams[s ? s->id : 0], e->clock), hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { return join(M.host, e->clock), hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 0, hipSuccess; }
// the only runtime copies are the ring (or queue) writes, from the staging rows
hipError_t hipMemcpyAsync(void *, const void *src, size_t, hipMemcpyKind, hipStream_t s) {
  const void *base = nullptr;  // the staging rows the copy starts in
  for (auto &st : M.staged)
    if (st.first <= src && (!base || st.first > base)) base = st.first;
  const uint64_t t = M.staged[base];
  const Op op = queue(s, std::to_string(t) + " ring_write");
  reads(op, base);
  CacheState &c = M.cache[M.cache_of[base]];
  for (auto &f : c.fetches)
    if (f.first <= t && !before(f.second, op)) error(f.second.name + " not before " + op.name);
  for (auto &f : c.prefetches)
    if (f.first + 2 <= t && !before(f.second, op)) error(f.second.name + " not before " + op.name);
  c.writes.push_back({t, op});
  return hipSuccess;
}
}

// ------------------------------------------------------------- launchers
namespace lsm {

void launch_dedup(const DevState &, const int64_t *, uint64_t, const int64_t *, uint64_t, Scratch &sc,
                  int64_t *unique_out, Counters *, DedupResult *dd, uint32_t t, hipStream_t s) {
  M.batch[sc.gate].p = M.plan;
  const Op op = queue(s, "dedup");
  reset_gate(op, sc);
  if (!M.plan.err) writes(op, unique_out);
  publish(op, dd, t, M.plan);
}

void launch_probe(const DevState &, uint64_t, uint64_t t, Scratch &sc, Counters *, StatGrids &, hipStream_t s) {
  M.batch[sc.gate].t = t;
  const Op op = queue(s, tag("probe", sc));
  if (of(sc).p.err) return;
  writes(op, sc.gate, kGateHead);
  writes(op, sc.host_list, 0);
}

void launch_refresh(const DevState &, uint32_t, const Counters *, hipStream_t s) { queue(s, "refresh"); }
void launch_group_by_set(const DevState &, uint64_t, uint32_t, Scratch &, Counters *, StatGrids &, hipStream_t s) {
  queue(s, "group");
}
void launch_set_walk(const DevState &, uint64_t, uint32_t, Scratch &, Counters *, StatGrids &, hipStream_t s) {
  queue(s, "walk");
}

static void resolved(const Op &op, Scratch &sc, uint8_t *outcome) {
  if (of(sc).p.err) return;
  writes(op, sc.gate, kGateLists);
  writes(op, sc.host_list, 1);
  writes(op, sc.hbm.src);
  writes(op, sc.fill.src);
  writes(op, outcome);
}
void launch_ring_resolve(const DevState &, uint64_t, uint64_t, Scratch &sc, uint8_t *outcome, Counters *, StatGrids &,
                         hipStream_t s) {
  resolved(queue(s, tag("resolve", sc)), sc, outcome);
}

// the gather whose counters the next finish publishes (an empty gather has none)
static const DevState *finish_dev = nullptr;
static const void *finish_gate = nullptr;

static void enqueued(const Op &op, Scratch &sc, int64_t *inverse) {
  if (of(sc).p.err) return;
  writes(op, sc.gate, kGateStage);
  writes(op, sc.stage.src);
  writes(op, inverse);
}
void launch_ring_enqueue(const DevState &d, const int64_t *, uint64_t, uint64_t, int64_t *inverse, Scratch &sc,
                         Counters *, StatGrids &, hipStream_t s) {
  enqueued(queue(s, tag("enqueue", sc)), sc, inverse);
  finish_dev = &d;
  finish_gate = sc.gate;
}

void launch_finish(Counters *, Counters *host, const uint32_t *, const StatGrids &, uint64_t *, const QueueFinish &qf,
                   const AnnounceArgs &, hipStream_t s) {
  const Op op = queue(s, "finish");
  if (qf.gate) writes(op, qf.gate, kGateQueue);
  std::memset(host, 0, sizeof(*host));
  if (finish_dev && !M.batch[finish_gate].p.err) counters(*finish_dev, M.batch[finish_gate], host);
  finish_dev = nullptr;
}

void launch_tiny(const DevState &d, Scratch &sc, const TinyArgs &a, Counters *, hipStream_t s) {
  Batch &b = M.batch[sc.gate];
  b.p = M.plan;
  b.t = a.t;
  const Op op = queue(s, tag("tiny", sc));
  reset_gate(op, sc);
  publish(op, a.dd, a.tag, b.p);
  if (b.p.err) return;
  writes(op, a.unique_out);
  writes(op, sc.host_list, 0);
  resolved(op, sc, a.outcome);
  enqueued(op, sc, a.inverse);
  counters(d, b, a.hc);
}

void launch_move_rows(const DevState &d, uint64_t, const Scratch &sc, uint8_t *out, hipStream_t s) {
  const Op op = queue(s, tag("move_rows", sc));
  fetch_early(op, sc, out);
  fetch_late(op, d, sc, out);
  hit(op, d, sc, out);
  if (d.V) stage(op, d, sc);
}

void launch_copy(CopyMode mode, const DevState &d, uint64_t, const Scratch &sc, uint8_t *out, hipStream_t s) {
  switch (mode) {
    case CopyMode::kHostEarly: return fetch_early(queue(s, tag("host_early", sc)), sc, out);
    case CopyMode::kHostLate: return fetch_late(queue(s, tag("host_late", sc)), d, sc, out);
    case CopyMode::kHbmToOut: return hit(queue(s, tag("hit_copy", sc)), d, sc, out);
    case CopyMode::kCacheToStage: return stage(queue(s, tag("stage", sc)), d, sc);
    case CopyMode::kOutToCache: return fill(queue(s, tag("fill", sc)), d, sc, out);
  }
}

void launch_prefetch(const DevState &d, const Gate *gate, const uint8_t *staging, uint32_t, uint32_t par,
                     hipStream_t s) {
  const uint64_t t = M.batch[gate].t;
  const Op op = queue(s, std::to_string(t) + " prefetch");
  reads(op, gate, kGateQueue);
  reads(op, staging);
  writes(op, d.rows, 1 + (int)par);
  CacheState &c = M.cache[d.sets];
  for (uint64_t e : c.enqueued) {
    if (e >= t) continue;
    bool there = false;
    for (auto &w : c.writes)
      if (w.first == e) {
        there = true;
        if (!before(w.second, op)) error(w.second.name + " not before " + op.name);
      }
    if (!there) error("queue write of gather " + std::to_string(e) + " not queued before " + op.name);
  }
  c.prefetches.push_back({t, op});
}

void launch_publish_count(const Gate *gate, const uint32_t *count, uint32_t *dst, hipStream_t s) {
  const Op op = queue(s, "publish_count");
  const bool early = count == &gate->n_early;
  reads(op, gate, early ? kGateHead : kGateLists);
  const Plan &p = M.batch[gate].p;
  *dst = p.err ? 0 : early ? p.early : p.late;
}

void launch_expand(const uint8_t *, const int64_t *, uint64_t, uint64_t, uint8_t *, hipStream_t) {}
void launch_window_set(const int64_t *, uint64_t, uint64_t, uint32_t, uint32_t, uint64_t *, bool, uint32_t *,
                       hipStream_t s) {
  queue(s, "window_set");
}
void launch_window_rollback(const int64_t *, uint64_t, uint64_t, uint32_t, uint32_t, uint64_t *, hipStream_t s) {
  queue(s, "window_rollback");
}
void launch_copy_plain(const void *, void *, uint64_t, bool, hipStream_t) {}
uint64_t set_of_host(uint64_t x, uint64_t n) { return x % n; }

}  // namespace lsm

// --------------------------------------------------------- the test's side
extern "C" {
// What the next gather's batch finds.
void model_plan(uint32_t unique, uint32_t early, uint32_t late, uint32_t enq, int err) {
  M.plan = Plan{unique, early, late, enq, err != 0};
}
// Whether the caller's stream still has work queued when a call looks at it.
void model_caller_busy(int busy) { M.caller_busy = busy != 0; }
// The caller's stream reads a gather's outputs.
void model_read_outputs(const void *out, const void *unique, const void *inverse, const void *outcome) {
  const Op op = queue(nullptr, "read_outputs");
  reads(op, out, kOutHost);
  reads(op, out, kOutHit);
  for (const void *p : {unique, inverse, outcome}) reads(op, p);
}
const char *model_log() { return M.log.c_str(); }
void model_clear_log() { M.log.clear(); }
const char *model_errors() { return M.errors.c_str(); }
void model_reset() { M = Model{}; }
}

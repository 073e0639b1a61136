// gfx950 kernels of the feature-gather cache (LSM-GNN, arXiv 2407.15264).
//
// One gather runs as a short pipeline of stream-ordered kernels.  Every count
// that depends on the batch (unique IDs, touched sets, work-list lengths, the
// ring tail) stays in device memory, so the host queues the whole pipeline
// before it learns anything about the batch.  Each kernel reads the error flag
// first (Counters::err, or the gather's gate in the row copies) and does
// nothing once an out-of-range ID was seen, so an invalid batch changes no state.
//
//   dedup       byte map over node IDs marked with plain stores, per-chunk
//               popcount, chunk scan, ascending compaction that records each
//               node's unique index; the inverse index is one lookup
//   probe       each unique ID's set looked up in the batch-start state (the
//               misses this already fixes are listed for the host fetch) and
//               counted; a set whose IDs are all resident is settled here, since
//               hits change nothing
//   group       segment allocation and placement of the other sets' IDs
//   set walk    eight lanes per set (one per way) order its IDs and walk them in
//               ascending order: tag probe, then on a fill the
//               empty way or the minimum (level, static score, way) victim
//               (Sec. 4.2 levels; Sec. 4.3.2 swap when the victim ring is on)
//   ring        the resolve scans the enqueue flags into FIFO sequence numbers in
//               ascending-ID order; victim hits are resolved arithmetically:
//               an entry with sequence q is still in the ring at x's turn iff
//               q + V >= tail0 + (enqueues before x)  (Sec. 4.3.1)
//   data        row copies with 128-bit loads/stores: hits HBM->out, misses
//               and victim hits pinned host->out (a dense list, small grid),
//               enqueued rows HBM->staging in ring order (a runtime copy then
//               writes them to the pinned ring), then fills out->HBM for each
//               way's final occupant
#include "internal.h"

namespace lsm {

// ---------------------------------------------------------------- helpers
// set index: SplitMix64 output for state x (Steele, Lea, Flood 2014), reduced
// with Lemire's multiply-shift on its high 32 bits
__host__ __device__ __forceinline__ uint32_t set_index(uint64_t x, uint64_t S) {
  uint64_t z = x + 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z ^= z >> 31;
  return (uint32_t)(((z >> 32) * S) >> 32);
}

uint64_t set_of_host(uint64_t x, uint64_t num_sets) { return set_index(x, num_sets); }

// Block-wide exclusive scan of one value per thread (kBlock threads).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t &total) {
  __shared__ uint32_t wsum[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63) wsum[wid] = x;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kBlock / 64; ++w) {
    const uint32_t sw = wsum[w];
    base += (w < wid) ? sw : 0u;
    tot += sw;
  }
  __syncthreads();
  total = tot;
  return base + x - v;
}

// The same for 64-bit values.
__device__ __forceinline__ uint64_t block_exclusive_scan64(uint64_t v, uint64_t &total) {
  __shared__ uint64_t wsum[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint64_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63) wsum[wid] = x;
  __syncthreads();
  uint64_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kBlock / 64; ++w) {
    const uint64_t sw = wsum[w];
    base += (w < wid) ? sw : 0ull;
    tot += sw;
  }
  __syncthreads();
  total = tot;
  return base + x - v;
}

__device__ __forceinline__ uint32_t block_sum(uint32_t v) {
  uint32_t tot;
  (void)block_exclusive_scan(v, tot);
  return tot;
}

// Rank of this thread among the block's threads with `pred` set, from ballots,
// and how many there are.  For kN predicates at once: one pair of barriers.
template <int kN>
__device__ __forceinline__ void block_ranks(const bool (&pred)[kN], uint32_t (&rank)[kN], uint32_t (&total)[kN]) {
  __shared__ uint32_t wcnt[kN][kBlock / 64];
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    const uint64_t m = __ballot(pred[i]);
    rank[i] = (uint32_t)__popcll(m & lt);
    if (lane == 0) wcnt[i][wid] = (uint32_t)__popcll(m);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    total[i] = 0;
#pragma unroll
    for (uint32_t w = 0; w < kBlock / 64; ++w) {
      const uint32_t c = wcnt[i][w];
      rank[i] += w < wid ? c : 0u;
      total[i] += c;
    }
  }
  __syncthreads();
}

// A gather's gate as the dedup leaves it: the error flag and the unique count,
// every list empty.
__device__ __forceinline__ Gate gate_with(uint32_t err, uint32_t n_unique) {
  Gate g{};
  g.err = err;
  g.n_unique = n_unique;
  return g;
}

// The dedup's result for the host, which polls for it.
__device__ __forceinline__ void publish_dedup(DedupResult *dd, uint32_t tag, uint32_t err, uint32_t n_unique) {
  __hip_atomic_store(&dd->word, dedup_word(tag, err, n_unique), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

static inline unsigned grid_for(uint64_t work, uint64_t per_block, unsigned cap) {
  uint64_t b = (work + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

// ------------------------------------------------------------------ finish
// Last kernel of every call: add up the per-block partial counts, publish all
// counters to pinned host memory, advance the ring tail by the call's enqueues
// (keeping the previous tail) and zero the device counters for the next call
// (they start zeroed at create).
//
// With an announcement (ann.ids != NULL) the launch has more blocks, which all
// also set the announced minibatch's bit for each of its IDs, unless the
// gather's gate holds an error: the announced bits are first read by the next
// gather's set walk.  Only that bit of a node's window changes in this kernel
// (duplicates write the same value), so a plain read-modify-write is exact.
//
// A node's window word holds the gather index it was last written for (upper
// half) and one bit per announced minibatch after that one: bits that are
// behind by now fall out when the word is read, so no pass clears a served
// minibatch's bits, and no copy of the announced lists is kept for it: with such
// a pass (a random read-modify-write per request) and the copy, four gathers
// of 900 K requests took 1133 us beside their row copies, now 1063.
__device__ __forceinline__ uint32_t window_bits(uint64_t w, uint32_t now) {
  const uint32_t behind = now - (uint32_t)(w >> 32);
  return behind < 32u ? (uint32_t)w >> behind : 0u;  // bit i: minibatch now + 1 + i
}

__device__ __forceinline__ void window_set(uint64_t *win, uint64_t x, uint32_t now, uint32_t bit) {
  const uint64_t w = win[x];
  const uint64_t v = (uint64_t)now << 32 | window_bits(w, now) | 1u << bit;
  if (v != w) win[x] = v;
}

__device__ __forceinline__ void announce(const AnnounceArgs &a) {
  if (a.gate->err) return;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < a.n; i += gridDim.x * kBlock)
    window_set(a.win, (uint64_t)a.ids[i], a.now, a.bit);
}

__device__ __forceinline__ void finish(Counters *cn, Counters *host, const uint32_t *part, const StatGrids &grids,
                                       uint64_t *tail, const QueueFinish &qf) {
  __shared__ uint32_t red[kNumStat][kBlock / 64];
  __shared__ uint32_t sums[kNumStat];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  // Each pass loads one partial of every slot before adding any: the loads
  // are independent, so a pass costs one memory round trip (several µs while
  // host-link reads are in flight beside this kernel) instead of one per slot.
  uint32_t gmax = 0;
#pragma unroll
  for (int st = 0; st < kNumStat; ++st) gmax = grids.g[st] > gmax ? grids.g[st] : gmax;
  uint32_t v[kNumStat];
#pragma unroll
  for (int st = 0; st < kNumStat; ++st) v[st] = 0;
  for (uint32_t b = threadIdx.x; b < gmax; b += kBlock) {
    uint32_t a[kNumStat];
#pragma unroll
    for (int st = 0; st < kNumStat; ++st) a[st] = b < grids.g[st] ? part[st * kMaxGrid + b] : 0u;
#pragma unroll
    for (int st = 0; st < kNumStat; ++st) v[st] += a[st];
  }
#pragma unroll
  for (int st = 0; st < kNumStat; ++st) {
    uint32_t x = v[st];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if (lane == 0) red[st][wid] = x;
  }
  __syncthreads();
  // the counters are staged in LDS and copied word by word by the whole block
  // (a private copy would live in scratch memory: its queue arrays are indexed
  // at run time)
  constexpr uint32_t kWords = sizeof(Counters) / 4;
  static_assert(sizeof(Counters) % 4 == 0 && kWords <= kBlock, "counters are copied one word per thread");
  __shared__ Counters c;
  if (threadIdx.x < kWords) reinterpret_cast<uint32_t *>(&c)[threadIdx.x] = reinterpret_cast<const uint32_t *>(cn)[threadIdx.x];
  if (threadIdx.x < kNumStat) {
    uint32_t v = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) v += red[threadIdx.x][w];
    sums[threadIdx.x] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    c.hits = sums[kStHits] + sums[kStSettled];
    c.fills = sums[kStFills];
    c.evictions = sums[kStEvictions];
    c.enqueued = sums[kStEnqueued];
    c.dropped = sums[kStDropped];
    c.n_fill = sums[kStFinal];
    c.victim_hits = sums[kStVictimHits];
    c.misses = sums[kStMisses];
    c.n_hbm = sums[kStHbm];
    c.n_host = sums[kStHost] + sums[kStEarly];  // both parts of the host-fetch list
    c.n_enq_copy = sums[kStEnqCopy];
    c.req_hits = sums[kStReqHits];
    c.req_victim_hits = sums[kStReqVictimHits];
    c.vh_ring = sums[kStVhRing];
    c.vh_staged = sums[kStVhStaged];
    c.vh_same = sums[kStVhSame];
    // queue mode: candidates that found their queue full were dropped
    c.enqueued -= c.q_overflow;
    c.dropped += c.q_overflow;
    if (tail && !c.err) {  // a rejected gather leaves both tails alone
      tail[1] = tail[0];
      tail[0] += c.enq_total;
    }
    if (qf.qcount && !c.err) {
      // the served queue is empty from now on; the next gather's queue holds
      // qcount[next] entries, the last q_placed[next] of them staged by this
      // gather after the rows it staged for the lower slots
      qf.qcount[qf.cur] = 0;
      uint32_t off = 0;
      for (uint32_t k = 0; k < qf.next; ++k) off += c.q_placed[k];
      const uint32_t cnt = qf.qcount[qf.next];
      qf.gate->q_count = cnt;
      qf.gate->q_before = cnt - c.q_placed[qf.next];
      qf.gate->q_stage_off = off;
    }
  }
  __syncthreads();
  if (threadIdx.x < kWords) {
    // written through: the host reads them once a later kernel's word is there
    __hip_atomic_store(reinterpret_cast<uint32_t *>(host) + threadIdx.x,
                       reinterpret_cast<const uint32_t *>(&c)[threadIdx.x], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
    reinterpret_cast<uint32_t *>(cn)[threadIdx.x] = 0u;
  }
}

__global__ __launch_bounds__(kBlock) void k_finish(Counters *cn, Counters *host, const uint32_t *part,
                                                   StatGrids grids, uint64_t *tail, QueueFinish qf,
                                                   AnnounceArgs ann) {
  if (ann.ids) announce(ann);
  if (blockIdx.x == 0) finish(cn, host, part, grids, tail, qf);
}

void launch_finish(Counters *cn, Counters *host, const uint32_t *stat_part, const StatGrids &grids,
                   uint64_t *tail, const QueueFinish &qf, const AnnounceArgs &ann, hipStream_t s) {
  const unsigned g = ann.ids ? grid_for(ann.n, kBlock, kMaxGrid) : 1u;
  hipLaunchKernelGGL(k_finish, dim3(g), dim3(kBlock), 0, s, cn, host, stat_part, grids, tail, qf, ann);
}

// ------------------------------------------------------------------- dedup
// A byte per node marks the batch's requests.  Plain byte stores need no
// atomics: every writer of a byte writes the same value, and bytes of
// different nodes never interfere.  A bit per node would make the popcount
// and compaction passes read N/8 bytes instead of N, but its marks need
// atomic ORs, and repeated IDs of hub nodes queue on one word: measured on
// the MI355X, the byte map gives 478 GB/s on the 100M-node workload (the
// largest N here, 100 MB per pass) against 428-437 with the bitmap.
//
// Validate and mark.  Out-of-range IDs set Counters::err; valid ones are still
// marked, and the compaction kernel then clears the map without compacting it,
// so a rejected batch leaves no trace.  The list announced with the gather
// (if any) is validated here too; its bits are set only after the gather has
// been accepted.
__global__ void k_mark(const int64_t *ids, uint32_t n, const int64_t *ann_ids, uint32_t ann_n, uint64_t N,
                       uint8_t *present, Counters *cn) {
  bool bad = false;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const int64_t x = ids[i];
    if (x < 0 || (uint64_t)x >= N) {
      bad = true;
    } else {
      present[x] = 1;
    }
  }
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < ann_n; i += gridDim.x * kBlock) {
    const int64_t x = ann_ids[i];
    bad |= x < 0 || (uint64_t)x >= N;
  }
  if (__ballot(bad) && __lane_id() == 0) atomicOr(&cn->err, 1u);
}

// Each thread owns kW consecutive words of the map (kW / 4 128-bit loads);
// marked bytes hold exactly 1, so a popcount of a word counts them.  With 64
// bytes per thread whatever the number of nodes, 16 K nodes were one block's
// work (compaction 7.4 us, with 16 bytes 3.8) and 1M nodes 64 blocks'.
template <int kW>
__device__ __forceinline__ void load_words(const uint8_t *present, uint32_t (&w)[kW]) {
  const u32x4 *p = reinterpret_cast<const u32x4 *>(present + ((size_t)blockIdx.x * kBlock + threadIdx.x) * 4 * kW);
#pragma unroll
  for (int k = 0; k < kW / 4; ++k) {
    const u32x4 a = p[k];
    w[4 * k] = a.x; w[4 * k + 1] = a.y; w[4 * k + 2] = a.z; w[4 * k + 3] = a.w;
  }
}

template <int kW>
__global__ __launch_bounds__(kBlock) void k_chunk_popc(const uint8_t *present, uint32_t *chunk_sums,
                                                       const Counters *cn) {
  if (cn->err) return;
  uint32_t w[kW];
  load_words(present, w);
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < kW; ++k) c += __popc(w[k]);
  const uint32_t tot = block_sum(c);
  if (threadIdx.x == 0) chunk_sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kBlock) void k_chunk_scan(uint32_t *chunk_sums, uint32_t nchunks, Counters *cn,
                                                       DedupResult *dd, uint32_t tag, Gate *gate) {
  const uint32_t err = cn->err;
  if (err) {
    if (threadIdx.x == 0) {
      *gate = gate_with(err, 0);
      publish_dedup(dd, tag, err, 0);
    }
    return;
  }
  uint32_t carry = 0;
  for (uint32_t base = 0; base < nchunks; base += kBlock) {
    const uint32_t i = base + threadIdx.x;
    const uint32_t v = i < nchunks ? chunk_sums[i] : 0u;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan(v, tot);
    if (i < nchunks) chunk_sums[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) {
    cn->n_unique = carry;
    *gate = gate_with(0, carry);
    publish_dedup(dd, tag, 0, carry);
  }
}

// The compaction: each node of the chunk with its bit set, ascending, gets the
// next unique index.  kFused: the chunk's first index is the sum of the
// earlier chunks' counts, added up by the block itself (few chunks: this
// saves the separate one-block scan), and the last chunk's block publishes
// the unique count; otherwise chunk_off holds the scanned offsets.  Each
// node's own unique index is written later (k_place).
template <int kW, bool kFused>
__global__ __launch_bounds__(kBlock) void k_compact(uint8_t *present, const uint32_t *chunk_off, uint32_t *uniq,
                                                    int64_t *uniq_out, Counters *cn, uint32_t nchunks,
                                                    DedupResult *dd, uint32_t tag, Gate *gate) {
  uint32_t w[kW];
  load_words(present, w);
  const size_t b0 = ((size_t)blockIdx.x * kBlock + threadIdx.x) * 4 * kW;  // first byte of this thread
  const uint32_t err = cn->err;
  // the marks are this block's to read and clear, whether or not the batch is
  // rejected (cleared later, by a store per unique ID, they were as many
  // scattered lines)
#pragma unroll
  for (int k = 0; k < kW; ++k)
    if (w[k]) reinterpret_cast<uint32_t *>(present + b0)[k] = 0;
  if (err) {
    if (kFused && blockIdx.x == 0 && threadIdx.x == 0) {
      *gate = gate_with(err, 0);
      publish_dedup(dd, tag, err, 0);
    }
    return;
  }
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < kW; ++k) c += __popc(w[k]);
  uint32_t tot;
  const uint32_t ex = block_exclusive_scan(c, tot);
  uint32_t first;
  if constexpr (kFused) {
    uint32_t v = 0;
    for (uint32_t j = threadIdx.x; j < blockIdx.x; j += kBlock) v += chunk_off[j];
    first = block_sum(v);
    if (blockIdx.x == nchunks - 1 && threadIdx.x == 0) {
      const uint32_t total = first + tot;
      cn->n_unique = total;
      *gate = gate_with(0, total);
      publish_dedup(dd, tag, 0, total);
    }
  } else {
    first = chunk_off[blockIdx.x];
  }
  if (tot == 0) return;
  uint32_t pos = first + ex;
#pragma unroll
  for (int k = 0; k < kW; ++k) {
    uint32_t word = w[k];
    while (word) {  // marked bytes ascending: bit 8j is set for byte j of word k
      const uint32_t x = (uint32_t)(b0 + 4 * k + (__builtin_ctz(word) >> 3));
      uniq[pos] = x;
      uniq_out[pos] = (int64_t)x;
      ++pos;
      word &= word - 1u;
    }
  }
}

constexpr uint32_t kFusedChunkMax = 2048;  // at most this many chunk sums are added up by each block

template <int kW>
static void launch_compaction(const DevState &d, const Scratch &sc, int64_t *unique_out, Counters *cn, DedupResult *dd,
                              uint32_t tag, hipStream_t s) {
  const dim3 g((unsigned)d.nchunks);
  const uint32_t n = (uint32_t)d.nchunks;
  hipLaunchKernelGGL(k_chunk_popc<kW>, g, dim3(kBlock), 0, s, d.present, d.chunk_sums, cn);
  static_assert(kSmallChunkNodes / kChunkSmall <= kFusedChunkMax, "the small chunks' sums are always few");
  if (kW == kWordsSmall || n <= kFusedChunkMax) {
    hipLaunchKernelGGL((k_compact<kW, true>), g, dim3(kBlock), 0, s, d.present, d.chunk_sums, sc.uniq, unique_out, cn,
                       n, dd, tag, sc.gate);
  } else if constexpr (kW != kWordsSmall) {
    hipLaunchKernelGGL(k_chunk_scan, dim3(1), dim3(kBlock), 0, s, d.chunk_sums, n, cn, dd, tag, sc.gate);
    hipLaunchKernelGGL((k_compact<kW, false>), g, dim3(kBlock), 0, s, d.present, d.chunk_sums, sc.uniq, unique_out,
                       cn, n, dd, tag, sc.gate);
  }
}

void launch_dedup(const DevState &d, const int64_t *ids, uint64_t n, const int64_t *ann_ids, uint64_t ann_n,
                  Scratch &sc, int64_t *unique_out,
                  Counters *cn, DedupResult *dd, uint32_t tag, hipStream_t s) {
  const uint64_t work = n > ann_n ? n : ann_n;
  const unsigned g = grid_for(work, kBlock, kMaxGrid);
  hipLaunchKernelGGL(k_mark, dim3(g), dim3(kBlock), 0, s, ids, (uint32_t)n, ann_ids, (uint32_t)ann_n, d.N,
                     d.present, cn);
  if (d.N <= kSmallChunkNodes)
    launch_compaction<kWordsSmall>(d, sc, unique_out, cn, dd, tag, s);
  else
    launch_compaction<kWordsLarge>(d, sc, unique_out, cn, dd, tag, s);
}

// ------------------------------------------------------------ group by set
// Every thread of the block must call this; index[i] is the list index of a
// thread with pred[i] set (one atomic per block and list).
template <int kN>
__device__ __forceinline__ void block_append(const bool (&pred)[kN], uint32_t *const (&counter)[kN],
                                             uint32_t (&index)[kN]) {
  __shared__ uint32_t base[kN];
  uint32_t tot[kN];
  block_ranks(pred, index, tot);
#pragma unroll
  for (int i = 0; i < kN; ++i)
    if (threadIdx.x == 64u * (i % (kBlock / 64)) && tot[i]) base[i] = atomicAdd(counter[i], tot[i]);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kN; ++i) index[i] += base[i];
  __syncthreads();
}

__device__ __forceinline__ uint32_t block_append(bool pred, uint32_t *counter) {
  uint32_t index[1];
  block_append<1>({pred}, {counter}, index);
  return index[0];
}

// Sums of kN per-thread counters over the block, stored as this block's
// partials of slots [slot, slot + kN): one barrier for all of them.  With a
// block scan per counter and list, the walk of a 9 K-request batch took 12.6 us
// against 9.6, its resolve 10.2 against 7.9.  A kernel that calls this twice
// with one kN has a barrier in between.
template <int kN>
__device__ __forceinline__ void block_counts(const uint32_t (&v)[kN], uint32_t *part, int slot) {
  __shared__ uint32_t wsum[kN][kBlock / 64];
  uint32_t x[kN];
#pragma unroll
  for (int i = 0; i < kN; ++i) x[i] = v[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int i = 0; i < kN; ++i) x[i] += __shfl_xor(x[i], o);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int i = 0; i < kN; ++i) wsum[i][threadIdx.x >> 6] = x[i];
  __syncthreads();
  if (threadIdx.x < kN) {
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) t += wsum[threadIdx.x][w];
    part[(slot + threadIdx.x) * kMaxGrid + blockIdx.x] = t;
  }
}

// Per unique ID, right after the dedup: its set, its arrival order among the
// set's IDs, and what the batch-start state says about it.
//
// Misses known from the batch-start state are listed here, so that their rows
// start crossing the link while the rest of the metadata runs: a unique ID x
// that no way of its set holds at batch start is filled at its turn (only x
// itself inserts x), and with no entry for it in the victim buffer (FIFO: no
// ring entry naming x; queues: no entry in the queue of this iteration) the
// fill is a miss, whatever the walk decides.  The resolve, which finds the
// same outcome, leaves these out of its list.
//
// A set none of whose IDs is missing changes nothing in this gather, so its
// IDs' outcomes are settled by this probe alone; the others are marked for the
// walk (SetBatch::dirty holds 1 + the gather index).  Where nearly every row is
// resident this leaves nothing to group: 365 us per gather against 409 with
// every touched set walked (900 K requests, 235 K unique 2 KiB rows, pipelined);
// where nearly every set misses it costs nothing measurable.
//
// Bound by latency: a 128-byte set record and an atomic on the set's counter
// per unique ID, both in flight together.
//
// Returns whether this thread saw an ID that is not resident.
__device__ __forceinline__ bool probe(const DevState &d, const Scratch &sc, uint64_t t, const Counters *cn) {
  const uint32_t U = cn->n_unique;
  uint32_t c_early = 0;
  bool missed = false;
  for (uint32_t base = blockIdx.x * kBlock; base < U; base += gridDim.x * kBlock) {
    const uint32_t u = base + threadIdx.x;
    bool early = false;
    uint32_t x = 0;
    if (threadIdx.x == 0) sc.scan_part[base / kScanChunk] = 0;  // counted up by the walk
    if (u < U) {
      x = sc.uniq[u];
      const uint32_t s = set_index(x, d.S);
      const u32x4 *tp = reinterpret_cast<const u32x4 *>(d.sets[s].tag);
      const u32x4 a = tp[0], b = tp[1];
      sc.arrival[u] = atomicAdd(&d.batch[s].count, 1u);
      sc.uset[u] = s;
      uint32_t m = 0;  // the ways that hold x
#pragma unroll
      for (int w = 0; w < 4; ++w) m |= (a[w] == x ? 1u << w : 0u) | (b[w] == x ? 16u << w : 0u);
      if (m) {
        sc.slot[u] = s * kWays + (uint32_t)__builtin_ctz(m);
      } else {
        missed = true;
        d.batch[s].dirty = (uint32_t)t + 1u;
        bool entry = false;
        if (d.V) {
          const uint64_t vp = d.vpos[x];
          if (d.qmode)
            entry = (vp >> 32) == t + 1;
          else if (vp)
            entry = d.ring_tag[(vp - 1) % d.V] == x;
        }
        early = !entry;
      }
      sc.early[u] = early ? 1 : 0;
      c_early += early;
    }
    const uint32_t i = block_append(early, &sc.gate->n_early);
    if (early) {
      sc.host_list[i] = u;
      sc.host_src[i] = kSrcStore | x;
    }
  }
  block_counts<1>({c_early}, sc.stat_part, kStEarly);
  return missed;
}

__global__ __launch_bounds__(kBlock) void k_probe(const DevState d, Scratch sc, uint64_t t, const Counters *cn) {
  if (cn->err) return;
  (void)probe(d, sc, t, cn);
}

void launch_probe(const DevState &d, uint64_t n, uint64_t t, Scratch &sc, Counters *cn, StatGrids &grids,
                  hipStream_t s) {
  const unsigned g = grid_for(n, kBlock, kMaxGrid);
  hipLaunchKernelGGL(k_probe, dim3(g), dim3(kBlock), 0, s, d, sc, t, cn);
  grids.g[kStEarly] = g;
}

// Per touched set (its first arrival's thread): a segment for the IDs of a set
// to be walked, and its entry in the work list its size calls for; a settled
// set gets none.  Resets the set's counter.
__device__ __forceinline__ void seg_alloc(const DevState &d, const Scratch &sc, uint32_t t, Counters *cn) {
  const uint32_t U = cn->n_unique;
  __shared__ uint32_t boff, bwork;
  for (uint32_t base = blockIdx.x * kBlock; base < U; base += gridDim.x * kBlock) {
    const uint32_t u = base + threadIdx.x;
    uint32_t s = 0, k = 0;
    bool walk = false;
    if (u < U && sc.arrival[u] == 0) {
      s = sc.uset[u];
      const u32x4 v = *reinterpret_cast<const u32x4 *>(d.batch + s);  // count, dirty
      k = v.x;
      d.batch[s].count = 0;
      walk = v.y == t + 1u;
      if (!walk) d.batch[s].off = kSettled;
    }
    const bool small = walk && k <= kSmallSet;
    uint64_t tot;  // segment entries below 2^40, small sets above
    const uint64_t ex = block_exclusive_scan64((walk ? (uint64_t)k : 0u) | (small ? 1ull << 40 : 0ull), tot);
    if (threadIdx.x == 0 && tot) {
      boff = atomicAdd(&cn->seg_cursor, (uint32_t)tot);
      bwork = atomicAdd(&cn->n_work, (uint32_t)(tot >> 40));
    }
    __syncthreads();
    if (walk) {
      const WorkSet e{s, boff + (uint32_t)ex, k};
      d.batch[s].off = e.off;
      if (small)
        sc.work[bwork + (uint32_t)(ex >> 40)] = e;
      else if (k <= kMidSet)
        sc.work_mid[atomicAdd(&cn->n_mid, 1u)] = e;
      else
        sc.work_big[atomicAdd(&cn->n_big, 1u)] = e;
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kBlock) void k_seg_alloc(const DevState d, Scratch sc, uint32_t t, Counters *cn) {
  if (cn->err) return;
  seg_alloc(d, sc, t, cn);
}

// Per unique ID: the node's unique index (read by the inverse index), the
// per-ID state reset; then a hit for an ID of a settled set, else its entry in the set's segment, in arrival
// order.
__device__ __forceinline__ void place(const DevState &d, const Scratch &sc, const Counters *cn) {
  const uint32_t U = cn->n_unique;
  uint32_t c_hit = 0;
  for (uint32_t u = blockIdx.x * kBlock + threadIdx.x; u < U; u += gridDim.x * kBlock) {
    const uint32_t x = sc.uniq[u];
    const uint32_t off = d.batch[sc.uset[u]].off;
    d.uidx[x] = u;
    sc.flags[u] = 0;
    sc.dead[u] = 0;
    sc.fill_dst[u] = 0;
    if (off == kSettled) {
      sc.kind[u] = kKindHit;
      ++c_hit;
    } else {
      sc.ent[off + sc.arrival[u]] = u32x4{x, u, d.stat[x], 0};
    }
  }
  block_counts<1>({c_hit}, sc.stat_part, kStSettled);
}

__global__ __launch_bounds__(kBlock) void k_place(const DevState d, Scratch sc, const Counters *cn) {
  if (cn->err) return;
  place(d, sc, cn);
}

void launch_group_by_set(const DevState &d, uint64_t n, uint32_t t, Scratch &sc, Counters *cn, StatGrids &grids,
                         hipStream_t s) {
  const unsigned g = grid_for(n, kBlock, kMaxGrid);
  hipLaunchKernelGGL(k_seg_alloc, dim3(g), dim3(kBlock), 0, s, d, sc, t, cn);
  hipLaunchKernelGGL(k_place, dim3(g), dim3(kBlock), 0, s, d, sc, cn);
  grids.g[kStSettled] = g;
}

// ---------------------------------------------------------------- set walk
// Class of a resident line from its window bits: bit i is set while minibatch
// t + 1 + i is announced and not yet served.
__device__ __forceinline__ uint32_t class_from_bits(uint32_t m, uint32_t L, uint32_t T) {
  const uint32_t rel = m & ((1u << L) - 1u);
  if (rel == 0) return kClsNone;
  return (uint32_t)__builtin_ctz(rel) + 1u <= T ? kClsNear : kClsFar;
}

// Distance from gather t to the line's next announced use (1..L), or 0 when
// none of the next L minibatches names it.
__device__ __forceinline__ uint32_t dist_from_bits(uint32_t m, uint32_t L) {
  const uint32_t rel = m & ((1u << L) - 1u);
  return rel ? (uint32_t)__builtin_ctz(rel) + 1u : 0u;
}

// The update of the dynamic information (Sec. 4.2) with an update period U >
// 1, before every U-th gather: each resident line records 1 + its next reuse
// iteration from the announced-batch bits (0: none).  Skipped when the
// gather's IDs were rejected; the retry of the same gather runs it.
__global__ __launch_bounds__(kBlock) void k_refresh(const DevState d, uint32_t t, const Counters *cn) {
  if (cn->err) return;
  const uint64_t lines = d.S * kWays;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < lines; i += (uint64_t)gridDim.x * kBlock) {
    const uint32_t tag = d.sets[i / kWays].tag[i % kWays];
    uint32_t r = 0;
    if (tag != kEmpty) {
      const uint32_t dist = dist_from_bits(window_bits(d.win[tag], t), d.L);
      r = dist ? t + dist + 1u : 0u;
    }
    d.lreuse[i] = r;
  }
}

void launch_refresh(const DevState &d, uint32_t t, const Counters *cn, hipStream_t s) {
  hipLaunchKernelGGL(k_refresh, dim3(grid_for(d.S * kWays, kBlock, kMaxGrid)), dim3(kBlock), 0, s, d, t, cn);
}

// Class and next-reuse distance of a batch-start resident from the
// information recorded at the last update (update period U > 1): inserted at
// or after that update, or its recorded reuse has come -> recently inserted
// (distance 0); none recorded -> no reuse; else near or far by the distance.
__device__ __forceinline__ void class_from_record(uint32_t rec, uint32_t ins, uint32_t t, uint32_t t_upd, uint32_t T,
                                                  uint32_t &cls, uint32_t &dist) {
  dist = 0;
  if (ins >= t_upd) {
    cls = kClsRecent;
  } else if (rec == 0) {
    cls = kClsNone;
  } else if (rec - 1u <= t) {
    cls = kClsRecent;
  } else {
    dist = rec - 1u - t;
    cls = dist <= T ? kClsNear : kClsFar;
  }
}

// eviction level, lowest evicted first: none < far < recent < near, or with
// the victim ring on, far < none < recent < near
__device__ __forceinline__ uint32_t level_of(uint32_t cls, bool ring_on) {
  return (ring_on && cls <= kClsFar) ? (cls ^ 1u) : cls;
}

// Minimum of a 64-bit key over the 8 lanes of a set's lane group.
__device__ __forceinline__ uint64_t group_min(uint64_t v) {
#pragma unroll
  for (int o = 1; o < (int)kWays; o <<= 1) {
    const uint32_t lo = __shfl_xor((uint32_t)v, o, kWays);
    const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), o, kWays);
    const uint64_t w = ((uint64_t)hi << 32) | lo;
    v = w < v ? w : v;
  }
  return v;
}

// Orders stores and loads of the wave's LDS entries: the lanes of a wave run
// in lockstep and its LDS operations complete in order, so only the compiler
// has to be held back.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A set's IDs in ascending order, in LDS: entry j at index j * S.
template <uint32_t S>
struct SetEntries {
  uint32_t *x, *u, *st;
  __device__ __forceinline__ void get(uint32_t j, uint32_t &xo, uint32_t &uo, uint32_t &so) const {
    xo = x[j * S];
    uo = u[j * S];
    so = st[j * S];
  }
};

// Brings a segment of k <= 8 * G entries (arrival order) into LDS in ascending
// ID order, by G lanes of one wave (`l` this lane's number among them): each
// lane keeps up to eight entries in registers and ranks them against all k IDs.
template <uint32_t G, uint32_t S>
__device__ __forceinline__ void order_entries(const u32x4 *seg, uint32_t k, uint32_t l, const SetEntries<S> &e) {
  u32x4 v[8];
  uint32_t r[8];
#pragma unroll
  for (uint32_t q = 0; q < 8; ++q) {
    r[q] = 0;
    v[q] = u32x4{0, 0, 0, 0};
    if (l + q * G < k) {
      v[q] = seg[l + q * G];
      e.x[(l + q * G) * S] = v[q].x;
    }
  }
  wave_lds_fence();
  if (k > G) {
    for (uint32_t j = 0; j < k; ++j) {
      const uint32_t y = e.x[j * S];
#pragma unroll
      for (uint32_t q = 0; q < 8; ++q) r[q] += y < v[q].x ? 1u : 0u;
    }
  } else {
    for (uint32_t j = 0; j < k; ++j) r[0] += e.x[j * S] < v[0].x ? 1u : 0u;
  }
  wave_lds_fence();
#pragma unroll
  for (uint32_t q = 0; q < 8; ++q) {
    if (l + q * G < k) {
      e.x[r[q] * S] = v[q].x;
      e.u[r[q] * S] = v[q].y;
      e.st[r[q] * S] = v[q].z;
    }
  }
  wave_lds_fence();
}

// A set of more than kMidSet IDs: one block sorts its segment ascending with
// an LSD radix sort over 8-bit digits of the unique index, in O(k) per pass,
// ping-ponging between seg and seg_u.  Each pass: digit histogram in LDS,
// exclusive scan, then the scatter in index order, 256 entries at a time: an
// entry's place among the chunk's entries with the same digit comes from eight
// ballots per wave (the lanes whose digit matches) and the counts of the lower
// waves.  lds: (1 + kBlock / 64) * 256 words.
__device__ __forceinline__ void sort_big_segment(const DevState &d, const Scratch &sc, uint32_t off, uint32_t k,
                                                 uint32_t U, uint32_t *lds) {
  const uint32_t bits = U > 1 ? 32u - (uint32_t)__builtin_clz(U - 1u) : 1u;
  const uint32_t passes = (bits + 7u) / 8u;
  uint32_t *base = lds;
  uint32_t(*wcnt)[256] = reinterpret_cast<uint32_t(*)[256]>(lds + 256);
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  const uint64_t lt = lane ? (~0ull >> (64u - lane)) : 0ull;
  uint32_t *src = sc.seg + off, *dst = sc.seg_u + off;
  for (uint32_t j = threadIdx.x; j < k; j += kBlock) src[j] = sc.ent[off + j].y;
  __syncthreads();
  for (uint32_t p = 0; p < passes; ++p) {
    const uint32_t shift = 8u * p;
    base[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < k; j += kBlock) atomicAdd(&base[(src[j] >> shift) & 255u], 1u);
    __syncthreads();
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan(base[threadIdx.x], tot);
    __syncthreads();
    base[threadIdx.x] = ex;
    for (uint32_t c0 = 0; c0 < k; c0 += kBlock) {
#pragma unroll
      for (int w = 0; w < kBlock / 64; ++w) wcnt[w][threadIdx.x] = 0;
      __syncthreads();
      const uint32_t j = c0 + threadIdx.x;
      const bool valid = j < k;
      const uint32_t v = valid ? src[j] : 0u;
      const uint32_t dg = (v >> shift) & 255u;
      uint64_t m = __ballot(valid);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const bool on = (dg >> bit) & 1u;
        const uint64_t bb = __ballot(valid && on);
        m &= on ? bb : ~bb;
      }
      if (valid && (m & lt) == 0) wcnt[wid][dg] = (uint32_t)__popcll(m);
      __syncthreads();
      if (valid) {
        uint32_t r = base[dg] + (uint32_t)__popcll(m & lt);
        for (uint32_t w = 0; w < wid; ++w) r += wcnt[w][dg];
        dst[r] = v;
      }
      __syncthreads();
      uint32_t add = 0;
#pragma unroll
      for (int w = 0; w < kBlock / 64; ++w) add += wcnt[w][threadIdx.x];
      base[threadIdx.x] += add;
    }
    __syncthreads();
    uint32_t *tmp = src;
    src = dst;
    dst = tmp;
  }
  // the sorted indices are in src
  for (uint32_t j = threadIdx.x; j < k; j += kBlock) {
    const uint32_t u = src[j];
    const uint32_t x = sc.uniq[u];
    sc.ent[off + j] = u32x4{x, u, d.stat[x], 0};
  }
  __syncthreads();
}

struct WalkCounts {
  uint32_t hit = 0, fill = 0, evict = 0, enq = 0, drop = 0, fin = 0;
};

// One set walked by a group of 8 lanes, lane w owning way w.  The group walks
// the set's k IDs in ascending order (the per-set order of the definition);
// `get(j, x, u, st)` gives the j-th to all its lanes.  Each step is a ballot
// for the tag probe, a ballot for an empty way, and on a full
// set the policy's victim: for the hybrid order (Sec. 4.2) a 3-step shuffle
// minimum of (level, static score, way); for the evaluation's ablations
// (Sec. 5) the minimum of (static score, way), of (no announced use first,
// then the furthest next use; way), or the set's round-robin pointer.
//
// A way's line is loaded before the set's IDs are ordered, so that the loads are
// under way together.  What its class is computed from is not: reading every
// line's window bits ahead, needed or not, slowed the host fetch beside the
// walk by 1 % (pipelined 1M-node stream, 4545 us against 4486 for 8 gathers).
struct Way {
  uint32_t tag, st, ins;
};
__device__ __forceinline__ Way load_way(const DevState &d, uint32_t s, uint32_t w) {
  const SetRec *rec = d.sets + s;
  return Way{rec->tag[w], rec->stat[w], rec->ins[w]};
}

template <int P, typename Get>
__device__ __forceinline__ void walk_set(const DevState &d, const Scratch &sc, uint32_t t, uint32_t s, uint32_t k,
                                         const Way &way, uint32_t lane, WalkCounts &c, const Get &get) {
  const bool ring_on = d.V > 0;
  const uint32_t recent_lvl = level_of(kClsRecent, ring_on);
  const uint32_t w = lane & (kWays - 1);   // the way this lane owns
  const uint32_t gsh = lane & ~(kWays - 1);  // first lane of the group in the wave
  const bool lead = w == 0;
  SetRec *rec = d.sets + s;
  uint32_t tag = way.tag, st = way.st, ins = way.ins;
  uint32_t cls = kClsNone, lvl = 0, dist = 0;
  bool known = false;  // class (and next-use distance) of this way for this gather computed
  uint32_t rr = 0;     // round-robin pointer (the record holds its complement)
  if constexpr (P == kPolicyRoundRobin) rr = ~rec->rr_inv & (kWays - 1);
  const uint32_t rr0 = rr;
  int32_t last = -1;   // unique index of this way's last fill
  bool dirty = false;
  // the way's batch-start line, and the unique index whose fill sent it to the
  // victim ring (only batch-start lines go there): an ID requested later in
  // the batch than its line was evicted finds its entry through these
  const uint32_t tag0 = tag;
  uint32_t sent = kEmpty;
  const bool fifo = ring_on && !d.qmode;
  for (uint32_t j = 0; j < k; ++j) {
    uint32_t x, u, xs;
    get(j, x, u, xs);
    const uint32_t hitm = (uint32_t)(__ballot(tag == x) >> gsh) & 0xffu;
    if (hitm) {
      if (lead) {
        sc.kind[u] = kKindHit;
        sc.slot[u] = s * kWays + (uint32_t)__builtin_ctz(hitm);
        ++c.hit;
      }
      continue;
    }
    dirty = true;
    const uint32_t emptym = (uint32_t)(__ballot(tag == kEmpty) >> gsh) & 0xffu;
    uint32_t pick, z = kEmpty;
    uint8_t f = 0;
    if (fifo) {
      const uint32_t em = (uint32_t)(__ballot(sent != kEmpty && tag0 == x) >> gsh) & 0xffu;
      const uint32_t e = __shfl(sent, em ? (int)__builtin_ctz(em) : 0, kWays);
      if (lead) sc.this_enq[u] = em ? e : kEmpty;
    }
    if (emptym) {
      pick = (uint32_t)__builtin_ctz(emptym);
    } else {
      if (!known) {  // batch-start resident
        if (d.U > 1) {  // from the information recorded at the last update
          class_from_record(d.lreuse[(uint64_t)s * kWays + w], ins, t, t - t % d.U, d.T, cls, dist);
        } else {        // exact: from its announced-use bits
          const uint32_t m = window_bits(d.win[tag], t);
          cls = (ins == t) ? kClsRecent : class_from_bits(m, d.L, d.T);
          if (P == kPolicyDynamic || d.qmode) dist = dist_from_bits(m, d.L);
        }
        lvl = level_of(cls, ring_on);
        known = true;
      }
      if constexpr (P == kPolicyHybrid) {
        pick = (uint32_t)(group_min(((uint64_t)lvl << 35) | ((uint64_t)st << 3) | w) & 7u);
      } else if constexpr (P == kPolicyStatic) {
        pick = (uint32_t)(group_min(((uint64_t)st << 3) | w) & 7u);
      } else if constexpr (P == kPolicyDynamic) {
        pick = (uint32_t)(group_min((uint64_t)((dist ? 32u - dist : 0u) << 3) | w) & 7u);
      } else {
        pick = rr;
        rr = (rr + 1u) & (kWays - 1);
      }
      z = __shfl(tag, (int)pick, kWays);
      const uint32_t pc = __shfl(cls, (int)pick, kWays);
      const uint32_t pd = __shfl(dist, (int)pick, kWays);
      const bool enq = ring_on && (pc == kClsFar || pc == kClsNear);
      if (enq && w == pick) sent = u;
      if (lead) {
        ++c.evict;
        if (enq) {
          f = (uint8_t)(kFlagEnqueue | (pd << kFlagDistShift));
          ++c.enq;
          if (fifo) atomicAdd(&sc.scan_part[u / kScanChunk], 1u);
        } else {
          ++c.drop;
        }
      }
    }
    if (lead) {
      ++c.fill;
      sc.kind[u] = kKindFill;
      sc.slot[u] = s * kWays + pick;
      sc.evicted[u] = z;
      sc.flags[u] = f;
    }
    if (w == pick) {
      tag = x;
      st = xs;
      ins = t;
      cls = kClsRecent;
      lvl = recent_lvl;
      dist = 0;  // a line inserted by this gather has no dynamic information yet
      known = true;
      last = (int32_t)u;
    }
  }
  if (last >= 0) {  // the way's final occupant refills the cache row
    sc.fill_dst[last] = s * kWays + w + 1;
    ++c.fin;
  }
  if (dirty) {
    rec->tag[w] = tag;
    rec->stat[w] = st;
    rec->ins[w] = ins;
  }
  if constexpr (P == kPolicyRoundRobin)
    if (lead && rr != rr0) rec->rr_inv = ~rr;
}

// The sets to walk, by size: more than kMidSet IDs, a block sorts the segment
// in memory and its first 8 lanes walk it; more than kSmallSet, a wave orders
// the IDs in LDS (512 entries, 6 KB per wave) and its first 8 lanes walk them;
// the others, 8 lanes each, the wave's LDS shared by its 8 groups (64 entries
// each).  Ordering here instead of in kernels of its own (a rank pass that
// loaded every segment k times, and a sort launched for the large sets whether
// there were any or not) took the probe, the grouping and the walk from eight
// launches to four: a blocking gather of 250 requests 144 -> 135 us, of 9 K
// requests 189 -> 171 us.
template <int P>
__device__ __forceinline__ void walk_sets(const DevState &d, const Scratch &sc, uint32_t t, const Counters *cn) {
  __shared__ uint32_t lds[3 * kMidSet * (kBlock / 64)];
  static_assert(sizeof(lds) >= (1 + kBlock / 64) * 256 * 4, "the large-set sort works in the same LDS");
  static_assert(kMidSet == 8 * 64 && kSmallSet == 8 * kWays, "eight entries per ordering lane");
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  WalkCounts c;
  for (uint32_t i = blockIdx.x; i < cn->n_big; i += gridDim.x) {
    const WorkSet e = sc.work_big[i];
    sort_big_segment(d, sc, e.off, e.k, cn->n_unique, lds);
    if (threadIdx.x < kWays) {
      u32x4 v{};  // entry (j & ~7) + lane, loaded 8 at a time
      const Way way = load_way(d, e.set, lane);
      walk_set<P>(d, sc, t, e.set, e.k, way, lane, c, [&](uint32_t j, uint32_t &x, uint32_t &u, uint32_t &st) {
        if ((j & (kWays - 1)) == 0 && j + lane < e.k) v = sc.ent[e.off + j + lane];
        const int src = (int)(j & (kWays - 1));
        x = __shfl(v.x, src, kWays);
        u = __shfl(v.y, src, kWays);
        st = __shfl(v.z, src, kWays);
      });
    }
    __syncthreads();
  }
  uint32_t *wl = lds + 3 * kMidSet * wid;  // this wave's
  const SetEntries<1> mid{wl, wl + kMidSet, wl + 2 * kMidSet};
  const uint32_t waves = gridDim.x * (kBlock / 64);
  for (uint32_t i = blockIdx.x * (kBlock / 64) + wid; i < cn->n_mid; i += waves) {
    const WorkSet e = sc.work_mid[i];
    const Way way = load_way(d, e.set, lane & (kWays - 1));
    order_entries<64>(sc.ent + e.off, e.k, lane, mid);
    if (lane < kWays)
      walk_set<P>(d, sc, t, e.set, e.k, way, lane, c, [&](uint32_t j, uint32_t &x, uint32_t &u, uint32_t &st) {
        mid.get(j, x, u, st);
      });
    wave_lds_fence();
  }
  // the wave's groups interleave their entries, so that they read different
  // LDS banks at the same step
  const uint32_t g0 = lane / kWays;
  const SetEntries<kWays> small{wl + g0, wl + kMidSet + g0, wl + 2 * kMidSet + g0};
  const uint32_t groups = gridDim.x * (kBlock / kWays);
  const uint32_t nw = cn->n_work;
  for (uint32_t i = blockIdx.x * (kBlock / kWays) + (threadIdx.x / kWays); i < nw; i += groups) {
    const WorkSet e = sc.work[i];
    const Way way = load_way(d, e.set, lane & (kWays - 1));
    order_entries<kWays>(sc.ent + e.off, e.k, lane & (kWays - 1), small);
    walk_set<P>(d, sc, t, e.set, e.k, way, lane, c, [&](uint32_t j, uint32_t &x, uint32_t &u, uint32_t &st) {
      small.get(j, x, u, st);
    });
    wave_lds_fence();
  }
  static_assert(kStFinal == kStHits + 5, "the walk's counters are consecutive");
  block_counts<6>({c.hit, c.fill, c.evict, c.enq, c.drop, c.fin}, sc.stat_part, kStHits);
}

template <int P>
__global__ __launch_bounds__(kBlock) void k_set_walk(const DevState d, Scratch sc, uint32_t t, Counters *cn) {
  if (cn->err) return;
  walk_sets<P>(d, sc, t, cn);
}

#ifndef LSM_WALK_GRID
#define LSM_WALK_GRID 4096  // set-walk blocks of 32 lane groups: enough sets in flight to hide the record loads
#endif
void launch_set_walk(const DevState &d, uint64_t n, uint32_t t, Scratch &sc, Counters *cn, StatGrids &grids,
                     hipStream_t s) {
  const unsigned g = grid_for(n * kWays, kBlock, LSM_WALK_GRID);
  switch (d.policy) {
    case kPolicyStatic:
      hipLaunchKernelGGL(k_set_walk<kPolicyStatic>, dim3(g), dim3(kBlock), 0, s, d, sc, t, cn);
      break;
    case kPolicyDynamic:
      hipLaunchKernelGGL(k_set_walk<kPolicyDynamic>, dim3(g), dim3(kBlock), 0, s, d, sc, t, cn);
      break;
    case kPolicyRoundRobin:
      hipLaunchKernelGGL(k_set_walk<kPolicyRoundRobin>, dim3(g), dim3(kBlock), 0, s, d, sc, t, cn);
      break;
    default:
      hipLaunchKernelGGL(k_set_walk<kPolicyHybrid>, dim3(g), dim3(kBlock), 0, s, d, sc, t, cn);
  }
  for (int st = kStHits; st <= kStFinal; ++st) grids.g[st] = g;
}

// ---------------------------------------------------------- ring sequences
// The exclusive scan of the enqueue flags in ascending-ID order gives each
// enqueue its ring sequence number.  The walk counts the enqueues per chunk of
// kScanChunk unique IDs; the resolve adds up the counts of the chunks before
// its own, unless there are more than kFusedScanMax of them: then this one
// block scans them first.
__global__ __launch_bounds__(kBlock) void k_scan_top(uint32_t *part, Counters *cn) {
  if (cn->err) return;
  const uint32_t U = cn->n_unique;
  const uint32_t nb = (U + kScanChunk - 1) / kScanChunk;
  constexpr int kPer = 8;
  uint32_t carry = 0;
  for (uint32_t base = 0; base < nb; base += kBlock * kPer) {
    const uint32_t i = base + threadIdx.x * kPer;
    uint32_t v[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) sum += v[q] = i + q < nb ? part[i + q] : 0u;
    uint32_t tot;
    uint32_t run = carry + block_exclusive_scan(sum, tot);
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (i + q < nb) part[i + q] = run;
      run += v[q];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) cn->enq_total = carry;
}

// Enqueue flags set in [a, b).
__device__ __forceinline__ uint32_t count_enqueues(const uint8_t *flags, uint32_t a, uint32_t b) {
  uint32_t c = 0;
  for (; a < b && (a & 3u); ++a) c += flags[a] & kFlagEnqueue;
  for (; a + 4 <= b; a += 4)
    c += (uint32_t)__popc(*reinterpret_cast<const uint32_t *>(flags + a) & (0x01010101u * kFlagEnqueue));
  for (; a < b; ++a) c += flags[a] & kFlagEnqueue;
  return c;
}

// At most this many chunk counts are added up by each block of the resolve (16
// loads per thread); beyond, one block scans them first.
constexpr uint32_t kFusedScanMax = 4096;

// Where the resolve finds the enqueue counts of the chunks.
enum : int { kScanNone, kScanCounts, kScanOffsets };

// The first enqueue of each of nb <= kFusedScanMax chunks, from their counts,
// into LDS.
__device__ __forceinline__ void chunk_offsets(const uint32_t *cnt, uint32_t nb, uint32_t *offs) {
  const uint32_t per = (nb + kBlock - 1) / kBlock, j0 = threadIdx.x * per, j1 = j0 + per < nb ? j0 + per : nb;
  uint32_t sum = 0, tot;
  for (uint32_t j = j0; j < j1; ++j) sum += cnt[j];
  uint32_t run = block_exclusive_scan(sum, tot);
  for (uint32_t j = j0; j < j1; ++j) {
    offs[j] = run;
    run += cnt[j];
  }
  __syncthreads();
}

// Whether at most V lines were sent to the ring from the fill of unique index
// e up to, not including, that of u > e (the entry e made is then still there
// at u's turn).  before: u's rank among the enqueues of its chunk; first: each
// chunk's first enqueue.
__device__ __forceinline__ bool at_most_enqueued(const Scratch &sc, uint64_t V, uint32_t e, uint32_t u,
                                                 const uint32_t *first, uint32_t before) {
  const uint32_t ce = e / kScanChunk, cu = u / kScanChunk;
  if (ce == cu) return count_enqueues(sc.flags, e, u) <= V;
  return (uint64_t)before + count_enqueues(sc.flags, e, (ce + 1) * kScanChunk) + (first[cu] - first[ce + 1]) <= V;
}

// ------------------------------------------------------------ victim queues
// Queue mode (Sec. 4.3.1): an enqueue candidate u goes to the queue of its
// line's next reuse iteration j = t + distance (slot j mod (L+1)) at the
// position the queue's counter gives in ascending-u order, or is dropped when
// that position is C or more.  Per-block counts per slot, one block's scan of
// them per slot, then each candidate's rank among its block's candidates for
// the same slot (one ballot per slot).
__device__ __forceinline__ bool q_candidate(const Scratch &sc, uint32_t u, uint32_t U, uint64_t t, uint32_t slots,
                                            uint32_t &key) {
  if (u >= U || sc.kind[u] != kKindFill) return false;
  const uint32_t f = sc.flags[u];
  if (!(f & kFlagEnqueue)) return false;
  key = (uint32_t)((t + (f >> kFlagDistShift)) % slots);
  return true;
}

__global__ __launch_bounds__(kBlock) void k_qcount(const DevState d, Scratch sc, uint64_t t, const Counters *cn) {
  if (cn->err) return;
  const uint32_t U = cn->n_unique;
  const uint32_t slots = d.L + 1;
  const uint32_t nb = (U + kBlock - 1) / kBlock;
  __shared__ uint32_t cnt[kMaxQueues];
  for (uint32_t b = blockIdx.x; b < nb; b += gridDim.x) {
    if (threadIdx.x < kMaxQueues) cnt[threadIdx.x] = 0;
    __syncthreads();
    uint32_t key = 0;
    if (q_candidate(sc, b * kBlock + threadIdx.x, U, t, slots, key)) atomicAdd(&cnt[key], 1u);
    __syncthreads();
    if (threadIdx.x < slots) sc.qpart[(uint64_t)threadIdx.x * nb + b] = cnt[threadIdx.x];
    __syncthreads();
  }
}

// One block: per slot, the exclusive scan of the per-block counts, then the
// slot's placements (up to C entries in all) and the counters the finish and
// the host read.  The queue counters advance here; the placement kernel reads
// the values from before this gather from the call's counters.
__global__ __launch_bounds__(kBlock) void k_qtop(const DevState d, Scratch sc, Counters *cn) {
  if (cn->err) return;
  const uint32_t U = cn->n_unique;
  const uint32_t slots = d.L + 1;
  const uint32_t nb = (U + kBlock - 1) / kBlock;
  __shared__ uint32_t tot[kMaxQueues];
  for (uint32_t k = 0; k < slots; ++k) {
    uint32_t carry = 0;
    uint32_t *row = sc.qpart + (uint64_t)k * nb;
    for (uint32_t base = 0; base < nb; base += kBlock) {
      const uint32_t i = base + threadIdx.x;
      const uint32_t v = i < nb ? row[i] : 0u;
      uint32_t blk;
      const uint32_t ex = block_exclusive_scan(v, blk);
      if (i < nb) row[i] = carry + ex;
      carry += blk;
    }
    if (threadIdx.x == 0) tot[k] = carry;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t placed_all = 0, over = 0;
    for (uint32_t k = 0; k < slots; ++k) {
      const uint32_t before = d.qcount[k];
      const uint32_t room = (uint32_t)d.C - before;
      const uint32_t placed = tot[k] < room ? tot[k] : room;
      cn->q_before[k] = before;
      cn->q_placed[k] = placed;
      d.qcount[k] = before + placed;
      placed_all += placed;
      over += tot[k] - placed;
    }
    cn->enq_total = placed_all;
    cn->q_overflow = over;
  }
}

// Position of every candidate: the slot's entries before this gather, the
// candidates of lower blocks and those of lower lanes of this block.  A placed
// entry records its tag and its node's latest entry, and lists its row for
// staging: the gather's placements are staged slot by slot, in position order.
// Runs after the resolve kernel, which reads the nodes' entries from before
// this gather.
__global__ __launch_bounds__(kBlock) void k_qplace(const DevState d, Scratch sc, uint64_t t, Counters *cn) {
  if (cn->err) return;
  const uint32_t U = cn->n_unique;
  const uint32_t slots = d.L + 1;
  const uint32_t nb = (U + kBlock - 1) / kBlock;
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  __shared__ uint32_t wcnt[kBlock / 64][kMaxQueues];
  __shared__ uint32_t off[kMaxQueues];
  if (threadIdx.x == 0) {
    uint32_t o = 0;
    for (uint32_t k = 0; k < slots; ++k) {
      off[k] = o;
      o += cn->q_placed[k];
    }
  }
  __syncthreads();
  uint32_t c_copy = 0;
  for (uint32_t b = blockIdx.x; b < nb; b += gridDim.x) {
    const uint32_t u = b * kBlock + threadIdx.x;
    uint32_t key = 0;
    const bool cand = q_candidate(sc, u, U, t, slots, key);
    uint32_t rank = 0;
    for (uint32_t k = 0; k < slots; ++k) {
      const uint64_t m = __ballot(cand && key == k);
      if (cand && key == k) rank = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
      if (lane == 0) wcnt[wid][k] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    bool stage = false;
    uint32_t pos = 0;
    if (cand) {
      for (uint32_t w = 0; w < wid; ++w) rank += wcnt[w][key];
      const uint32_t before = cn->q_before[key];
      const uint64_t p = (uint64_t)before + sc.qpart[(uint64_t)key * nb + b] + rank;
      if (p < d.C) {
        const uint32_t z = sc.evicted[u];
        const uint64_t j = t + (sc.flags[u] >> kFlagDistShift);
        d.ring_tag[key * d.C + p] = z;
        d.vpos[z] = ((j + 1) << 32) | p;
        pos = off[key] + (uint32_t)(p - before);
        stage = true;
        ++c_copy;
      }
    }
    const uint32_t i = block_append(stage, &sc.gate->n_stage);
    if (stage) {
      sc.stage.src[i] = sc.slot[u];
      sc.stage.dst[i] = pos;
    }
  }
  block_counts<1>({c_copy}, sc.stat_part, kStEnqCopy);
}

// Victim-ring probe of every fill and the row source of every unique ID.  Builds
// the gather's row-copy lists: the rest of the host fetch's (rows from pinned
// host memory, after the early misses; dense, in arbitrary order), the hit
// copy's (one entry per unique ID: its HBM row, or none) and the fills' (each
// way's final occupant; dense, in arbitrary order).
//
// Ring mode: the enqueues' sequence numbers are scanned here (`scan`): each
// block adds up all chunks' counts once, those before its own chunk apart, and
// scans its own chunk's flags.  With the scan in two kernels of its own and a
// scattered record of every evicted line requested later in the batch (which
// the walk now knows by itself), a blocking gather of 9 K requests took 171 us
// against 160.
//
// A batch that enqueues more than V may have pushed out an entry it made
// itself before its line is requested.  A block that meets such a request
// first scans all chunks' counts into LDS: gathers of 1 M unique IDs with 50 K
// enqueues for a ring of 2000 took 1046 us where each such request added up
// the counts between by itself, now 682.
__device__ __forceinline__ void resolve(const DevState &d, const Scratch &sc, uint64_t t, uint8_t *outcome, int scan,
                                        Counters *cn) {
  static_assert(kScanChunk == kBlock, "one chunk of enqueue flags per block pass");
  __shared__ uint32_t offs[kFusedScanMax];
  const uint32_t U = cn->n_unique;
  const uint64_t tail0 = d.tail[0], tail_prev = d.tail[1];
  uint32_t enq_total = scan == kScanOffsets ? cn->enq_total : 0u;
  // the previous gather's surviving entries, [q_lo_prev, tail0), were staged
  // in that order in its staging buffer
  const uint64_t q_lo_prev = tail0 - ((tail0 - tail_prev) < d.V ? (tail0 - tail_prev) : d.V);
  const uint64_t stage_prev = d.stage_row0 + ((t + 1u) & 1u) * d.stage_rows;
  const uint32_t n_early = sc.gate->n_early;  // the list's first entries, written by k_probe
  uint32_t c_vhit = 0, c_miss = 0, c_hbm = 0, c_host = 0, c_vring = 0, c_vstaged = 0, c_vsame = 0;
  for (uint32_t base = blockIdx.x * kBlock; base < U; base += gridDim.x * kBlock) {
    const uint32_t u = base + threadIdx.x;
    bool from_host = false, from_hbm = false, refill = false;
    uint64_t code = 0;
    uint32_t fd = 0;
    uint32_t rank = 0, enq_before = 0;  // u's enqueues before it: in its chunk, in the batch
    if (scan != kScanNone) {
      const uint32_t chunk = base / kScanChunk;
      uint32_t off;
      if (scan == kScanCounts) {
        const uint32_t nb = (U + kScanChunk - 1) / kScanChunk;
        uint64_t v = 0, sum;  // all chunks' enqueues, those before this chunk in the upper half
        for (uint32_t j = threadIdx.x; j < nb; j += kBlock) {
          const uint64_t p = sc.scan_part[j];
          v += p | (j < chunk ? p << 32 : 0ull);
        }
        (void)block_exclusive_scan64(v, sum);
        enq_total = (uint32_t)sum;
        off = (uint32_t)(sum >> 32);
        if (base == 0 && threadIdx.x == 0) cn->enq_total = enq_total;
      } else {
        off = sc.scan_part[chunk];
      }
      uint32_t ranks[1], tot[1];
      block_ranks<1>({u < U && (sc.flags[u] & kFlagEnqueue)}, ranks, tot);
      rank = ranks[0];
      enq_before = off + rank;
      if (u < U) sc.enq_before[u] = enq_before;
      if (scan == kScanCounts && enq_total > d.V) {
        const uint32_t e = u < U && sc.kind[u] == kKindFill ? sc.this_enq[u] : kEmpty;
        if (__syncthreads_or(e != kEmpty && u - e > d.V))
          chunk_offsets(sc.scan_part, (U + kScanChunk - 1) / kScanChunk, offs);
      }
    }
    const uint64_t tail_end = tail0 + enq_total;
    if (u < U) {
      const uint8_t kind = sc.kind[u];
      uint8_t oc = 0;  // LSMGNN_HIT
      if (kind == kKindHit) {
        code = kSrcHbm | sc.slot[u];
        ++c_hbm;
      } else if (sc.early[u]) {  // a miss already listed (its row is on its way)
        ++c_miss;
        oc = 2;  // LSMGNN_MISS
        code = kSrcStore;
      } else if (d.qmode) {
        // queue mode: a victim hit iff the node's latest entry is in the queue
        // of this iteration, whose rows were prefetched into buffer t & 1
        const uint32_t x = sc.uniq[u];
        const uint64_t vp = d.V ? d.vpos[x] : 0;
        if ((vp >> 32) == t + 1) {
          ++c_vhit;
          oc = 1;  // LSMGNN_VICTIM_HIT
          code = kSrcHbm | (d.S * kWays + (t & 1) * d.C + (vp & 0xffffffffu));
          ++c_hbm;
        } else {
          ++c_miss;
          oc = 2;  // LSMGNN_MISS
          code = kSrcStore | x;
          ++c_host;
        }
      } else {
        const uint32_t x = sc.uniq[u];
        uint64_t q = 0;
        bool live = false;
        const uint32_t e = d.V ? sc.this_enq[u] : kEmpty;
        const bool same_batch = e != kEmpty;
        if (same_batch) {
          live = enq_total <= d.V || u - e <= d.V ||
                 at_most_enqueued(sc, d.V, e, u, scan == kScanOffsets ? sc.scan_part : offs, rank);
        } else if (d.V) {
          const uint64_t vp = d.vpos[x];
          if (vp) {
            q = vp - 1;
            live = d.ring_tag[q % d.V] == x && q + d.V >= tail0 + enq_before;
          }
        }
        if (live) {
          ++c_vhit;
          oc = 1;  // LSMGNN_VICTIM_HIT
          if (same_batch) {
            // evicted earlier in this batch: its row is still in the cache slot
            // the evicting fill took, which no copy has overwritten yet
            code = kSrcHbm | sc.slot[e];
            sc.dead[e] = 1;
            ++c_hbm;
            ++c_vsame;
          } else {
            // The entry leaves the ring: removed now, unless an enqueue of this
            // batch takes its slot anyway.  Its row is the victim buffer's:
            //  - an entry of the previous gather is read from that gather's
            //    staging rows in HBM (its ring write may still be running);
            //  - an older one from the pinned ring.  The ring rows it is read
            //    from are overwritten only by this gather's ring write, which
            //    the runtime queues after this gather's host fetch.
            if (q + d.V >= tail_end) d.ring_tag[q % d.V] = kEmpty;
            if (q >= tail_prev) {
              code = kSrcHbm | (stage_prev + (q - q_lo_prev));
              ++c_hbm;
              ++c_vstaged;
            } else {
              code = kSrcRing | (q % d.V);
              ++c_host;
              ++c_vring;
            }
          }
        } else {
          ++c_miss;
          oc = 2;  // LSMGNN_MISS
          code = kSrcStore | x;
          ++c_host;
        }
      }
      from_host = (code & ~kSrcIndex) != kSrcHbm && !sc.early[u];
      from_hbm = (code & ~kSrcIndex) == kSrcHbm;
      fd = sc.fill_dst[u];
      refill = fd != 0;
      sc.oc[u] = oc;
      if (outcome) outcome[u] = oc;
      // the hit copy's list is indexed by unique index (its destination row),
      // so the copy writes the output rows in order
      sc.hbm.src[u] = from_hbm ? (uint32_t)(code & kSrcIndex) : kNoRow;
    }
    uint32_t index[2];
    block_append<2>({from_host, refill}, {&sc.gate->n_host, &sc.gate->n_fill}, index);
    if (from_host) {
      sc.host_list[n_early + index[0]] = u;
      sc.host_src[n_early + index[0]] = code;
    }
    if (refill) {
      sc.fill.src[index[1]] = u;
      sc.fill.dst[index[1]] = fd - 1;
    }
  }
  static_assert(kStVhSame == kStVictimHits + 6, "the resolve's counters are consecutive");
  block_counts<7>({c_vhit, c_miss, c_hbm, c_host, c_vring, c_vstaged, c_vsame}, sc.stat_part, kStVictimHits);
}

__global__ __launch_bounds__(kBlock) void k_resolve(const DevState d, Scratch sc, uint64_t t, uint8_t *outcome,
                                                    int scan, Counters *cn) {
  if (cn->err) return;
  resolve(d, sc, t, outcome, scan, cn);
}

// One pass over the raw requests: the inverse index (if asked for), and the
// outcome counts (each request takes its unique ID's outcome).
__device__ __forceinline__ void request_counts(const DevState &d, const Scratch &sc, const int64_t *ids, uint32_t n,
                                               int64_t *inv) {
  uint32_t c_hit = 0, c_vhit = 0;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const uint32_t u = d.uidx[ids[i]];
    if (inv) inv[i] = (int64_t)u;
    const uint8_t o = sc.oc[u];
    c_hit += o == 0;   // LSMGNN_HIT
    c_vhit += o == 1;  // LSMGNN_VICTIM_HIT
  }
  static_assert(kStReqVictimHits == kStReqHits + 1, "the requests' counters are consecutive");
  block_counts<2>({c_hit, c_vhit}, sc.stat_part, kStReqHits);
}

__global__ __launch_bounds__(kBlock) void k_request_counts(const DevState d, Scratch sc, const int64_t *ids,
                                                           uint32_t n, int64_t *inv, const Counters *cn) {
  if (cn->err) return;
  request_counts(d, sc, ids, n, inv);
}

// Ring bookkeeping for this batch's enqueues; lists the row copies of the
// entries that are still in the ring at the end of the batch.  Those entries
// have the sequence numbers [q_lo, tail_end), q_lo = tail_end - min(E, V) for E
// enqueues, and their rows are staged in that order (entries removed again in
// this batch leave a hole that nothing reads).
__device__ __forceinline__ void enqueue_entries(const DevState &d, const Scratch &sc, const Counters *cn) {
  const uint32_t U = cn->n_unique;
  const uint64_t tail0 = d.tail[0];
  const uint64_t E = cn->enq_total;
  const uint64_t tail_end = tail0 + E;
  const uint64_t q_lo = tail_end - (E < d.V ? E : d.V);
  uint32_t c_copy = 0;
  for (uint32_t base = blockIdx.x * kBlock; base < U; base += gridDim.x * kBlock) {
    const uint32_t u = base + threadIdx.x;
    bool stage = false;
    uint32_t pos = 0;
    if (u < U && sc.kind[u] == kKindFill && (sc.flags[u] & kFlagEnqueue)) {
      const uint64_t q = tail0 + sc.enq_before[u];
      const uint32_t z = sc.evicted[u];
      d.vpos[z] = q + 1;
      if (q + d.V >= tail_end) {
        if (sc.dead[u]) {
          d.ring_tag[q % d.V] = kEmpty;
        } else {
          d.ring_tag[q % d.V] = z;
          stage = true;
          pos = (uint32_t)(q - q_lo);
          ++c_copy;
        }
      }
    }
    const uint32_t i = block_append(stage, &sc.gate->n_stage);
    if (stage) {
      sc.stage.src[i] = sc.slot[u];
      sc.stage.dst[i] = pos;
    }
  }
  block_counts<1>({c_copy}, sc.stat_part, kStEnqCopy);
}

__global__ __launch_bounds__(kBlock) void k_enq_finalize(const DevState d, Scratch sc, const int64_t *ids, uint32_t n,
                                                         int64_t *inv, Counters *cn) {
  if (cn->err) return;
  enqueue_entries(d, sc, cn);
  // the pass over the requests, in the same launch
  request_counts(d, sc, ids, n, inv);
}

void launch_ring_resolve(const DevState &d, uint64_t n, uint64_t t, Scratch &sc, uint8_t *outcome, Counters *cn,
                         StatGrids &grids, hipStream_t s) {
  const unsigned g = grid_for(n, kBlock, kMaxGrid);
  const bool ring = d.V && !d.qmode;
  const bool queues = d.V && d.qmode && d.L > 0;  // with L = 0 no line has a reuse iteration
  int scan = kScanNone;
  if (ring) {
    scan = (n + kScanChunk - 1) / kScanChunk <= kFusedScanMax ? kScanCounts : kScanOffsets;
    if (scan == kScanOffsets) hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kBlock), 0, s, sc.scan_part, cn);
  }
  if (queues) {
    hipLaunchKernelGGL(k_qcount, dim3(g), dim3(kBlock), 0, s, d, sc, t, cn);
    hipLaunchKernelGGL(k_qtop, dim3(1), dim3(kBlock), 0, s, d, sc, cn);
  }
  hipLaunchKernelGGL(k_resolve, dim3(g), dim3(kBlock), 0, s, d, sc, t, outcome, scan, cn);
  for (int st = kStVictimHits; st <= kStHost; ++st) grids.g[st] = g;
  for (int st = kStVhRing; st <= kStVhSame; ++st) grids.g[st] = g;
}

void launch_ring_enqueue(const DevState &d, const int64_t *ids, uint64_t n, uint64_t t, int64_t *inverse, Scratch &sc,
                         Counters *cn, StatGrids &grids, hipStream_t s) {
  const unsigned g = grid_for(n, kBlock, kMaxGrid);
  const bool ring = d.V && !d.qmode;
  const bool queues = d.V && d.qmode && d.L > 0;
  if (ring) {  // with the pass over the requests
    hipLaunchKernelGGL(k_enq_finalize, dim3(g), dim3(kBlock), 0, s, d, sc, ids, (uint32_t)n, inverse, cn);
    grids.g[kStEnqCopy] = g;
  } else {
    if (queues) {
      hipLaunchKernelGGL(k_qplace, dim3(g), dim3(kBlock), 0, s, d, sc, t, cn);
      grids.g[kStEnqCopy] = g;
    }
    hipLaunchKernelGGL(k_request_counts, dim3(g), dim3(kBlock), 0, s, d, sc, ids, (uint32_t)n, inverse, cn);
  }
  grids.g[kStReqHits] = g;
  grids.g[kStReqVictimHits] = g;
}

// --------------------------------------------------------- small gathers
// All the metadata of a gather of at most kTinyRequests requests, in one block:
// such a gather costs its launches, not its work (each of the eleven kernels
// runs for 2-8 us on it, and the host takes about 3 us to submit one).  The
// passes are those of the kernels above, one after the other; only the dedup
// is another: the requests are sorted in LDS, so that nothing depends on the
// number of nodes, as the scans of the byte map do.
__device__ __forceinline__ void tiny_sort(uint64_t *key, uint32_t n) {
  uint32_t P = 64;  // the next power of two
  while (P < n) P *= 2;
  for (uint32_t i = n + threadIdx.x; i < P; i += kBlock) key[i] = ~0ull;
  __syncthreads();
  for (uint32_t k = 2; k <= P; k *= 2)
    for (uint32_t j = k / 2; j > 0; j /= 2) {
      for (uint32_t p = threadIdx.x; p < P / 2; p += kBlock) {
        const uint32_t lo = 2 * p - (p & (j - 1)), hi = lo + j;  // j apart, j-bit clear in lo
        const uint64_t a = key[lo], b = key[hi];
        if ((a > b) == ((lo & k) == 0)) {
          key[lo] = b;
          key[hi] = a;
        }
      }
      __syncthreads();
    }
}

// The rest of a gather all of whose IDs are resident: hits change nothing, so
// there is nothing to group, walk, scan or resolve (a blocking lookup of 250
// resident rows 48 -> 42 us).
__device__ __forceinline__ void tiny_all_hits(const DevState &d, const Scratch &sc, const TinyArgs &a, uint32_t U) {
  for (uint32_t u = threadIdx.x; u < U; u += kBlock) {
    d.uidx[sc.uniq[u]] = u;
    d.batch[sc.uset[u]].count = 0;
    sc.hbm.src[u] = sc.slot[u];
    if (a.outcome) a.outcome[u] = 0;  // LSMGNN_HIT
  }
  __syncthreads();
  if (a.inverse)
    for (uint32_t i = threadIdx.x; i < a.n; i += kBlock) a.inverse[i] = (int64_t)d.uidx[a.ids[i]];
  if (threadIdx.x == 0) {
    sc.stat_part[kStSettled * kMaxGrid] = U;
    sc.stat_part[kStHbm * kMaxGrid] = U;
    sc.stat_part[kStReqHits * kMaxGrid] = a.n;
  }
}

template <int P>
__global__ __launch_bounds__(kBlock) void k_tiny(const DevState d, Scratch sc, TinyArgs a, Counters *cn) {
  __shared__ uint64_t key[kTinyRequests];
  const uint32_t n = a.n;
  // validate
  bool bad = false;
  for (uint32_t i = threadIdx.x; i < n; i += kBlock) {
    const int64_t x = a.ids[i];
    bad |= x < 0 || (uint64_t)x >= d.N;
    key[i] = (uint64_t)x;
  }
  for (uint32_t i = threadIdx.x; i < a.ann_n; i += kBlock) {
    const int64_t x = a.ann_ids[i];
    bad |= x < 0 || (uint64_t)x >= d.N;
  }
  if (__syncthreads_or(bad)) {
    if (threadIdx.x == 0) {
      *sc.gate = gate_with(1, 0);
      publish_dedup(a.dd, a.tag, 1, 0);
    }
    return;
  }
  // the first of each run of equal IDs gets the next unique index
  tiny_sort(key, n);
  uint32_t U = 0;
  for (uint32_t base = 0; base < n; base += kBlock) {
    const uint32_t i = base + threadIdx.x;
    const bool first = i < n && (i == 0 || key[i] != key[i - 1]);
    uint32_t rank[1], tot[1];
    block_ranks<1>({first}, rank, tot);
    const uint32_t u = U + rank[0];
    U += tot[0];
    if (first) {
      sc.uniq[u] = (uint32_t)key[i];
      a.unique_out[u] = (int64_t)key[i];
    }
  }
  if (threadIdx.x == 0) {
    cn->n_unique = U;
    *sc.gate = gate_with(0, U);
    publish_dedup(a.dd, a.tag, 0, U);
  }
  __syncthreads();
  StatGrids grids{};
  if (!__syncthreads_or(probe(d, sc, a.t, cn))) {
    tiny_all_hits(d, sc, a, U);
    grids.g[kStSettled] = grids.g[kStHbm] = grids.g[kStReqHits] = 1;
  } else {
    seg_alloc(d, sc, (uint32_t)a.t, cn);
    __syncthreads();
    place(d, sc, cn);
    __syncthreads();
    walk_sets<P>(d, sc, (uint32_t)a.t, cn);
    __syncthreads();
    resolve(d, sc, a.t, a.outcome, d.V ? kScanCounts : kScanNone, cn);
    __syncthreads();
    if (d.V) enqueue_entries(d, sc, cn);
    request_counts(d, sc, a.ids, n, a.inverse);
#pragma unroll
    for (int st = 0; st < kNumStat; ++st) grids.g[st] = 1;
    grids.g[kStEnqCopy] = d.V ? 1 : 0;
  }
  if (a.ann.ids) announce(a.ann);
  __syncthreads();
  finish(cn, a.hc, sc.stat_part, grids, d.tail, QueueFinish{});
}

void launch_tiny(const DevState &d, Scratch &sc, const TinyArgs &a, Counters *cn, hipStream_t s) {
  switch (d.policy) {
    case kPolicyStatic:
      hipLaunchKernelGGL(k_tiny<kPolicyStatic>, dim3(1), dim3(kBlock), 0, s, d, sc, a, cn);
      break;
    case kPolicyDynamic:
      hipLaunchKernelGGL(k_tiny<kPolicyDynamic>, dim3(1), dim3(kBlock), 0, s, d, sc, a, cn);
      break;
    case kPolicyRoundRobin:
      hipLaunchKernelGGL(k_tiny<kPolicyRoundRobin>, dim3(1), dim3(kBlock), 0, s, d, sc, a, cn);
      break;
    default:
      hipLaunchKernelGGL(k_tiny<kPolicyHybrid>, dim3(1), dim3(kBlock), 0, s, d, sc, a, cn);
  }
}

// -------------------------------------------------------------- row copies
// Work item w = (unique index e, 16-byte vector v): consecutive lanes take
// consecutive vectors of one row, so a wave moves whole rows with 128-bit
// accesses, and each lane keeps kUnroll vectors in flight before storing.
// The HBM-side modes read the per-unique descriptor and skip rows they do not
// own; the host fetch walks the dense host-fetch list instead.  Counts come
// from the gather's gate; a rejected gather moves nothing.
constexpr int kUnroll = 4;

// Copy of a row list: item w = (list entry i, 16-byte vector v).  Each block
// takes a tile of kListUnroll * kBlock consecutive items (whole rows, their
// 16-byte vectors on consecutive lanes), the tiles striding over the grid;
// loads and stores carry the non-temporal hint (every row moves once).
// Measured on the MI355X against grid-strided items without the hint:
// 5.7-6.0 against 4.9-5.2 TB/s for 1-2 KiB random rows.  The mode only names
// the instance (hit copy, staging, fills) so that profiles tell them apart.
constexpr int kListUnroll = 2;
//
// The hit copy's list (M = kHbmToOut) is dense by destination: entry i moves
// to output row i, from row sidx[i] unless that is kNoRow (the unique ID's
// row comes over the host link).  Writing the output rows in order measured
// 6.0 TB/s against 5.2-5.4 for the same rows listed in per-block runs of
// arbitrary order (600 K random 2 KiB rows from a 96 GiB region).
template <CopyMode M, bool kPow2>
__global__ __launch_bounds__(kBlock) void k_list_copy(const uint8_t *src, const uint32_t *sidx, uint8_t *dst,
                                                      const uint32_t *didx, const Gate *gate, const uint32_t *count,
                                                      uint64_t R, uint32_t nvec, uint32_t vshift) {
  constexpr bool kDense = M == CopyMode::kHbmToOut;
  if (gate->err) return;
  const uint64_t total = (uint64_t)*count * nvec;
  constexpr uint64_t tile = (uint64_t)kListUnroll * kBlock;
  for (uint64_t base = (uint64_t)blockIdx.x * tile; base < total; base += (uint64_t)gridDim.x * tile) {
    u32x4 v[kListUnroll];
    uint8_t *dp[kListUnroll];
#pragma unroll
    for (int k = 0; k < kListUnroll; ++k) {
      const uint64_t w = base + (uint64_t)k * kBlock + threadIdx.x;
      dp[k] = nullptr;
      if (w < total) {
        const uint32_t i = kPow2 ? (uint32_t)(w >> vshift) : (uint32_t)(w / nvec);
        const uint64_t byte = (w - (uint64_t)i * nvec) * 16u;
        const uint32_t si = sidx[i];
        if (!kDense || si != kNoRow) {
          v[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + (uint64_t)si * R + byte));
          dp[k] = dst + (uint64_t)(kDense ? i : didx[i]) * R + byte;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kListUnroll; ++k)
      if (dp[k]) __builtin_nontemporal_store(v[k], reinterpret_cast<u32x4 *>(dp[k]));
  }
}

// Host fetch: item w = (host-list entry i, 16-byte vector v).  The list entry
// is the same for all lanes of a row (broadcast loads), and the entries of the
// next pass are loaded while this pass's host reads are in flight, so the
// reads never wait behind a dependent HBM load.  With a pageable store the
// host has already copied entry i's row to bounce row i.
#ifndef LSM_HOST_UNROLL
#define LSM_HOST_UNROLL 4
#endif
//
// The list has two parts: its first n_early entries (misses known at batch
// start, `late` false) and the n_host entries after them (the resolve's,
// `late` true); each launch moves one part.
template <bool kPow2>
__global__ __launch_bounds__(kBlock) void k_host_fetch(const DevState d, Scratch sc, uint8_t *out, uint32_t nvec,
                                                       uint32_t vshift, int late) {
  constexpr int kU = LSM_HOST_UNROLL;
  const Gate g = *sc.gate;
  if (g.err) return;
  const uint64_t R = d.R;
  const uint32_t first = late ? g.n_early : 0u;
  const uint64_t total = (uint64_t)(late ? g.n_host : g.n_early) * nvec;
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  const uint32_t *list = sc.host_list + first;
  const uint64_t *src = sc.host_src + first;
  const u32x4 *bounce = sc.bounce ? reinterpret_cast<const u32x4 *>(sc.bounce) + (uint64_t)first * nvec : nullptr;
  auto entry = [&](uint64_t w, uint32_t &e, uint64_t &code) {
    if (w < total) {
      const uint32_t i = kPow2 ? (uint32_t)(w >> vshift) : (uint32_t)(w / nvec);
      e = list[i];
      code = src[i];
    }
  };
  uint32_t e[kU];
  uint64_t code[kU];
  uint64_t w0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
#pragma unroll
  for (int k = 0; k < kU; ++k) entry(w0 + k * stride, e[k], code[k]);
  for (; w0 < total; w0 += stride * kU) {
    u32x4 v[kU];
    uint8_t *dst[kU];
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const uint64_t w = w0 + k * stride;
      dst[k] = nullptr;
      if (w < total) {
        const uint64_t byte = (kPow2 ? (w & (nvec - 1)) : (w % nvec)) * 16u;
        // bounce row i holds entry i: vector w is the w-th of the buffer
        const u32x4 *sp =
            bounce ? bounce + w
                   : reinterpret_cast<const u32x4 *>(
                            ((code[k] & ~kSrcIndex) == kSrcRing ? d.ring_rows : d.store) + (code[k] & kSrcIndex) * R +
                            byte);
        v[k] = *sp;
        dst[k] = out + (uint64_t)e[k] * R + byte;
      }
    }
    const uint64_t w1 = w0 + stride * kU;
#pragma unroll
    for (int k = 0; k < kU; ++k) entry(w1 + k * stride, e[k], code[k]);
    // the output rows are written once and read next by other kernels: the
    // non-temporal hint keeps them from displacing what the kernels beside
    // this one hold in L2 (measured: never slower, up to 3.5 % faster on the
    // 100M-node workload)
#pragma unroll
    for (int k = 0; k < kU; ++k)
      if (dst[k]) __builtin_nontemporal_store(v[k], reinterpret_cast<u32x4 *>(dst[k]));
  }
}

// Grid caps.  Every outstanding host-link read queues in front of the memory
// requests of the kernels that run beside it (the next gather's metadata, the
// hit copy, the fills, the ring write), so the host fetch keeps only about
// 640 KB in flight (40 blocks x 256 lanes x 4 x 16 B): enough to cover the
// link's latency, not more.  A sweep of block counts and unroll depths on
// the full pipeline chose it.  The runtime picks another grid per gather
// (DevState::host_grid): fewer blocks when more traffic shares the host or
// the link, more when the fetch reads a pageable store's contiguous bounce
// rows.
#ifndef LSM_HOST_GRID
#define LSM_HOST_GRID 40
#endif
#ifndef LSM_HBM_GRID
// the HBM-side copies: 65536 blocks.  A resident stream's hit copies beside the
// next gather's metadata: 1142 us for four gathers, 1219 with 8192 blocks, 1280
// with 1024, 1250 with 262144
#define LSM_HBM_GRID 65536
#endif
// Staging and fills move the evicted and the missed rows, often few or none of
// the batch's, while their grid is sized for all of it: blocks that find
// nothing cost 20 us per launch at 65536 of them, under 5 us at 8192, and a
// long list moves as fast with either.
constexpr unsigned kListGrid = 8192;

template <CopyMode M>
static void launch_list(const uint8_t *src, const RowList &l, uint8_t *dst, const Gate *gate, const uint32_t *count,
                        uint64_t n, uint64_t R, hipStream_t s) {
  const uint32_t nvec = (uint32_t)(R / 16);
  const unsigned g = grid_for(n * nvec, (uint64_t)kBlock * kListUnroll,
                              M == CopyMode::kHbmToOut ? LSM_HBM_GRID : kListGrid);
  if ((nvec & (nvec - 1)) == 0)
    hipLaunchKernelGGL((k_list_copy<M, true>), dim3(g), dim3(kBlock), 0, s, src, l.src, dst, l.dst, gate, count, R,
                       nvec, (uint32_t)__builtin_ctz(nvec));
  else
    hipLaunchKernelGGL((k_list_copy<M, false>), dim3(g), dim3(kBlock), 0, s, src, l.src, dst, l.dst, gate, count, R,
                       nvec, 0u);
}

void launch_copy(CopyMode mode, const DevState &d, uint64_t n, const Scratch &sc, uint8_t *out, hipStream_t s) {
  const uint32_t nvec = (uint32_t)(d.R / 16);
  const bool pow2 = (nvec & (nvec - 1)) == 0;
  const uint32_t vshift = pow2 ? (uint32_t)__builtin_ctz(nvec) : 0u;
  if (mode == CopyMode::kHostLate || mode == CopyMode::kHostEarly) {
    const unsigned g = grid_for(n * nvec, (uint64_t)kBlock * kUnroll, d.host_grid ? d.host_grid : LSM_HOST_GRID);
    const int late = mode == CopyMode::kHostLate;
    if (pow2)
      hipLaunchKernelGGL((k_host_fetch<true>), dim3(g), dim3(kBlock), 0, s, d, sc, out, nvec, vshift, late);
    else
      hipLaunchKernelGGL((k_host_fetch<false>), dim3(g), dim3(kBlock), 0, s, d, sc, out, nvec, vshift, late);
    return;
  }
  switch (mode) {
    case CopyMode::kHbmToOut:
      launch_list<CopyMode::kHbmToOut>(d.rows, sc.hbm, out, sc.gate, &sc.gate->n_unique, n, d.R, s);
      break;
    case CopyMode::kCacheToStage:
      launch_list<CopyMode::kCacheToStage>(d.rows, sc.stage, sc.staging, sc.gate, &sc.gate->n_stage, n, d.R, s);
      break;
    default:
      launch_list<CopyMode::kOutToCache>(out, sc.fill, d.rows, sc.gate, &sc.gate->n_fill, n, d.R, s);
      break;
  }
}

// A gather on one stream: the host fetch, the hit copy and the staging in one
// launch, in tiles as the list copy takes them.  The first blocks, at most
// kMoveHostBlocks, take the host rows, one tile each where the gather fetches
// what it was expected to; one that fetches more keeps no more in flight over
// the link, in front of the HBM rows beside it.  With a block per host tile
// whatever the list, and the streams chosen by the last gather alone, a lookup
// and two gathers of 60 K missing 1 KiB rows took 2203 us, now 2116.
constexpr unsigned kMoveHostBlocks = kSerialBytes / (16 * kListUnroll * kBlock);
template <bool kPow2>
__global__ __launch_bounds__(kBlock) void k_move_rows(const DevState d, Scratch sc, uint8_t *out, uint32_t nvec,
                                                      uint32_t vshift) {
  const Gate g = *sc.gate;
  if (g.err) return;
  const uint64_t R = d.R;
  constexpr uint64_t tile = (uint64_t)kListUnroll * kBlock;
  // tiles first, first + step, ... of `total` vectors; rows(i, src, dst) gives
  // entry i's rows, if it has any
  auto move = [&](uint64_t total, uint64_t first, uint64_t step, auto rows) {
    for (uint64_t base = first * tile; base < total; base += step * tile) {
      u32x4 v[kListUnroll];
      uint8_t *dp[kListUnroll];
#pragma unroll
      for (int k = 0; k < kListUnroll; ++k) {
        const uint64_t w = base + (uint64_t)k * kBlock + threadIdx.x;
        dp[k] = nullptr;
        if (w < total) {
          const uint64_t i = kPow2 ? w >> vshift : w / nvec;
          const uint64_t byte = (w - i * nvec) * 16u;
          const uint8_t *sp = nullptr;
          rows(i, sp, dp[k]);
          if (dp[k]) {
            v[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(sp + byte));
            dp[k] += byte;
          }
        }
      }
#pragma unroll
      for (int k = 0; k < kListUnroll; ++k)
        if (dp[k]) __builtin_nontemporal_store(v[k], reinterpret_cast<u32x4 *>(dp[k]));
    }
  };
  const uint64_t n_host = ((uint64_t)g.n_early + g.n_host) * nvec;
  const uint64_t tiles = (n_host + tile - 1) / tile;
  const uint64_t hb = tiles < kMoveHostBlocks ? tiles : kMoveHostBlocks;  // blocks with host rows
  if (blockIdx.x < hb)
    move(n_host, blockIdx.x, hb, [&](uint64_t i, const uint8_t *&sp, uint8_t *&dp) {
      const uint64_t code = sc.host_src[i];
      sp = ((code & ~kSrcIndex) == kSrcRing ? d.ring_rows : d.store) + (code & kSrcIndex) * R;
      dp = out + (uint64_t)sc.host_list[i] * R;
    });
  const uint64_t n_out = g.n_unique, n_hbm = n_out + (d.V ? g.n_stage : 0u);
  const uint64_t first = blockIdx.x >= hb ? blockIdx.x - hb : blockIdx.x + gridDim.x - hb;
  move(n_hbm * nvec, first, gridDim.x, [&](uint64_t i, const uint8_t *&sp, uint8_t *&dp) {
    if (i < n_out) {
      const uint32_t row = sc.hbm.src[i];
      if (row != kNoRow) {
        sp = d.rows + (uint64_t)row * R;
        dp = out + i * R;
      }
    } else {
      const uint64_t j = i - n_out;
      sp = d.rows + (uint64_t)sc.stage.src[j] * R;
      dp = sc.staging + (uint64_t)sc.stage.dst[j] * R;
    }
  });
}

void launch_move_rows(const DevState &d, uint64_t n, const Scratch &sc, uint8_t *out, hipStream_t s) {
  const uint32_t nvec = (uint32_t)(d.R / 16);
  // a block per tile of the batch's rows beside those of the host rows
  const unsigned g = grid_for(n * nvec, (uint64_t)kBlock * kListUnroll, LSM_HBM_GRID) + kMoveHostBlocks;
  if ((nvec & (nvec - 1)) == 0)
    hipLaunchKernelGGL(k_move_rows<true>, dim3(g), dim3(kBlock), 0, s, d, sc, out, nvec,
                       (uint32_t)__builtin_ctz(nvec));
  else
    hipLaunchKernelGGL(k_move_rows<false>, dim3(g), dim3(kBlock), 0, s, d, sc, out, nvec, 0u);
}

// Queue mode: the queue of the next gather into its prefetch buffer.  Rows of
// entries placed by earlier gathers cross the host link (a small grid, like
// the host fetch); those placed by the gather just issued are still in its
// staging rows in HBM.
__global__ __launch_bounds__(kBlock) void k_prefetch(const DevState d, const Gate *gate, const uint8_t *staging,
                                                     uint32_t slot, uint32_t par, uint32_t nvec) {
  const uint32_t cnt = gate->q_count, before = gate->q_before, off = gate->q_stage_off;
  const uint64_t R = d.R;
  const uint64_t total = (uint64_t)cnt * nvec;
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  uint8_t *pf = d.rows + (d.S * kWays + (uint64_t)par * d.C) * R;
  const uint8_t *q = d.ring_rows + (uint64_t)slot * d.C * R;
  for (uint64_t w0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x; w0 < total; w0 += stride * kUnroll) {
    u32x4 v[kUnroll];
    uint8_t *dp[kUnroll];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
      const uint64_t w = w0 + k * stride;
      dp[k] = nullptr;
      if (w < total) {
        const uint64_t i = w / nvec;
        const uint64_t byte = (w - i * nvec) * 16u;
        const uint8_t *src = i < before ? q + i * R + byte : staging + (off + (i - before)) * R + byte;
        v[k] = *reinterpret_cast<const u32x4 *>(src);
        dp[k] = pf + i * R + byte;
      }
    }
#pragma unroll
    for (int k = 0; k < kUnroll; ++k)
      if (dp[k]) *reinterpret_cast<u32x4 *>(dp[k]) = v[k];
  }
}

void launch_prefetch(const DevState &d, const Gate *gate, const uint8_t *staging, uint32_t slot, uint32_t par,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_prefetch, dim3(LSM_HOST_GRID), dim3(kBlock), 0, s, d, gate, staging, slot, par,
                     (uint32_t)(d.R / 16));
}

// ------------------------------------------------------------ calibration
// Plain contiguous copy with the same 128-bit access pattern and unrolling as
// the row copies; used to measure the host-link and HBM ceilings and to scale
// hardware byte counters against a copy of known size.
__global__ __launch_bounds__(kBlock) void k_copy_plain(const u32x4 *src, u32x4 *dst, uint64_t nvec) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t w0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x; w0 < nvec; w0 += stride * kUnroll) {
    u32x4 v[kUnroll];
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
      const uint64_t w = w0 + k * stride;
      if (w < nvec) v[k] = src[w];
    }
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) {
      const uint64_t w = w0 + k * stride;
      if (w < nvec) dst[w] = v[k];
    }
  }
}

__global__ void k_publish_count(const Gate *gate, const uint32_t *count, uint32_t *dst) {
  if (threadIdx.x == 0) *dst = gate->err ? 0u : *count;
}

void launch_publish_count(const Gate *gate, const uint32_t *count, uint32_t *dst, hipStream_t s) {
  hipLaunchKernelGGL(k_publish_count, dim3(1), dim3(64), 0, s, gate, count, dst);
}

// Device-to-device: tiles of 4 * kBlock vectors per block with the
// non-temporal hint, the copy pattern of the row lists.
__global__ __launch_bounds__(kBlock) void k_copy_tiles(const u32x4 *src, u32x4 *dst, uint64_t nvec) {
  constexpr uint64_t tile = 4 * (uint64_t)kBlock;
  for (uint64_t base = (uint64_t)blockIdx.x * tile; base < nvec; base += (uint64_t)gridDim.x * tile) {
    u32x4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t w = base + (uint64_t)k * kBlock + threadIdx.x;
      if (w < nvec) v[k] = __builtin_nontemporal_load(src + w);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t w = base + (uint64_t)k * kBlock + threadIdx.x;
      if (w < nvec) __builtin_nontemporal_store(v[k], dst + w);
    }
  }
}

void launch_copy_plain(const void *src, void *dst, uint64_t bytes, bool device_to_device, hipStream_t s) {
  const uint64_t nvec = bytes / 16;
  if (device_to_device)
    hipLaunchKernelGGL(k_copy_tiles, dim3(grid_for(nvec, 4 * (uint64_t)kBlock, 262144)), dim3(kBlock), 0, s,
                       static_cast<const u32x4 *>(src), static_cast<u32x4 *>(dst), nvec);
  else
    hipLaunchKernelGGL(k_copy_plain, dim3(grid_for(nvec, (uint64_t)kBlock * kUnroll, 4096)), dim3(kBlock), 0, s,
                       static_cast<const u32x4 *>(src), static_cast<u32x4 *>(dst), nvec);
}

// ------------------------------------------------------------------ window
// Announce: validate the IDs and, when the list is recorded, set the
// minibatch's bit for every ID (see window_bits).  Only that bit of a node's
// window changes in this kernel (duplicates write the same value), so a plain
// read-modify-write is exact.
__global__ void k_window_set(const int64_t *ids, uint32_t n, uint64_t N, uint32_t now, uint32_t bit, uint64_t *win,
                             int record, uint32_t *err) {
  bool bad = false;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const int64_t x = ids[i];
    if (x < 0 || (uint64_t)x >= N)
      bad = true;
    else if (record)
      window_set(win, (uint64_t)x, now, bit);
  }
  if (__ballot(bad) && __lane_id() == 0)  // every writer stores the same value
    __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// After a rejected announcement (the host launches it only then): clear the
// bit again (it was clear before: a minibatch is announced once).
__global__ void k_window_rollback(const int64_t *ids, uint32_t n, uint64_t N, uint32_t now, uint32_t bit,
                                  uint64_t *win) {
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const int64_t x = ids[i];
    if (x >= 0 && (uint64_t)x < N) win[x] = (uint64_t)now << 32 | (window_bits(win[x], now) & ~(1u << bit));
  }
}

void launch_window_set(const int64_t *ids, uint64_t n, uint64_t N, uint32_t now, uint32_t bit, uint64_t *win,
                       bool record, uint32_t *err, hipStream_t s) {
  const unsigned g = grid_for(n, kBlock, kMaxGrid);
  hipLaunchKernelGGL(k_window_set, dim3(g), dim3(kBlock), 0, s, ids, (uint32_t)n, N, now, bit, win, record ? 1 : 0,
                     err);
}

void launch_window_rollback(const int64_t *ids, uint64_t n, uint64_t N, uint32_t now, uint32_t bit, uint64_t *win,
                            hipStream_t s) {
  const unsigned g = grid_for(n, kBlock, kMaxGrid);
  hipLaunchKernelGGL(k_window_rollback, dim3(g), dim3(kBlock), 0, s, ids, (uint32_t)n, N, now, bit, win);
}

// ------------------------------------------------------ request order
// Per-position output: row i of `out` <- row inv[i] of `rows` (the unique-row
// output of a gather), for the n requests in their original order.  Item w =
// (request i, 16-byte vector v), in tiles as the list copies take them; the
// inverse entry is a broadcast load.  Bound by HBM bandwidth.  The output is
// written once, with the non-temporal hint, so that it does not take the place
// of rows in the last-level cache: rows that are still there (those of the
// gather before, if nothing else ran) or that several requests name.  203 K
// requests of 190 K distinct 4 KiB rows: 316 -> 296 us with the rows just
// written, 320 -> 280 with the same call repeated, 348 -> 346 after 1 GiB of
// other writes; 900 K requests of 235 K 2 KiB rows 626 -> 562, 627 -> 546 and
// 662 -> 598.  With the hint on the loads too, repeated rows are 10-40 % slower.
template <bool kPow2>
__global__ __launch_bounds__(kBlock) void k_expand(const uint8_t *rows, const int64_t *inv, uint64_t n, uint64_t R,
                                                   uint32_t nvec, uint32_t vshift, uint8_t *out) {
  const uint64_t total = n * nvec;
  constexpr uint64_t tile = (uint64_t)kListUnroll * kBlock;
  for (uint64_t base = (uint64_t)blockIdx.x * tile; base < total; base += (uint64_t)gridDim.x * tile) {
    u32x4 v[kListUnroll];
#pragma unroll
    for (int k = 0; k < kListUnroll; ++k) {
      const uint64_t w = base + (uint64_t)k * kBlock + threadIdx.x;
      if (w < total) {
        const uint64_t i = kPow2 ? (w >> vshift) : (w / nvec);
        const uint64_t byte = (w - i * nvec) * 16u;
        v[k] = *(reinterpret_cast<const u32x4 *>(rows + (uint64_t)inv[i] * R + byte));
      }
    }
#pragma unroll
    for (int k = 0; k < kListUnroll; ++k) {
      const uint64_t w = base + (uint64_t)k * kBlock + threadIdx.x;
      if (w < total) __builtin_nontemporal_store(v[k], reinterpret_cast<u32x4 *>(out) + w);
    }
  }
}

void launch_expand(const uint8_t *rows, const int64_t *inv, uint64_t n, uint64_t R, uint8_t *out, hipStream_t s) {
  const uint32_t nvec = (uint32_t)(R / 16);
  const unsigned g = grid_for(n * nvec, (uint64_t)kBlock * kListUnroll, 262144);  // nothing runs beside it
  if ((nvec & (nvec - 1)) == 0)
    hipLaunchKernelGGL(k_expand<true>, dim3(g), dim3(kBlock), 0, s, rows, inv, n, R, nvec,
                       (uint32_t)__builtin_ctz(nvec), out);
  else
    hipLaunchKernelGGL(k_expand<false>, dim3(g), dim3(kBlock), 0, s, rows, inv, n, R, nvec, 0u, out);
}

}  // namespace lsm

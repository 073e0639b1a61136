// Neighbour sampling on the GPU: the raw request lists of GraphSAGE
// minibatches (uniform sampling of a fixed number of neighbours per hop,
// Sec. 2.1), produced on the device, as the GPU-side sampler of the system
// overview (Sec. 4) does, so that the cache's gather and announcement take
// them without a host round trip.
//
// One minibatch, from its seed nodes and the fanouts f_0 .. f_{H-1}:
//   frontier_0 = the seeds, sorted, duplicates removed;
//   hop h: each frontier node v, in ascending order, draws k = min(f_h, deg v)
//     distinct positions of its adjacency list with Floyd's algorithm (Bentley
//     and Floyd, CACM 1987) and lists them ascending; the hop's samples are
//     adj[off[v] + position] in that order; frontier_{h+1} = the hop's samples,
//     sorted, duplicates removed;
//   request list = seeds (as given) ++ samples of hop 0 ++ hop 1 ++ ...
// Random draws come from counter-based SplitMix64 streams (Steele, Lea and
// Flood, OOPSLA 2014): output k of the stream keyed by K is mix(K + (k+1) G).
// Minibatch b of a sampler seeded with s uses the key
//   key_b = derive(derive(s, 3), b),  derive(p, l) = output l of the stream
//   keyed by mix(p ^ 0x5851f42d4c957f2d);
// hop h of it derive(key_b, h), node v in that hop derive(key_hop, v), and
// the j-th draw of Floyd's algorithm for v is output j of that node's stream,
// reduced to [0, m) as ((r >> 32) * m) >> 32.
//
// Per hop, on the caller's stream:
//   counts   per chunk of the byte map of marked nodes: how many there are and
//            how many samples they draw
//   frontier the marked nodes in ascending order become the hop's frontier, each
//            with its first sample's place within the chunk's; the map is
//            cleared.  Each block adds up the chunks before its own; the last
//            one has the hop's totals (with many chunks one block scans them
//            first)
//   draw     8 to 64 lanes per frontier node, by the fanout: lane j makes
//            Floyd's j-th draw, the k steps are resolved in order with one
//            ballot each, and each lane's rank among the k positions places
//            its sample in the list; the next frontier's byte-map marks are
//            plain byte stores
// Every count stays on the device; the frontier of the last hop gives the list's
// length and the status, written to the caller's pinned memory at once.  The
// byte map holds one byte per node and is all zero between calls.
//
// A minibatch is bound by its chain of dependent launches (2-8 us each), so
// there are few: ten for three hops.  With the offsets in two kernels of their
// own, a separate scan of the chunks, a wave per node whatever the fanout and
// the result copied afterwards there were twenty-two.  1024 seeds of a 1 M-node
// graph at (15, 10, 5), waited for: 72 us against 102; 4096 seeds of a 10 M-node
// graph at (10, 5, 5), queued: 60 against 83.
//
// Typed graphs: the list split by node type (per tile of requests a count per
// type, then each tile adds up the tiles before it and ranks its requests by
// ballots), each ID replaced by its index within its type.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <mutex>

#include "lsmgnn.h"

namespace lsm_smp {

constexpr int kBlock = 256;
// Byte-map words per thread, and bytes (nodes) per block, a chunk: the small
// one for at most kSmallChunkNodes nodes, else the large one, so that the
// chunks are few.  A thread looks up its marked nodes' degrees one by one, and
// the nodes of a power-law graph's hubs lie together: with 64 bytes per thread
// the two passes over 10 M nodes took 11 and 13 us, with 16 they take 5 and 8.
constexpr int kWordsSmall = 4, kWordsLarge = 16;
constexpr uint64_t kSmallChunkNodes = 1ull << 24;
// at most this many small chunks, and large ones, are added up by each block
constexpr uint32_t kFusedSmall = 4096, kFusedLarge = 2048;
constexpr unsigned kMaxGrid = 4096;
constexpr uint32_t kMaxFanout = 64;  // one wave's lanes
constexpr uint32_t kMaxHops = 8;
constexpr uint64_t kGamma = 0x9e3779b97f4a7c15ull;
constexpr uint64_t kLabelSample = 3;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__host__ __device__ __forceinline__ uint64_t mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}
__host__ __device__ __forceinline__ uint64_t stream_at(uint64_t key, uint64_t k) { return mix(key + (k + 1) * kGamma); }
__host__ __device__ __forceinline__ uint64_t derive(uint64_t parent, uint64_t label) {
  return stream_at(mix(parent ^ 0x5851f42d4c957f2dull), label);
}

// Device-side state of one call.
struct Ctl {
  uint32_t err;       // a seed outside [0, N)
  uint32_t frontier;  // current frontier size
  uint64_t len;       // request-list length so far
  uint64_t hop_base;  // list position of the current hop's first sample
};

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

// 64-bit variant for the scan over tile sums
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

__global__ __launch_bounds__(kBlock) void k_validate(const int64_t *off, const uint32_t *adj, uint64_t N, uint64_t E,
                                                     uint32_t *err) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  bool bad = false;
  for (uint64_t u = (uint64_t)blockIdx.x * kBlock + threadIdx.x; u < N; u += stride) {
    const int64_t deg = off[u + 1] - off[u];
    bad |= deg < 0 || deg > (int64_t)0xffffffffll;
  }
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < E; e += stride) bad |= adj[e] >= N;
  if (bad) *err = 1u;
}

// The seeds open the list and mark the first frontier.
__global__ __launch_bounds__(kBlock) void k_seeds(const int64_t *seeds, uint64_t n, uint64_t N, int64_t *out,
                                                  uint64_t cap, uint8_t *present, Ctl *ctl) {
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock) {
    const int64_t x = seeds[i];
    if (x < 0 || (uint64_t)x >= N) {
      bad = true;
      continue;
    }
    if (i < cap) out[i] = x;
    present[x] = 1;
  }
  if (__ballot(bad) && __lane_id() == 0) atomicOr(&ctl->err, 1u);
}

template <int kW>
__device__ __forceinline__ uint64_t chunk_node(uint32_t chunk) {  // first node of this thread's words
  return ((uint64_t)chunk * kBlock + threadIdx.x) * 4 * kW;
}

template <int kW>
__device__ __forceinline__ void load_map(const uint8_t *present, uint64_t v0, uint32_t (&w)[kW]) {
  const u32x4 *p = reinterpret_cast<const u32x4 *>(present + v0);
#pragma unroll
  for (int k = 0; k < kW / 4; ++k) {
    const u32x4 a = p[k];
    w[4 * k] = a.x;
    w[4 * k + 1] = a.y;
    w[4 * k + 2] = a.z;
    w[4 * k + 3] = a.w;
  }
}

__device__ __forceinline__ uint32_t draws_of(const int64_t *off, uint64_t v, uint32_t fanout) {
  const uint64_t deg = (uint64_t)(off[v + 1] - off[v]);
  return (uint32_t)(fanout < deg ? fanout : deg);
}

// f(node) for each marked node of the thread's words, ascending (marked bytes
// hold exactly 1: bit 8j of a word is set for its byte j)
template <int kW, typename F>
__device__ __forceinline__ void for_marked(const uint32_t (&w)[kW], uint64_t v0, const F &f) {
#pragma unroll
  for (int k = 0; k < kW; ++k)
    for (uint32_t word = w[k]; word; word &= word - 1u) f(v0 + 4 * k + (__builtin_ctz(word) >> 3));
}

// Marked nodes and samples drawn, as one word: a large chunk has at most 2^14
// nodes and draws at most 2^20 samples, so the chunks that are added up draw
// 2^31 at most.
__device__ __forceinline__ uint64_t pack(uint32_t nodes, uint32_t draws) { return (uint64_t)nodes << 32 | draws; }

template <int kW>
__global__ __launch_bounds__(kBlock) void k_counts(const uint8_t *present, const int64_t *off, uint32_t fanout,
                                                   uint64_t *chunk_sum) {
  const uint64_t v0 = chunk_node<kW>(blockIdx.x);
  uint32_t w[kW];
  load_map<kW>(present, v0, w);
  uint32_t c = 0, d = 0;
  for_marked<kW>(w, v0, [&](uint64_t v) {
    ++c;
    d += draws_of(off, v, fanout);
  });
  uint64_t tot;
  (void)block_exclusive_scan64(pack(c, d), tot);
  if (threadIdx.x == 0) chunk_sum[blockIdx.x] = tot;
}

// The hop's totals: its frontier and its samples' places in the list; on the
// last hop the call's result (list length, status): LSMGNN_OK, E_RANGE for a bad
// seed, or E_INVAL for a list longer than the output.
struct Hop {
  uint64_t n_seeds;  // list length before the hop, if it is the first
  uint64_t cap;
  uint64_t *res;     // the last hop's, else NULL
  int first;
};
__device__ __forceinline__ void publish_hop(const Hop &h, uint32_t nodes, uint64_t draws, Ctl *ctl) {
  const uint64_t len = h.first ? h.n_seeds : ctl->len;
  ctl->frontier = nodes;
  ctl->hop_base = len;
  ctl->len = len + draws;
  if (h.res) {
    const uint64_t all = len + draws;
    const uint64_t st = ctl->err ? (uint64_t)LSMGNN_E_RANGE : all > h.cap ? (uint64_t)LSMGNN_E_INVAL : (uint64_t)LSMGNN_OK;
    __hip_atomic_store(h.res, all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(h.res + 1, st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    ctl->err = 0;  // for the next call
  }
}

// One block, more than kFusedLarge chunks: each chunk's first frontier entry
// and first sample.
__global__ __launch_bounds__(kBlock) void k_chunk_scan(const uint64_t *chunk_sum, uint32_t nchunks,
                                                       uint32_t *chunk_first, uint64_t *chunk_base, Hop hop,
                                                       Ctl *ctl) {
  uint32_t nodes = 0;
  uint64_t draws = 0;
  for (uint32_t base = 0; base < nchunks; base += kBlock) {
    const uint32_t i = base + threadIdx.x;
    const uint64_t v = i < nchunks ? chunk_sum[i] : 0ull;
    uint64_t tot;
    const uint64_t ex = block_exclusive_scan64(v, tot);  // 256 chunks draw at most 2^28 samples
    if (i < nchunks) {
      chunk_first[i] = nodes + (uint32_t)(ex >> 32);
      chunk_base[i] = draws + (uint32_t)ex;
    }
    nodes += (uint32_t)(tot >> 32);
    draws += (uint32_t)tot;
  }
  if (threadIdx.x == 0) publish_hop(hop, nodes, draws, ctl);
}

// The marked nodes, ascending, become the frontier; node_off: a node's first
// sample among its chunk's, chunk_base: the chunk's among the hop's.
template <int kW, bool kFused>
__global__ __launch_bounds__(kBlock) void k_frontier(uint8_t *present, const int64_t *off, uint32_t fanout,
                                                     const uint64_t *chunk_sum, const uint32_t *chunk_first,
                                                     uint64_t *chunk_base, uint32_t *frontier, uint32_t *node_off,
                                                     Hop hop, Ctl *ctl) {
  const uint64_t v0 = chunk_node<kW>(blockIdx.x);
  uint32_t w[kW];
  load_map<kW>(present, v0, w);
  uint64_t before = 0;  // the chunks before this one
  if constexpr (kFused) {
    uint64_t sum = 0;
    for (uint32_t j = threadIdx.x; j < blockIdx.x; j += kBlock) sum += chunk_sum[j];
    (void)block_exclusive_scan64(sum, before);
  }
  uint32_t c = 0, d = 0;
  for_marked<kW>(w, v0, [&](uint64_t v) {
    ++c;
    d += draws_of(off, v, fanout);
  });
  uint64_t tot;
  const uint64_t ex = block_exclusive_scan64(pack(c, d), tot);
  uint32_t pos = (uint32_t)(ex >> 32), place = (uint32_t)ex;
  if constexpr (kFused) {
    pos += (uint32_t)(before >> 32);
    if (threadIdx.x == 0) {
      chunk_base[blockIdx.x] = (uint32_t)before;
      if (blockIdx.x == gridDim.x - 1) {
        const uint64_t all = before + tot;
        publish_hop(hop, (uint32_t)(all >> 32), (uint32_t)all, ctl);
      }
    }
  } else {
    pos += chunk_first[blockIdx.x];
  }
#pragma unroll
  for (int k = 0; k < kW; ++k)
    if (w[k]) reinterpret_cast<uint32_t *>(present + v0)[k] = 0u;
  for_marked<kW>(w, v0, [&](uint64_t v) {
    frontier[pos] = (uint32_t)v;
    node_off[pos] = place;
    ++pos;
    place += draws_of(off, v, fanout);
  });
}

// G lanes per frontier node (G >= fanout): lane j makes Floyd's j-th draw; the
// k steps are then resolved in order with one ballot each (a draw already
// taken yields the step's own bound instead), and each lane's rank among the k
// positions gives its place in the ascending list.
template <int G>
__global__ __launch_bounds__(kBlock) void k_draw(const uint32_t *frontier, const int64_t *off, const uint32_t *adj,
                                                 uint32_t fanout, uint64_t key_hop, const uint64_t *chunk_base,
                                                 uint32_t chunk_shift, const uint32_t *node_off, int64_t *out,
                                                 uint64_t cap, uint8_t *present, int mark, const Ctl *ctl) {
  const uint32_t f = ctl->frontier;
  const uint64_t hop_base = ctl->hop_base;
  const uint32_t lane = threadIdx.x & (G - 1);
  const uint64_t mine = (G == 64 ? ~0ull : (1ull << (G & 63)) - 1ull) << (threadIdx.x & 63u & ~(uint32_t)(G - 1));
  const uint32_t groups = gridDim.x * (kBlock / G);
  for (uint32_t i = blockIdx.x * (kBlock / G) + threadIdx.x / G; i < f; i += groups) {
    const uint32_t v = frontier[i];
    const int64_t o = off[v];
    const uint64_t deg = (uint64_t)(off[v + 1ull] - o);
    const uint32_t k = (uint32_t)(fanout < deg ? fanout : deg);
    if (k == 0) continue;
    uint32_t pos = lane, rank = lane;  // k == deg: every position, in order
    if (k < deg) {
      const uint64_t jj = deg - k + (uint64_t)lane;  // this lane's step bound
      uint32_t r = 0;
      if (lane < k) r = (uint32_t)(((stream_at(derive(key_hop, v), (uint64_t)lane) >> 32) * (jj + 1)) >> 32);
      for (uint32_t q = 0; q < k; ++q) {
        const uint32_t rq = __shfl(r, (int)q, G);
        const bool taken = (__ballot(lane < q && pos == rq) & mine) != 0ull;
        if (lane == q) pos = taken ? (uint32_t)jj : r;
      }
      rank = 0;  // the positions are distinct
      for (uint32_t q = 0; q < k; ++q) rank += __shfl(pos, (int)q, G) < pos ? 1u : 0u;
    }
    if (lane < k) {
      const uint64_t p = hop_base + chunk_base[v >> chunk_shift] + node_off[i] + rank;
      const uint32_t u = adj[o + pos];
      if (p < cap) out[p] = (int64_t)u;
      if (mark) present[u] = 1;
    }
  }
}

// ------------------------------------------------------------ typed graphs
// A request list of global IDs split by node type, in request order, each ID
// replaced by its index within its type.  Tiles of kSplitTile requests, four
// per thread: per-tile counts per type, then each tile's lists start where the
// tiles before it end (added up by the tile's own block, or with many tiles by
// one block's scan first), and each request's rank among its tile's requests
// of its type comes from one ballot per type, wave and row of 64 requests.
// result[t] = length of type t's list; result[T] = status: LSMGNN_E_RANGE for an
// invalid ID or type, LSMGNN_E_INVAL when a list is longer than the outputs.
//
// Bound by the random lines of the two tables: a request's type is looked up by
// both kernels, its index by the second (389 K requests over 20 M nodes: 9 and
// 19 us, at 128 bytes a lookup 5.4 TB/s).  With tiles of 256, one block scanning
// all of them type by type (14 us) and the result words initialised, finished
// and copied by launches of their own it took 44 us, now 28.
constexpr uint32_t kMaxTypes = 16;
constexpr uint32_t kSplitItems = 4, kSplitTile = kBlock * kSplitItems;
constexpr uint32_t kSplitFusedMax = 1024;  // at most this many tiles are added up by each block
constexpr uint32_t kSplitCounts = 144;     // byte offset of the counts in the work memory
static_assert((kMaxTypes + 1) * 8 <= kSplitCounts && kSplitCounts + (kMaxTypes + 1) * 4 <= 256 + kMaxTypes * 4,
              "the result words and one tile's counts fit the smallest work memory");

struct TypeOuts {
  int64_t *p[kMaxTypes];
};

// Counts of tile b at cnt[b * (T + 1)]: per type, then the invalid requests.
__global__ __launch_bounds__(kBlock) void k_type_count(const int64_t *ids, uint64_t n, uint64_t N,
                                                       const uint8_t *node_type, uint32_t T, uint32_t *cnt) {
  __shared__ uint32_t h[kMaxTypes + 1];
  const uint64_t ntiles = (n + kSplitTile - 1) / kSplitTile;
  for (uint64_t b = blockIdx.x; b < ntiles; b += gridDim.x) {
    if (threadIdx.x <= T) h[threadIdx.x] = 0;
    __syncthreads();
    uint32_t t[kSplitItems];
#pragma unroll
    for (uint32_t q = 0; q < kSplitItems; ++q) {
      const uint64_t i = b * kSplitTile + q * kBlock + threadIdx.x;
      t[q] = kMaxTypes + 1;  // no request
      if (i < n) {
        const int64_t x = ids[i];
        t[q] = x < 0 || (uint64_t)x >= N ? T : node_type[x];
        t[q] = t[q] < T ? t[q] : T;
      }
    }
    // one LDS add per type and wave
    for (uint32_t k = 0; k <= T; ++k) {
      uint32_t c = 0;
#pragma unroll
      for (uint32_t q = 0; q < kSplitItems; ++q) c += (uint32_t)__popcll(__ballot(t[q] == k));
      if ((threadIdx.x & 63) == 0 && c) atomicAdd(&h[k], c);
    }
    __syncthreads();
    if (threadIdx.x <= T) cnt[b * (T + 1) + threadIdx.x] = h[threadIdx.x];
    __syncthreads();
  }
}

// The result words from the lists' lengths (threads 0..T - 1 hold one each,
// thread T the invalid requests).
__device__ __forceinline__ void publish_split(uint32_t T, uint64_t len, uint64_t cap, uint64_t *res) {
  const uint64_t over = __ballot(threadIdx.x < T && len > cap);  // T < 64: one wave
  if (threadIdx.x < T) __hip_atomic_store(res + threadIdx.x, len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (threadIdx.x == T) {
    const uint64_t st = len ? (uint64_t)LSMGNN_E_RANGE : over ? (uint64_t)LSMGNN_E_INVAL : (uint64_t)LSMGNN_OK;
    __hip_atomic_store(res + T, st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// One block, more than kSplitFusedMax tiles: the exclusive scan of the tiles'
// counts (in place) per type, and the result.
__global__ __launch_bounds__(kBlock) void k_type_scan(uint32_t *cnt, uint64_t ntiles, uint32_t T, uint64_t cap,
                                                      uint64_t *res) {
  __shared__ uint64_t len[kMaxTypes + 1];
  for (uint32_t t = 0; t <= T; ++t) {
    uint64_t carry = 0;
    for (uint64_t base = 0; base < ntiles; base += kBlock) {
      const uint64_t i = base + threadIdx.x;
      const uint32_t v = i < ntiles ? cnt[i * (T + 1) + t] : 0u;
      uint32_t tot;
      const uint32_t ex = block_exclusive_scan(v, tot);
      if (i < ntiles) cnt[i * (T + 1) + t] = (uint32_t)carry + ex;
      carry += tot;
    }
    if (threadIdx.x == 0) len[t] = carry;
  }
  __syncthreads();
  if (threadIdx.x < 64) publish_split(T, threadIdx.x <= T ? len[threadIdx.x] : 0, cap, res);
}

template <bool kFused>
__global__ __launch_bounds__(kBlock) void k_type_scatter(const int64_t *ids, uint64_t n, uint64_t N,
                                                         const uint8_t *node_type, const uint32_t *local, uint32_t T,
                                                         const uint32_t *cnt, TypeOuts outs, uint64_t cap,
                                                         uint64_t *res) {
  constexpr uint32_t kRows = kSplitItems * (kBlock / 64);  // rows of 64 requests
  __shared__ uint32_t rows[kRows][kMaxTypes];
  __shared__ uint32_t start[kMaxTypes + 1], all[kMaxTypes + 1];  // the tiles' before this one, and all of them
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;  // lanes below this one
  const uint64_t ntiles = (n + kSplitTile - 1) / kSplitTile;
  for (uint64_t b = blockIdx.x; b < ntiles; b += gridDim.x) {
    uint32_t t[kSplitItems], loc[kSplitItems], rank[kSplitItems];
#pragma unroll
    for (uint32_t q = 0; q < kSplitItems; ++q) {
      const uint64_t i = b * kSplitTile + q * kBlock + threadIdx.x;
      t[q] = kMaxTypes;  // no request, or an invalid one
      loc[q] = 0;
      if (i < n) {
        const int64_t x = ids[i];
        if (x >= 0 && (uint64_t)x < N) {
          const uint32_t y = node_type[x];
          loc[q] = local[x];
          t[q] = y < T ? y : kMaxTypes;
        }
      }
    }
    if constexpr (kFused) {
      // thread first * W + word adds up one word of every (kBlock / W)-th tile,
      // eight of them in flight beside the lookups above
      if (threadIdx.x <= T) start[threadIdx.x] = all[threadIdx.x] = 0;
      const uint32_t W = T + 1, per = kBlock / W, word = threadIdx.x % W, first = threadIdx.x / W;
      const uint32_t tiles = first < per ? (uint32_t)ntiles : 0u;
      uint32_t before = 0, sum = 0;
      for (uint32_t j = first; j < tiles; j += 8 * per) {
        uint32_t c[8];
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) c[q] = j + q * per < tiles ? cnt[(j + q * per) * W + word] : 0u;
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
          sum += c[q];
          before += j + q * per < b ? c[q] : 0u;
        }
      }
      __syncthreads();
      if (sum) atomicAdd(&all[word], sum);
      if (before) atomicAdd(&start[word], before);
      __syncthreads();
      if (b == 0 && threadIdx.x < 64) publish_split(T, threadIdx.x <= T ? all[threadIdx.x] : 0, cap, res);
    } else {
      if (threadIdx.x < T) start[threadIdx.x] = cnt[b * (T + 1) + threadIdx.x];
    }
#pragma unroll
    for (uint32_t q = 0; q < kSplitItems; ++q) {
      rank[q] = 0;
      for (uint32_t k = 0; k < T; ++k) {
        const uint64_t m = __ballot(t[q] == k);
        if (t[q] == k) rank[q] = (uint32_t)__popcll(m & lt);
        if (lane == 0) rows[q * (kBlock / 64) + wid][k] = (uint32_t)__popcll(m);
      }
    }
    __syncthreads();
    // rows in request order (row q * 4 + wave): their exclusive sums
    if (threadIdx.x < T) {
      uint32_t run = start[threadIdx.x];
      for (uint32_t r = 0; r < kRows; ++r) {
        const uint32_t c = rows[r][threadIdx.x];
        rows[r][threadIdx.x] = run;
        run += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kSplitItems; ++q)
      if (t[q] < T) {
        const uint64_t p = (uint64_t)rows[q * (kBlock / 64) + wid][t[q]] + rank[q];
        if (p < cap) outs.p[t[q]][p] = (int64_t)loc[q];
      }
    __syncthreads();
  }
}

// No requests: every list is empty.
__global__ void k_type_none(uint64_t *res, uint32_t T) {
  if (threadIdx.x < 64) publish_split(T, 0, 0, res);
}

static unsigned grid_for(uint64_t work, uint64_t per_block, unsigned cap) {
  uint64_t b = (work + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

}  // namespace lsm_smp

struct lsmgnn_sampler {
  int device = 0;
  const int64_t *off = nullptr;
  const uint32_t *adj = nullptr;
  uint64_t N = 0, nchunks = 0, chunk = 0;  // byte-map bytes per block
  uint32_t chunk_shift = 0;
  uint32_t hops = 0;
  uint32_t fanout[lsm_smp::kMaxHops] = {};
  uint64_t seed = 0;
  uint8_t *present = nullptr;  // byte map, nchunks * chunk bytes, zero between calls
  uint64_t *chunk_sum = nullptr, *chunk_base = nullptr;
  uint32_t *chunk_first = nullptr;  // only with more than kFusedLarge large chunks
  uint32_t *frontier = nullptr, *node_off = nullptr;
  lsm_smp::Ctl *ctl = nullptr;      // device; its error flag is zero between calls
  uint64_t *res = nullptr;          // device: (list length, status) of the last call queued
  uint64_t *res_host = nullptr, *res_dev = nullptr;  // pinned: the same, read by the blocking call
};

namespace {

struct DeviceScope {
  int prev = -1;
  bool ok = false;
  explicit DeviceScope(int dev) {
    ok = hipGetDevice(&prev) == hipSuccess && hipSetDevice(dev) == hipSuccess;
    if (!ok) (void)hipGetLastError();
  }
  ~DeviceScope() {
    if (prev >= 0) (void)hipSetDevice(prev);
  }
};

void sampler_free(lsmgnn_sampler *s) {
  for (void *p : {(void *)s->present, (void *)s->chunk_sum, (void *)s->chunk_base, (void *)s->chunk_first,
                  (void *)s->frontier, (void *)s->node_off, (void *)s->ctl, (void *)s->res})
    if (p) (void)hipFree(p);
  if (s->res_host) (void)hipHostFree(s->res_host);
  (void)hipGetLastError();
  delete s;
}

template <int kW>
void queue_frontier(lsmgnn_sampler *s, uint32_t fanout, const lsm_smp::Hop &hop, hipStream_t st) {
  using namespace lsm_smp;
  const dim3 g((unsigned)s->nchunks);
  hipLaunchKernelGGL(k_counts<kW>, g, dim3(kBlock), 0, st, s->present, s->off, fanout, s->chunk_sum);
  if (!s->chunk_first) {
    hipLaunchKernelGGL((k_frontier<kW, true>), g, dim3(kBlock), 0, st, s->present, s->off, fanout, s->chunk_sum,
                       s->chunk_first, s->chunk_base, s->frontier, s->node_off, hop, s->ctl);
  } else if constexpr (kW != kWordsSmall) {
    hipLaunchKernelGGL(k_chunk_scan, dim3(1), dim3(kBlock), 0, st, s->chunk_sum, (uint32_t)s->nchunks,
                       s->chunk_first, s->chunk_base, hop, s->ctl);
    hipLaunchKernelGGL((k_frontier<kW, false>), g, dim3(kBlock), 0, st, s->present, s->off, fanout, s->chunk_sum,
                       s->chunk_first, s->chunk_base, s->frontier, s->node_off, hop, s->ctl);
  }
}

template <int G>
void queue_draw(lsmgnn_sampler *s, uint64_t nodes, uint32_t fanout, uint64_t key_hop, int64_t *out, uint64_t cap,
                bool mark, hipStream_t st) {
  using namespace lsm_smp;
  hipLaunchKernelGGL(k_draw<G>, dim3(grid_for(nodes, kBlock / G, kMaxGrid)), dim3(kBlock), 0, st, s->frontier, s->off,
                     s->adj, fanout, key_hop, s->chunk_base, s->chunk_shift, s->node_off, out, cap, s->present,
                     mark ? 1 : 0, s->ctl);
}

// Queue one minibatch's sampling on `st`; (list length, status) goes to res
// (device memory, or pinned memory by its device address).
bool queue_sample(lsmgnn_sampler *s, const int64_t *seeds, uint64_t n_seeds, uint64_t batch, int64_t *out,
                  uint64_t out_cap, uint64_t *res, hipStream_t st) {
  using namespace lsm_smp;
  const uint64_t key_b = derive(derive(s->seed, kLabelSample), batch);
  if (n_seeds)
    hipLaunchKernelGGL(k_seeds, dim3(grid_for(n_seeds, kBlock, kMaxGrid)), dim3(kBlock), 0, st, seeds, n_seeds, s->N,
                       out, out_cap, s->present, s->ctl);
  // with a bad seed the frontier is still built (and the map cleared) from the
  // valid ones; the hops run, and the call reports E_RANGE
  uint64_t nodes = n_seeds < s->N ? n_seeds : s->N;  // bounds the hop's frontier
  for (uint32_t h = 0; h < s->hops; ++h) {
    const bool last = h + 1 == s->hops;
    const uint32_t fan = s->fanout[h];
    const Hop hop{n_seeds, out_cap, last ? res : nullptr, h == 0};
    if (s->N <= kSmallChunkNodes)
      queue_frontier<kWordsSmall>(s, fan, hop, st);
    else
      queue_frontier<kWordsLarge>(s, fan, hop, st);
    const uint64_t key_hop = derive(key_b, h);
    // the fewest lanes that hold a node's draws: with a wave per node, five
    // draws left 59 of 64 lanes idle
    if (fan <= 8)
      queue_draw<8>(s, nodes, fan, key_hop, out, out_cap, !last, st);
    else if (fan <= 16)
      queue_draw<16>(s, nodes, fan, key_hop, out, out_cap, !last, st);
    else if (fan <= 32)
      queue_draw<32>(s, nodes, fan, key_hop, out, out_cap, !last, st);
    else
      queue_draw<64>(s, nodes, fan, key_hop, out, out_cap, !last, st);
    nodes = fan && nodes > s->N / fan ? s->N : nodes * fan;
  }
  return hipGetLastError() == hipSuccess;
}

// The device address of pinned host memory, or NULL for memory that the GPU
// cannot write.
uint64_t *device_view(uint64_t *host) {
  void *p = nullptr;
  if (hipHostGetDevicePointer(&p, host, 0) == hipSuccess && p) return static_cast<uint64_t *>(p);
  (void)hipGetLastError();
  return nullptr;
}

}  // namespace

extern "C" {

lsmgnn_status lsmgnn_sampler_create(const int64_t *offsets, const uint32_t *adj, uint64_t num_nodes,
                                    const uint32_t *fanout, uint32_t hops, uint64_t seed, int device,
                                    lsmgnn_sampler **out) {
  using namespace lsm_smp;
  if (!out) return LSMGNN_E_INVAL;
  *out = nullptr;
  if (!offsets || !fanout || num_nodes == 0 || num_nodes > 0xffffffffull || hops == 0 || hops > kMaxHops)
    return LSMGNN_E_INVAL;
  for (uint32_t h = 0; h < hops; ++h)
    if (fanout[h] > kMaxFanout) return LSMGNN_E_INVAL;
  DeviceScope ds(device);
  if (!ds.ok) return LSMGNN_E_DEVICE;
  const uint64_t N = num_nodes;
  int64_t ends[2] = {0, 0};
  if (hipMemcpy(&ends[0], offsets, 8, hipMemcpyDeviceToHost) != hipSuccess ||
      hipMemcpy(&ends[1], offsets + N, 8, hipMemcpyDeviceToHost) != hipSuccess) {
    (void)hipGetLastError();
    return LSMGNN_E_DEVICE;
  }
  if (ends[0] != 0 || ends[1] < 0 || ends[1] > (int64_t)1 << 40) return LSMGNN_E_RANGE;
  const uint64_t E = (uint64_t)ends[1];
  if (E > 0 && !adj) return LSMGNN_E_INVAL;
  lsmgnn_sampler *s = new (std::nothrow) lsmgnn_sampler;
  if (!s) return LSMGNN_E_NOMEM;
  s->device = device;
  s->off = offsets;
  s->adj = adj;
  s->N = N;
  s->hops = hops;
  s->seed = seed;
  for (uint32_t h = 0; h < hops; ++h) s->fanout[h] = fanout[h];
  s->chunk = (uint64_t)kBlock * 4 * (N <= kSmallChunkNodes ? kWordsSmall : kWordsLarge);
  s->chunk_shift = (uint32_t)__builtin_ctzll(s->chunk);
  s->nchunks = (N + s->chunk - 1) / s->chunk;
  static_assert(kSmallChunkNodes / ((uint64_t)kBlock * 4 * kWordsSmall) <= kFusedSmall,
                "the small chunks' sums are always few");
  uint32_t *err = nullptr;
  bool ok = hipMalloc(&s->present, s->nchunks * s->chunk) == hipSuccess &&
            hipMalloc(&s->chunk_sum, s->nchunks * 8) == hipSuccess &&
            hipMalloc(&s->chunk_base, s->nchunks * 8) == hipSuccess &&
            (N <= kSmallChunkNodes || s->nchunks <= kFusedLarge ||
             hipMalloc(&s->chunk_first, s->nchunks * 4) == hipSuccess) &&
            hipMalloc(&s->frontier, N * 4) == hipSuccess && hipMalloc(&s->node_off, N * 4) == hipSuccess &&
            hipMalloc(&s->ctl, sizeof(Ctl)) == hipSuccess && hipMalloc(&s->res, 16) == hipSuccess &&
            hipHostMalloc(&s->res_host, 16, hipHostMallocDefault) == hipSuccess &&
            hipHostGetDevicePointer(reinterpret_cast<void **>(&s->res_dev), s->res_host, 0) == hipSuccess &&
            hipMalloc(&err, 4) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    if (err) (void)hipFree(err);
    sampler_free(s);
    return LSMGNN_E_NOMEM;
  }
  // the byte map starts zero; the graph is checked once so that no later
  // kernel reads outside it
  uint32_t herr = 0;
  ok = hipMemset(s->present, 0, s->nchunks * s->chunk) == hipSuccess &&
       hipMemset(s->ctl, 0, sizeof(Ctl)) == hipSuccess && hipMemset(err, 0, 4) == hipSuccess;
  if (ok) {
    hipLaunchKernelGGL(k_validate, dim3(grid_for(N > E ? N : E, kBlock, 8192)), dim3(kBlock), 0, 0, offsets, adj, N,
                       E, err);
    ok = hipGetLastError() == hipSuccess && hipMemcpy(&herr, err, 4, hipMemcpyDeviceToHost) == hipSuccess;
  }
  (void)hipFree(err);
  if (!ok) {
    (void)hipGetLastError();
    sampler_free(s);
    return LSMGNN_E_DEVICE;
  }
  if (herr) {
    sampler_free(s);
    return LSMGNN_E_RANGE;
  }
  *out = s;
  return LSMGNN_OK;
}

void lsmgnn_sampler_destroy(lsmgnn_sampler *s) {
  if (!s) return;
  DeviceScope ds(s->device);
  (void)hipDeviceSynchronize();
  sampler_free(s);
}

lsmgnn_status lsmgnn_sample(lsmgnn_sampler *s, const int64_t *seeds, uint64_t n_seeds, uint64_t batch, int64_t *out,
                            uint64_t out_cap, uint64_t *n_out, void *stream) {
  if (!s || !n_out || (n_seeds && !seeds) || (out_cap && !out)) return LSMGNN_E_INVAL;
  DeviceScope ds(s->device);
  if (!ds.ok) return LSMGNN_E_DEVICE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (!queue_sample(s, seeds, n_seeds, batch, out, out_cap, s->res_dev, st) ||
      hipStreamSynchronize(st) != hipSuccess) {
    (void)hipGetLastError();
    return LSMGNN_E_DEVICE;
  }
  *n_out = s->res_host[0];
  return static_cast<lsmgnn_status>(s->res_host[1]);
}

lsmgnn_status lsmgnn_sample_async(lsmgnn_sampler *s, const int64_t *seeds, uint64_t n_seeds, uint64_t batch,
                                  int64_t *out, uint64_t out_cap, uint64_t *result_host, void *stream) {
  if (!s || !result_host || (n_seeds && !seeds) || (out_cap && !out)) return LSMGNN_E_INVAL;
  DeviceScope ds(s->device);
  if (!ds.ok) return LSMGNN_E_DEVICE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the last frontier writes pinned memory itself; other memory gets a copy
  uint64_t *res = device_view(result_host);
  if (!queue_sample(s, seeds, n_seeds, batch, out, out_cap, res ? res : s->res, st) ||
      (!res && hipMemcpyAsync(result_host, s->res, 16, hipMemcpyDeviceToHost, st) != hipSuccess)) {
    (void)hipGetLastError();
    return LSMGNN_E_DEVICE;
  }
  return LSMGNN_OK;
}

uint64_t lsmgnn_split_work_bytes(uint64_t n, uint32_t num_types) {
  return ((n + lsm_smp::kBlock - 1) / lsm_smp::kBlock) * (uint64_t)num_types * 4 + 256;
}

}  // extern "C"

namespace {

// The split's arguments other than the work memory are valid.
bool split_args_ok(const int64_t *ids, uint64_t n, const uint8_t *node_type, const uint32_t *local,
                   uint32_t num_types, int64_t *const *outs, uint64_t out_cap, const uint64_t *result_host) {
  if (!result_host || !outs || !node_type || !local || num_types == 0 || num_types > lsm_smp::kMaxTypes ||
      (n && !ids))
    return false;
  for (uint32_t t = 0; t < num_types; ++t)
    if (out_cap && !outs[t]) return false;
  return true;
}

// Queue the split with `work` (device memory of at least
// lsmgnn_split_work_bytes(n, num_types) bytes) as its work memory.
lsmgnn_status queue_split(const int64_t *ids, uint64_t n, uint64_t num_nodes, const uint8_t *node_type,
                          const uint32_t *local, uint32_t num_types, int64_t *const *outs, uint64_t out_cap,
                          void *work, uint64_t *result_host, hipStream_t st) {
  using namespace lsm_smp;
  TypeOuts to{};
  for (uint32_t t = 0; t < num_types; ++t) to.p[t] = outs[t];
  // work: the device result (num_types lengths + status, 8 B each, used when
  // the result memory is not pinned), then the tile counts: m tiles of
  // num_types + 1 words.  There are 112 bytes and, since n > 1024 (m - 1), at
  // least 4 m - 3 times num_types words for them.
  uint64_t *res = device_view(result_host), *dev = static_cast<uint64_t *>(work);
  const bool copy = !res;
  if (copy) res = dev;
  uint32_t *cnt = reinterpret_cast<uint32_t *>(static_cast<uint8_t *>(work) + kSplitCounts);
  const uint64_t ntiles = (n + kSplitTile - 1) / kSplitTile;
  const unsigned g = grid_for(ntiles, 1, kMaxGrid);
  if (n) {
    hipLaunchKernelGGL(k_type_count, dim3(g), dim3(kBlock), 0, st, ids, n, num_nodes, node_type, num_types, cnt);
    if (ntiles <= kSplitFusedMax) {
      hipLaunchKernelGGL(k_type_scatter<true>, dim3(g), dim3(kBlock), 0, st, ids, n, num_nodes, node_type, local,
                         num_types, cnt, to, out_cap, res);
    } else {
      hipLaunchKernelGGL(k_type_scan, dim3(1), dim3(kBlock), 0, st, cnt, ntiles, num_types, out_cap, res);
      hipLaunchKernelGGL(k_type_scatter<false>, dim3(g), dim3(kBlock), 0, st, ids, n, num_nodes, node_type, local,
                         num_types, cnt, to, out_cap, res);
    }
  } else {
    hipLaunchKernelGGL(k_type_none, dim3(1), dim3(64), 0, st, res, num_types);
  }
  if (hipGetLastError() != hipSuccess ||
      (copy && hipMemcpyAsync(result_host, res, (num_types + 1) * 8, hipMemcpyDeviceToHost, st) != hipSuccess)) {
    (void)hipGetLastError();
    return LSMGNN_E_DEVICE;
  }
  return LSMGNN_OK;
}

}  // namespace

// Work memory of the allocation-free split: one array per device, held until
// the process ends, shared by every call on that device (calls that overlap
// on one device race; every call rewrites all of it that it reads).  Its
// host-side name is not a device address: kernels and copies get the address
// hipGetSymbolAddress returns, looked up once per device.
constexpr uint64_t kSplitScratchBytes = 256 + (uint64_t)(1u << 24) / lsm_smp::kBlock * lsm_smp::kMaxTypes * 4;
static_assert(kSplitScratchBytes == LSMGNN_SPLIT_SCRATCH_BYTES, "header and library disagree on the scratch size");
static __device__ __align__(256) uint8_t scratch[kSplitScratchBytes];

namespace {

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxScratchDevices] = {};

// Device address of `dev`'s scratch array (call with `dev` current), or NULL.
void *scratch_on(int dev) {
  if (dev < 0 || dev >= kMaxScratchDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

}  // namespace

extern "C" {

lsmgnn_status lsmgnn_split_by_type_async(const int64_t *ids, uint64_t n, uint64_t num_nodes, const uint8_t *node_type,
                                         const uint32_t *local, uint32_t num_types, int64_t *const *outs,
                                         uint64_t out_cap, void *work, uint64_t work_bytes, uint64_t *result_host,
                                         void *stream) {
  if (!split_args_ok(ids, n, node_type, local, num_types, outs, out_cap, result_host) || !work ||
      work_bytes < lsmgnn_split_work_bytes(n, num_types))
    return LSMGNN_E_INVAL;
  return queue_split(ids, n, num_nodes, node_type, local, num_types, outs, out_cap, work, result_host,
                     static_cast<hipStream_t>(stream));
}

lsmgnn_status lsmgnn_split_by_type_noalloc_async(const int64_t *ids, uint64_t n, uint64_t num_nodes,
                                                 const uint8_t *node_type, const uint32_t *local, uint32_t num_types,
                                                 int64_t *const *outs, uint64_t out_cap, uint64_t *result_host,
                                                 void *stream) {
  if (!split_args_ok(ids, n, node_type, local, num_types, outs, out_cap, result_host) ||
      lsmgnn_split_work_bytes(n, num_types) > kSplitScratchBytes)
    return LSMGNN_E_INVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  int dev = -1, prev = -1;
  if ((st ? hipStreamGetDevice(st, &dev) : hipGetDevice(&dev)) != hipSuccess || hipGetDevice(&prev) != hipSuccess) {
    (void)hipGetLastError();
    return LSMGNN_E_DEVICE;
  }
  // the lookup must run with the stream's device current
  if (dev != prev && hipSetDevice(dev) != hipSuccess) {
    (void)hipGetLastError();
    return LSMGNN_E_DEVICE;
  }
  void *work = scratch_on(dev);
  const lsmgnn_status rc = work ? queue_split(ids, n, num_nodes, node_type, local, num_types, outs, out_cap, work,
                                              result_host, st)
                                : LSMGNN_E_DEVICE;
  if (dev != prev) (void)hipSetDevice(prev);
  return rc;
}

}  // extern "C"

// Static score on the GPU: the normalized reverse PageRank that the hybrid
// policy's static information is built from (Sec. 4.2; the static policy of
// Sec. 5).
//
// The graph is the sampling adjacency in CSR form: node u lists the neighbours
// it samples, the reverse of the direction features flow in message passing.
// The walk moves from u to a uniformly chosen CSR entry of u with probability
// d (a repeated entry counts each time) and jumps to a uniformly chosen node
// otherwise; a node with no entries always jumps.  K power iterations from the
// uniform vector:
//
//   r'(v) = (1 - d)/N + d * (sum over entries u->v of r(u)/deg(u) + D/N),
//   D = total rank of the nodes without entries,
//
// then score(v) = floor(r(v) / max r * (2^32 - 1)).
//
//   sources   each entry's source node, a tile of entries per block
//   sort      the entries by target: a stable radix sort of (target, source)
//   pull      per iteration, a tile of sorted entries per block: each entry's
//             share r(u)/deg(u) is read, and runs of equal targets are summed
//             by a segmented scan; a run inside one tile is stored, the parts
//             of one that crosses tiles are added with a float64 atomic (so
//             results agree to rounding, not bit for bit)
//   update    r(v) from the sums, the next shares, and per-block partial sums
//             of D and maxima of r
//   scores    the maximum rank, then the scores
//
// The sums come from sorted entries and not from an atomic per entry, whose
// rate bounds a push: 2.5 ms per iteration for 16.8 M entries over 1 M nodes,
// against 94 us for the pull after one sort of 0.37 ms; the whole call of 20
// iterations took 61.8 ms, now 3.0.  Summing in order of a tree also rounds
// less: 1.3e-16 from an 80-bit evaluation in the 2-norm, 6.2e-15 before.  The
// sort needs 16 bytes per entry; where that cannot be had, or there are 2^32
// entries and more, each iteration pushes every entry's share with a hardware
// float64 atomic:
//   push      one thread per entry adds its source's share to its target
//
// The pull reads 8 bytes per entry in order and 8 at random from the shares:
// it is bound by the random reads.  This is a one-time preprocessing step, not
// part of the per-minibatch gather.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "lsmgnn.h"

namespace lsm_pr {

constexpr int kBlock = 256;
constexpr unsigned kMaxGrid = 8192;

static unsigned grid_for(uint64_t work, unsigned cap) {
  uint64_t b = (work + kBlock - 1) / kBlock;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

__device__ __forceinline__ double block_sum(double v) {
  __shared__ double part[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if (lane == 0) part[wid] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kBlock / 64; ++w) t += part[w];
  return t;  // meaningful in thread 0
}

// offsets non-decreasing from 0, every entry < N; a failure sets *err
__global__ __launch_bounds__(kBlock) void k_validate(const int64_t *off, const uint32_t *adj, uint64_t N, uint64_t E,
                                                     uint32_t *err) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  bool bad = false;
  for (uint64_t u = (uint64_t)blockIdx.x * kBlock + threadIdx.x; u < N; u += stride)
    bad |= off[u + 1] < off[u];
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < E; e += stride) bad |= adj[e] >= N;
  if (bad) *err = 1u;
}

constexpr uint32_t kTileItems = 16, kTile = kBlock * kTileItems;  // entries per block of the sort passes
constexpr uint32_t kBins = 256;                                    // most digits of a pass
constexpr uint32_t kPullItems = 8, kPullTile = kBlock * kPullItems;
constexpr unsigned kParts = 1024;  // blocks of the update, and so partial sums

// Block-wide exclusive scan of one value per thread; `op` is + or max on uint32.
template <typename Op>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, Op op) {
  __shared__ uint32_t wsum[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x = op(x, y);
  }
  if (lane == 63) wsum[wid] = x;
  uint32_t ex = __shfl_up(x, 1);
  if (lane == 0) ex = 0;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kBlock / 64; ++w)
    if (w < wid) ex = op(ex, wsum[w]);
  __syncthreads();
  return ex;
}

struct Sum {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; }
};
struct Max {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; }
};

// The last row of [lo, hi) that begins at or before entry e, by one wave's
// 64-way search of the offsets; row lo does.
__device__ __forceinline__ uint64_t last_row_from(const int64_t *off, uint64_t lo, uint64_t hi, uint64_t e) {
  while (hi - lo > 1) {
    const uint64_t step = (hi - lo + 63) / 64, at = lo + (threadIdx.x & 63u) * step;
    const uint64_t m = __ballot(at < hi && (uint64_t)off[at] <= e);  // lane 0 always
    const uint64_t k = 63u - (uint32_t)__clzll((long long)m);
    lo += k * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  return lo;
}

// The source node of each entry of the block's tile: the tile's first row by a
// search of the offsets, the rows that start inside it marked at their first
// entry, and a maximum scan over the marks.  (A thread per row, writing its
// entries one by one, took 2.3 ms where one row holds tens of thousands.)
// 256 rows without entries in a row are followed by a search for the next one
// that has some: walked, a run of 10 M of them took its block 26 ms.
__global__ __launch_bounds__(kBlock) void k_sources(const int64_t *off, uint64_t N, uint64_t E, uint32_t *src) {
  __shared__ uint32_t mark[kTile];
  __shared__ uint64_t first;
  const uint64_t tiles = (E + kTile - 1) / kTile;
  for (uint64_t b = blockIdx.x; b < tiles; b += gridDim.x) {
    const uint64_t e0 = b * kTile, e1 = e0 + kTile < E ? e0 + kTile : E;
    for (uint32_t i = threadIdx.x; i < kTile; i += kBlock) mark[i] = 0;
    if (threadIdx.x < 64) {
      const uint64_t r = last_row_from(off, 0, N, e0);
      if (threadIdx.x == 0) first = r;
    }
    __syncthreads();
    const uint64_t r0 = first;
    for (uint64_t rb = r0 + 1;;) {
      const uint64_t r = rb + threadIdx.x;
      const uint64_t o = r < N ? (uint64_t)off[r] : E;
      const bool in = o < e1, filled = in && (uint64_t)off[r + 1] > o;
      if (filled) mark[o - e0] = (uint32_t)r;
      if (__syncthreads_or(!in)) break;
      rb += kBlock;
      if (__syncthreads_or(filled)) continue;
      if (threadIdx.x < 64) {
        const uint64_t next = last_row_from(off, rb - 1, N, (uint64_t)off[rb - 1]);
        if (threadIdx.x == 0) first = next;
      }
      __syncthreads();
      rb = first;
    }
    uint32_t v[kTileItems], top = threadIdx.x == 0 ? (uint32_t)r0 : 0u;
#pragma unroll
    for (uint32_t q = 0; q < kTileItems; ++q) {
      const uint32_t m = mark[threadIdx.x * kTileItems + q];
      top = m > top ? m : top;
      v[q] = top;
    }
    const uint32_t before = block_scan(top, Max{});
#pragma unroll
    for (uint32_t q = 0; q < kTileItems; ++q)
      mark[threadIdx.x * kTileItems + q] = v[q] > before ? v[q] : before;
    __syncthreads();
    for (uint32_t i = threadIdx.x; e0 + i < e1; i += kBlock) src[e0 + i] = mark[i];
    __syncthreads();
  }
}

// One pass of the sort by `bits` bits of the target from `shift`: digit counts
// per tile (digit-major), a scan of each digit's row, then the scatter.
__global__ __launch_bounds__(kBlock) void k_digit_counts(const uint32_t *key, uint64_t E, uint32_t shift,
                                                         uint32_t bits, uint32_t *cnt, uint32_t tiles) {
  __shared__ uint32_t h[kBins];
  const uint32_t mask = (1u << bits) - 1u;
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t e0 = (uint64_t)blockIdx.x * kTile;
#pragma unroll
  for (uint32_t q = 0; q < kTileItems; ++q) {
    const uint64_t e = e0 + q * kBlock + threadIdx.x;
    if (e < E) atomicAdd(&h[(key[e] >> shift) & mask], 1u);
  }
  __syncthreads();
  if (threadIdx.x <= mask) cnt[(uint64_t)threadIdx.x * tiles + blockIdx.x] = h[threadIdx.x];
}

__global__ __launch_bounds__(kBlock) void k_digit_scan(uint32_t *cnt, uint32_t tiles, uint32_t *total) {
  uint32_t *row = cnt + (uint64_t)blockIdx.x * tiles;
  __shared__ uint32_t last;
  uint32_t carry = 0;
  for (uint32_t base = 0; base < tiles; base += kBlock * 8) {
    const uint32_t i = base + threadIdx.x * 8;
    uint32_t v[8], sum = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) sum += v[q] = i + q < tiles ? row[i + q] : 0u;
    uint32_t run = carry + block_scan(sum, Sum{});
    if (threadIdx.x == kBlock - 1) last = run + sum;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (i + q < tiles) row[i + q] = run;
      run += v[q];
    }
    __syncthreads();
    carry = last;
    __syncthreads();
  }
  if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// Stable scatter of a tile: each wave ranks its 1024 consecutive entries, 64 at
// a time, by ballots over the digit's bits; the tile is put in digit order in
// LDS and written from there, so that consecutive lanes write consecutive
// entries of a digit.
__global__ __launch_bounds__(kBlock) void k_scatter(const uint32_t *key, const uint32_t *val, uint64_t E,
                                                    uint32_t shift, uint32_t bits, const uint32_t *cnt,
                                                    uint32_t tiles, const uint32_t *total, uint32_t *key_out,
                                                    uint32_t *val_out) {
  __shared__ uint32_t lkey[kTile], lval[kTile];
  __shared__ uint32_t wcnt[kBlock / 64][kBins];
  __shared__ uint32_t goff[kBins];
  const uint32_t mask = (1u << bits) - 1u;
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
  const uint64_t e0 = (uint64_t)blockIdx.x * kTile;
  const uint64_t w0 = e0 + wid * (kTile / (kBlock / 64)) + lane;
#pragma unroll
  for (uint32_t w = 0; w < kBlock / 64; ++w) wcnt[w][threadIdx.x] = 0;
  uint32_t k[kTileItems], v[kTileItems], rank[kTileItems];
#pragma unroll
  for (uint32_t q = 0; q < kTileItems; ++q) {
    const uint64_t e = w0 + q * 64;
    k[q] = v[q] = 0;
    if (e < E) {
      k[q] = key[e];
      v[q] = val[e];
    }
  }
  __syncthreads();
#pragma unroll
  for (uint32_t q = 0; q < kTileItems; ++q) {
    const bool in = w0 + q * 64 < E;
    const uint32_t d = (k[q] >> shift) & mask;
    uint64_t m = __ballot(in);
    for (uint32_t bit = 0; bit < bits; ++bit) {
      const bool on = (d >> bit) & 1u;
      const uint64_t bb = __ballot(on);
      m &= on ? bb : ~bb;
    }
    const uint32_t before = wcnt[wid][d];
    rank[q] = before + (uint32_t)__popcll(m & lt);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // one wave's counters: read by all its lanes, then
    __builtin_amdgcn_wave_barrier();                        // advanced by each digit's first lane
    if (in && (m & lt) == 0) wcnt[wid][d] = before + (uint32_t)__popcll(m);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // first entry of each digit in the tile, and in the output
  uint32_t all = 0;
#pragma unroll
  for (uint32_t w = 0; w < kBlock / 64; ++w) all += wcnt[w][threadIdx.x];
  const uint32_t start = block_scan(all, Sum{});
  const uint32_t base = block_scan(threadIdx.x <= mask ? total[threadIdx.x] : 0u, Sum{});
  if (threadIdx.x <= mask) goff[threadIdx.x] = base + cnt[(uint64_t)threadIdx.x * tiles + blockIdx.x] - start;
  uint32_t run = start;
#pragma unroll
  for (uint32_t w = 0; w < kBlock / 64; ++w) {
    const uint32_t c = wcnt[w][threadIdx.x];
    wcnt[w][threadIdx.x] = run;
    run += c;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t q = 0; q < kTileItems; ++q)
    if (w0 + q * 64 < E) {
      const uint32_t l = wcnt[wid][(k[q] >> shift) & mask] + rank[q];
      lkey[l] = k[q];
      lval[l] = v[q];
    }
  __syncthreads();
  const uint32_t n = E - e0 < kTile ? (uint32_t)(E - e0) : kTile;
  for (uint32_t i = threadIdx.x; i < n; i += kBlock) {
    const uint32_t y = lkey[i];
    const uint32_t p = goff[(y >> shift) & mask] + i;
    key_out[p] = y;
    val_out[p] = lval[i];
  }
}

// next[v] = sum of the shares of v's sources (next is zero before).  Each
// thread sums the runs of equal targets in its 8 consecutive entries; a
// segmented scan over the block joins the runs that cross threads.
__global__ __launch_bounds__(kBlock) void k_pull(const uint32_t *dst, const uint32_t *src, uint64_t E,
                                                 const double *share, double *next) {
  constexpr uint32_t kNone = 0xffffffffu;  // no node has this number
  __shared__ double wsum[kBlock / 64];
  __shared__ uint32_t wflag[kBlock / 64];
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  const uint64_t e0 = (uint64_t)blockIdx.x * kPullTile + threadIdx.x * kPullItems;
  uint32_t t[kPullItems];
  double v[kPullItems];
  if (e0 + kPullItems <= E) {
    const uint4 a = *reinterpret_cast<const uint4 *>(dst + e0), b = *reinterpret_cast<const uint4 *>(dst + e0 + 4);
    const uint4 c = *reinterpret_cast<const uint4 *>(src + e0), d = *reinterpret_cast<const uint4 *>(src + e0 + 4);
    t[0] = a.x; t[1] = a.y; t[2] = a.z; t[3] = a.w; t[4] = b.x; t[5] = b.y; t[6] = b.z; t[7] = b.w;
    v[0] = share[c.x]; v[1] = share[c.y]; v[2] = share[c.z]; v[3] = share[c.w];
    v[4] = share[d.x]; v[5] = share[d.y]; v[6] = share[d.z]; v[7] = share[d.w];
  } else {
#pragma unroll
    for (uint32_t q = 0; q < kPullItems; ++q) {
      t[q] = kNone;
      v[q] = 0.0;
      if (e0 + q < E) {
        t[q] = dst[e0 + q];
        v[q] = share[src[e0 + q]];
      }
    }
  }
  uint32_t prev = __shfl_up(t[kPullItems - 1], 1), after = __shfl_down(t[0], 1);
  if (lane == 0) prev = e0 > 0 && e0 <= E ? dst[e0 - 1] : kNone;
  if (lane == 63) after = e0 + kPullItems < E ? dst[e0 + kPullItems] : kNone;
  const bool starts = t[0] != prev;  // the first run begins here

  bool split = false;  // a run ends inside
  double run = 0.0, first = 0.0;
#pragma unroll
  for (uint32_t q = 0; q < kPullItems; ++q) {
    if (q > 0 && t[q] != t[q - 1]) {
      if (!split)
        first = run;
      else
        next[t[q - 1]] = run;  // the whole run is this thread's
      split = true;
      run = 0.0;
    }
    run += v[q];
  }
  // inclusive segmented scan of the run open at each thread's end
  double s = run;
  uint32_t f = split || starts ? 1u : 0u;
#pragma unroll
  for (uint32_t o = 1; o < 64; o <<= 1) {
    const double ys = __shfl_up(s, o);
    const uint32_t yf = __shfl_up(f, o);
    if (lane >= o) {
      s = f ? s : ys + s;
      f |= yf;
    }
  }
  if (lane == 63) {
    wsum[wid] = s;
    wflag[wid] = f;
  }
  __syncthreads();
  double cs = 0.0;  // the run open at the end of the waves before
  uint32_t cf = 0;
  for (uint32_t w = 0; w < wid; ++w) {
    cs = wflag[w] ? wsum[w] : cs + wsum[w];
    cf |= wflag[w];
  }
  double in_s = __shfl_up(s, 1);  // the run open before this thread, and whether it began in the tile
  uint32_t in_f = __shfl_up(f, 1);
  if (lane == 0) {
    in_s = 0.0;
    in_f = 0;
  }
  in_s = in_f ? in_s : cs + in_s;
  in_f |= cf;
  auto close = [&](uint32_t node, double total, bool began) {
    if (node == kNone) return;
    if (began)
      next[node] = total;
    else
      unsafeAtomicAdd(next + node, total);
  };
  // the thread's first run, if it ends inside; which is t[0]'s
  if (split) close(t[0], starts ? first : in_s + first, starts || in_f);
  // the run open at its end, if it ends there; or the tile does
  const bool ends = t[kPullItems - 1] != after;
  if (ends || threadIdx.x == kBlock - 1) {
    const bool own = split || starts;
    close(t[kPullItems - 1], own ? run : in_s + run, ends && (own || in_f));
  }
}

__global__ __launch_bounds__(kBlock) void k_push(const uint32_t *src, const uint32_t *adj, const double *share,
                                                 double *next, uint64_t E) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < E; e += stride) {
    const double s = share[src[e]];
    if (s != 0.0) unsafeAtomicAdd(next + adj[e], s);
  }
}

// Sum, or maximum, of up to kParts non-negative partials, in every thread.
template <bool kMax>
__device__ __forceinline__ double reduce_parts(const double *part, unsigned n) {
  __shared__ double w[kBlock / 64];
  double t = 0.0;
  for (unsigned b = threadIdx.x; b < n; b += kBlock) t = kMax ? fmax(t, part[b]) : t + part[b];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double y = __shfl_xor(t, o);
    t = kMax ? fmax(t, y) : t + y;
  }
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = t;
  __syncthreads();
  t = w[0];
#pragma unroll
  for (int i = 1; i < kBlock / 64; ++i) t = kMax ? fmax(t, w[i]) : t + w[i];
  return t;
}

// r(v): the uniform start (`start`), or from the sums and the dangling mass D
// of the ranks before (dpart); then the shares and the partial sums of D for
// the next iteration, and the sums cleared for it; the last one leaves the
// ranks and their per-block maxima instead.
__global__ __launch_bounds__(kBlock) void k_update(const int64_t *off, uint64_t N, double d, bool start, bool last,
                                                   double *next, double *share, const double *dpart, double *dpart_out,
                                                   unsigned nparts, double *r, double *mpart) {
  double base = 1.0 / (double)N, jump = 0.0;
  if (!start) {
    base = (1.0 - d) / (double)N;
    jump = reduce_parts<false>(dpart, nparts) / (double)N;
  }
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  double dang = 0.0, top = 0.0;
  for (uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v < N; v += stride) {
    const double x = start ? base : base + d * (next[v] + jump);
    if (last) {
      r[v] = x;
      top = fmax(top, x);
    } else {
      next[v] = 0.0;
      const int64_t deg = off[v + 1] - off[v];
      if (deg == 0) dang += x;
      share[v] = deg == 0 ? 0.0 : x / (double)deg;
    }
  }
  if (last) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) top = fmax(top, __shfl_xor(top, o));
    __shared__ double w[kBlock / 64];
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = top;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int i = 1; i < kBlock / 64; ++i) top = fmax(top, w[i]);
      mpart[blockIdx.x] = top;
    }
  } else {
    const double t = block_sum(dang);
    if (threadIdx.x == 0) dpart_out[blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(kBlock) void k_scores(const double *r, uint64_t N, const double *mpart, unsigned nparts,
                                                   uint32_t *score) {
  const double m = reduce_parts<true>(mpart, nparts);
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v < N; v += stride)
    score[v] = (uint32_t)floor(r[v] / m * 4294967295.0);
}

// Sorts the entries by target; *key and *val point at the sorted targets and
// sources in buf (4 arrays of `stride` entries, the last holding the entries'
// sources at the start).
void sort_entries(const uint32_t *adj, uint64_t N, uint64_t E, uint32_t *buf, uint64_t stride, uint32_t *cnt,
                  uint32_t *total, hipStream_t s, const uint32_t **key, const uint32_t **val) {
  uint32_t bits = 1;
  while (bits < 32 && (1ull << bits) < N) ++bits;
  const uint32_t passes = (bits + 7) / 8, width = (bits + passes - 1) / passes;
  const uint32_t tiles = (uint32_t)((E + kTile - 1) / kTile);
  const uint32_t *k_in = adj, *v_in = buf + 3 * stride;
  for (uint32_t p = 0; p < passes; ++p) {
    const uint32_t shift = p * width, w = shift + width <= bits ? width : bits - shift;
    uint32_t *k_out = buf + (p & 1) * 2 * stride, *v_out = k_out + stride;
    hipLaunchKernelGGL(k_digit_counts, dim3(tiles), dim3(kBlock), 0, s, k_in, E, shift, w, cnt, tiles);
    hipLaunchKernelGGL(k_digit_scan, dim3(1u << w), dim3(kBlock), 0, s, cnt, tiles, total);
    hipLaunchKernelGGL(k_scatter, dim3(tiles), dim3(kBlock), 0, s, k_in, v_in, E, shift, w, cnt, tiles, total, k_out,
                       v_out);
    k_in = k_out;
    v_in = v_out;
  }
  *key = k_in;
  *val = v_in;
}

}  // namespace lsm_pr

extern "C" lsmgnn_status lsmgnn_pagerank_scores(const int64_t *offsets, const uint32_t *adj, uint64_t num_nodes,
                                                double damping, uint32_t iterations, uint32_t *scores, double *rank,
                                                int device, void *stream) {
  using namespace lsm_pr;
  if (!offsets || !scores || num_nodes == 0 || num_nodes > 0xffffffffull || !(damping >= 0.0 && damping < 1.0))
    return LSMGNN_E_INVAL;
  int prev = -1;
  if (hipGetDevice(&prev) != hipSuccess || hipSetDevice(device) != hipSuccess) {
    (void)hipGetLastError();
    return LSMGNN_E_DEVICE;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  const uint64_t N = num_nodes;
  lsmgnn_status st = LSMGNN_OK;
  int64_t ends[2] = {0, 0};
  uint32_t *err = nullptr, *buf = nullptr, *src = nullptr;
  double *r = rank, *work = nullptr, *next, *share, *dpart[2], *mpart;
  uint32_t herr = 0;
  uint64_t E = 0, stride = 0, tiles = 0;
  const uint32_t *key = nullptr, *val = nullptr;
  bool sorted = false;
  const unsigned gN = grid_for(N, kParts);
  // the edge count and the first offset, read once the caller's work is done
  if (hipMemcpyAsync(&ends[0], offsets, 8, hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipMemcpyAsync(&ends[1], offsets + N, 8, hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    st = LSMGNN_E_DEVICE;
    goto done;
  }
  if (ends[0] != 0 || ends[1] < 0 || ends[1] > (int64_t)1 << 40) {
    st = LSMGNN_E_RANGE;
    goto done;
  }
  E = (uint64_t)ends[1];
  if (E > 0 && !adj) {
    st = LSMGNN_E_INVAL;
    goto done;
  }
  // float64 work memory: the sums, the shares, the ranks unless the caller
  // takes them, the partials
  if (hipMalloc(&err, 4) != hipSuccess ||
      hipMalloc(&work, ((rank ? 2 : 3) * N + 3 * (uint64_t)kParts) * 8) != hipSuccess) {
    (void)hipGetLastError();
    st = LSMGNN_E_NOMEM;
    goto done;
  }
  next = work;
  share = next + N;
  dpart[0] = share + N;
  dpart[1] = dpart[0] + kParts;
  mpart = dpart[1] + kParts;
  if (!r) r = mpart + kParts;
  if (hipMemsetAsync(err, 0, 4, s) != hipSuccess) {
    st = LSMGNN_E_DEVICE;
    goto done;
  }
  hipLaunchKernelGGL(k_validate, dim3(grid_for(N > E ? N : E, kMaxGrid)), dim3(kBlock), 0, s, offsets, adj, N, E, err);
  if (hipMemcpyAsync(&herr, err, 4, hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess) {
    st = LSMGNN_E_DEVICE;
    goto done;
  }
  if (herr) {
    st = LSMGNN_E_RANGE;
    goto done;
  }
  if (E) {
    // the sort's arrays (16-byte aligned rows) and digit counts, or at least
    // the entries' sources
    stride = (E + 63) / 64 * 64;
    tiles = (E + kTile - 1) / kTile;
    sorted = E < 1ull << 32 && iterations > 0 &&
             hipMalloc(&buf, (4 * stride + (tiles + 1) * kBins) * 4) == hipSuccess;
    if (!sorted) {
      (void)hipGetLastError();
      if (iterations > 0 && hipMalloc(&buf, E * 4) != hipSuccess) {
        (void)hipGetLastError();
        st = LSMGNN_E_NOMEM;
        goto done;
      }
    }
    src = sorted ? buf + 3 * stride : buf;
    if (iterations > 0)
      hipLaunchKernelGGL(k_sources, dim3(grid_for((E + kTileItems - 1) / kTileItems, 1u << 20)), dim3(kBlock), 0, s, offsets, N,
                         E, src);
    if (sorted)
      sort_entries(adj, N, E, buf, stride, buf + 4 * stride + kBins, buf + 4 * stride, s, &key, &val);
  }
  hipLaunchKernelGGL(k_update, dim3(gN), dim3(kBlock), 0, s, offsets, N, damping, true, iterations == 0, next, share,
                     dpart[0], dpart[0], gN, r, mpart);
  for (uint32_t k = 0; k < iterations; ++k) {
    if (sorted)
      hipLaunchKernelGGL(k_pull, dim3((unsigned)((E + kPullTile - 1) / kPullTile)), dim3(kBlock), 0, s, key, val, E,
                         share, next);
    else if (E)
      hipLaunchKernelGGL(k_push, dim3(grid_for(E, kMaxGrid)), dim3(kBlock), 0, s, src, adj, share, next, E);
    hipLaunchKernelGGL(k_update, dim3(gN), dim3(kBlock), 0, s, offsets, N, damping, false, k + 1 == iterations, next,
                       share, dpart[k & 1], dpart[(k + 1) & 1], gN, r, mpart);
  }
  hipLaunchKernelGGL(k_scores, dim3(gN), dim3(kBlock), 0, s, r, N, mpart, gN, scores);
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) st = LSMGNN_E_DEVICE;
done:
  (void)hipStreamSynchronize(s);
  for (void *p : {(void *)err, (void *)work, (void *)buf})
    if (p) (void)hipFree(p);
  (void)hipGetLastError();
  if (prev >= 0) (void)hipSetDevice(prev);
  return st;
}

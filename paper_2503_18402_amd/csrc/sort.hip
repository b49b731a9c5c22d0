// Binning: one (tile, Gaussian) pair per tile of every visible footprint,
// grouped by tile, ordered within a tile by (depth, Gaussian index), plus the
// per-tile ranges.
//
// That order is the one of the stable ascending sort of
// key = (tile_id << 32) | bits(depth_f32) over pairs emitted in Gaussian index
// order.  Because the index breaks every tie, the order is unique, so any
// correct sort produces it.  Instead of sorting all pairs globally on every key
// digit, the pairs are bucketed by tile and each tile's (short) list is sorted
// on chip:
//   0. offsets: each pair's position in index order (Gaussian by Gaussian,
//              tiles row-major in its box) from a scan of the tile counts;
//   1. count:  one atomic increment per pair on its tile's counter; the
//              value it returns is the pair's rank in its tile, kept at the
//              pair's index-order position;
//   2. scan:   one block scans the counters into each tile's first slot and
//              checks the pair total against the capacity;
//   3. bucket: every pair stores the 64-bit sort key
//              (bits(depth_f32) << 32) | Gaussian index at its tile's first
//              slot plus its rank: no atomics;
//   4. sort:   each tile's keys are sorted by a bitonic network on 32-bit words and
//              the values written (and the keys when asked for): lists of up to
//              512 keys by one wave in registers, up to 2048 by a 256-thread
//              block in registers with LDS exchanges for the strides that
//              cross waves, longer ones by a 1024-thread block (lists of more
//              than 8192 keys merge their sorted chunks on the 64-bit keys).
// Launches of few Gaussians and tiles run in one kernel instead (k_bin_direct).
// The slot order after step 3 depends on atomic timing; after step 4 it does
// not.  A block whose pairs fall on at most 2048 tiles it can index (all tiles
// of its view at low resolutions, where every tile collects thousands of
// pairs; or the bounding rectangle of its footprints' tiles, when its
// Gaussians sit close together in space) counts in LDS first and reserves one
// slot range per touched tile in step 3 instead, through a cursor that starts
// after the tile's ranked pairs.  The counters, cursors and first slots live in
// the caller's ranges array (during steps 1-3: ranges[2t] = ranked count, then
// first slot; ranges[2t+1] = LDS-counted count, then cursor, then end), so the
// workspace holds the bucketed keys, the ranks, the offsets' block sums and
// four counts.
//
// The pair expansion spreads each block's pairs evenly over its threads, so a
// Gaussian with a footprint of thousands of tiles does not serialise on one lane.
#include <algorithm>
#include <mutex>

#include "scan.hpp"

namespace gsk {
namespace {

struct TileInfo {  // per view: first global tile, one past its last tile, grid width
  int32_t tile_base[GS_MAX_VIEWS];
  int32_t tile_end[GS_MAX_VIEWS];
  int32_t gw[GS_MAX_VIEWS];
};

constexpr int kXT = 256;        // threads per expansion block

struct Items {  // the (view, Gaussian) items of a preprocess output
  TileInfo TI;
  const char* proj;
  size_t stride, tt_off;
  char* goff_proj;  // non-null: record each item's first pair position (at goff_off)
  size_t goff_off;
  int n;
  int tile_log2;
  int rounds;  // a block takes kXT * rounds items of one view,
  int bpv;     // a view bpv blocks
  // views, most tiles first: the launch's last blocks are light (16 views of mixed sizes,
  // fewest tiles first: count and place 306 + 442 us, so 262 + 312)
  int order[GS_MAX_VIEWS];
};

// Which items a block takes.  `id` numbers the blocks in index order.
struct BlockItems {
  int v, id;
  int64_t g0;  // first Gaussian
};
__device__ __forceinline__ BlockItems block_items(const Items& S) {
  const int slot = int(blockIdx.x) / S.bpv, c = int(blockIdx.x) - slot * S.bpv;
  BlockItems b;
  b.v = S.order[slot];
  b.id = b.v * S.bpv + c;
  b.g0 = int64_t(c) * kXT * S.rounds;
  return b;
}

constexpr int kAggBins = 2048;  // most tiles a block aggregates in LDS
constexpr int kAggRounds = 4;   // items per aggregating block: at most kXT * kAggRounds
// (4 items a thread: 1024-item blocks leave the last ones of a launch less to do than
// 2048-item blocks, 16 views of mixed sizes: 199 + 234 us against 262 + 312; 512-item
// blocks there 142 + 238, but 434 + 780 against 400 + 720 at 16 views of 4M Gaussians,
// with twice the blocks' positions to scan, 55 us against 30)
// but no fewer blocks than this while items allow: each block walks its rounds
// one after the other (load, scan, LDS bins), so 2048 blocks (8 per CU) hide
// that latency; at 1M Gaussians on views of a few hundred tiles, 512 blocks
// took 1.8-2.3x as long when the Gaussians are stored in spatial order (blocks
// touch few tiles), while in index order (every block touches most tiles) the
// 4x more reservation atomics cost 1.4x
constexpr int kAggBlocks = 2048;

// An item's footprint box and depth, read once per kernel: a block's kXT * rounds
// items stay in registers between its passes over them (their records lie 48 bytes
// apart, so a pass over memory moves three times what it uses).
struct Item {
  uint32_t lo, hi, z;  // lo > hi in x: no pairs
  __device__ bool visible() const { return box_x(lo) <= box_x(hi); }
};
constexpr uint32_t kNoBox = 1u;

__device__ __forceinline__ Item load_item(const Items& S, int v, int64_t g) {
  Item it{kNoBox, 0u, 0u};
  if (g < S.n) {
    const char* pv = S.proj + size_t(v) * S.stride;
    if (reinterpret_cast<const uint32_t*>(pv + S.tt_off)[g] > 0u) {
      const float4 r2 = reinterpret_cast<const float4*>(pv)[3 * g + 2];
      it.z = __float_as_uint(r2.y);
      it.lo = __float_as_uint(r2.z);
      it.hi = __float_as_uint(r2.w);
    }
  }
  return it;
}

// Calls f(global tile id, sort key, index-order position, tile x | tile y << 16
// in its view's grid) once for every pair of view v's items [first, first + kXT),
// whose first pair sits at index-order position pbase; `it` is the thread's item.
// The pairs are dealt to the block's threads in turn, kPairs of them a thread and
// step: f.issue() starts a pair's atomic or loads, f.commit() uses what it returned,
// so their latencies overlap.  (One pair a step over the owning wave's lanes alone:
// a footprint of thousands of tiles then keeps its wave, and at the end the whole
// launch, for one round trip per 64 pairs: 16 views of mixed sizes of 1M Gaussians
// stored by place, whose fullest block has 78 thousand pairs and its fullest wave 11
// thousand, counted in 445 us and placed in 515 so; dealt to the block 306 and 442, with
// the launch's order of views and 1024-item blocks 199 and 234.)  Every thread of the block
// must call it.  Returns the items' pair count.
constexpr int kPairs = 4;

template <class F>
__device__ inline uint32_t for_each_pair(const Items& S, int v, int64_t first, const Item& it,
                                         uint32_t pbase, F&& f) {
  __shared__ uint32_t s_end[kXT];   // inclusive prefix of pair counts
  __shared__ uint32_t s_wtot[kXT / 64];
  __shared__ uint32_t s_base[kXT];  // global id of the footprint's first tile
  __shared__ uint32_t s_w[kXT];     // footprint width in tiles
  __shared__ uint64_t s_key[kXT];   // bits(depth) << 32 | Gaussian index
  __shared__ uint32_t s_xy[kXT];    // footprint's first tile: x | y << 16
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t g = first + tid;
  const uint32_t gw = uint32_t(S.TI.gw[v]);
  uint32_t cnt = 0, base = 0, w = 1, xy = 0;
  uint64_t key = 0;
  if (it.visible()) {
    const int tx0 = box_x(it.lo) >> S.tile_log2, ty0 = box_y(it.lo) >> S.tile_log2;
    const int tx1 = box_x(it.hi) >> S.tile_log2, ty1 = box_y(it.hi) >> S.tile_log2;
    w = uint32_t(tx1 - tx0 + 1);
    cnt = w * uint32_t(ty1 - ty0 + 1);
    base = uint32_t(S.TI.tile_base[v]) + uint32_t(ty0) * gw + uint32_t(tx0);
    xy = uint32_t(tx0) | (uint32_t(ty0) << 16);
    key = (uint64_t(it.z) << 32) | uint64_t(g);
  }
  uint32_t inc = wave_incl_scan(cnt);
  if (lane == 63) s_wtot[tid >> 6] = inc;
  s_base[tid] = base;
  s_w[tid] = w;
  s_key[tid] = key;
  s_xy[tid] = xy;
  __syncthreads();
  uint32_t all = 0;
#pragma unroll
  for (int w = 0; w < kXT / 64; ++w) {
    const uint32_t t = s_wtot[w];
    inc += (w < (tid >> 6)) ? t : 0u;
    all += t;
  }
  s_end[tid] = inc;
  if (S.goff_proj && g < S.n)
    reinterpret_cast<uint32_t*>(S.goff_proj + size_t(v) * S.stride + S.goff_off)[g] =
        pbase + (inc - cnt);
  __syncthreads();
  for (uint32_t j0 = uint32_t(tid); j0 < all; j0 += kPairs * kXT) {
    uint32_t t[kPairs], at[kPairs], xy[kPairs], got[kPairs];
#pragma unroll
    for (int u = 0; u < kPairs; ++u) {
      const uint32_t j = j0 + u * kXT;
      if (j < all) {
        // the item owning pair j: the first k with s_end[k] > j
        int k = 0;
#pragma unroll
        for (int step = kXT / 2; step > 0; step >>= 1)
          if (s_end[k + step - 1] <= j) k += step;
        const uint32_t local = j - (k > 0 ? s_end[k - 1] : 0u);
        const uint32_t wk = s_w[k];
        const uint32_t ty = local / wk, tx = local - ty * wk;
        at[u] = uint32_t(k);
        t[u] = s_base[k] + ty * gw + tx;
        xy[u] = s_xy[k] + tx + (ty << 16);
      }
    }
#pragma unroll
    for (int u = 0; u < kPairs; ++u) {
      const uint32_t j = j0 + u * kXT;
      if (j < all) got[u] = f.issue(t[u], pbase + j, xy[u]);
    }
#pragma unroll
    for (int u = 0; u < kPairs; ++u) {
      const uint32_t j = j0 + u * kXT;
      if (j < all) f.commit(got[u], s_key[at[u]], pbase + j);
    }
  }
  __syncthreads();  // the arrays are rewritten by the next call
  return all;
}

// Pair count of each block's items (the block decomposition of k_tile_count
// and k_bucket), from which block_first (or, for many blocks, k_tile_spine) forms
// each block's first index-order position.  Also clears the tiles' counters
// (p[0, np), and their copies q[0, nq)) for k_tile_count.
__global__ __launch_bounds__(kXT) void k_tile_reduce(Items S, uint32_t* __restrict__ block_pairs,
                                                     uint32_t* __restrict__ p, int64_t np,
                                                     uint32_t* __restrict__ q, int64_t nq) {
  __shared__ uint32_t s_w[kXT / 64];
  const int64_t t0 = int64_t(blockIdx.x) * kXT + threadIdx.x, nt = int64_t(gridDim.x) * kXT;
  for (int64_t i = t0; i < np; i += nt) p[i] = 0u;
  for (int64_t i = t0; i < nq; i += nt) q[i] = 0u;
  if (S.n == 0) return;
  const BlockItems B = block_items(S);
  const uint32_t* tt =
      reinterpret_cast<const uint32_t*>(S.proj + size_t(B.v) * S.stride + S.tt_off);
  uint32_t acc = 0;
  for (int r = 0; r < S.rounds; ++r) {
    const int64_t g = B.g0 + int64_t(r) * kXT + threadIdx.x;
    if (g < S.n) acc += tt[g];
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) acc += uint32_t(__shfl_xor(int(acc), d, 64));
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < kXT / 64; ++w) t += s_w[w];
    block_pairs[B.id] = t;
  }
}

// Many blocks: their pair counts into their first index-order positions, in place.
// One block, kSpineItems counts a thread and step, a wave's 64 kSpineItems in a row.
constexpr int kSpineThreads = 1024;
constexpr int kSpineItems = 16;

__global__ __launch_bounds__(kSpineThreads) void k_tile_spine(uint32_t* __restrict__ pos, int n) {
  __shared__ uint32_t s_w[kSpineThreads / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (int base = 0; base < n; base += kSpineThreads * kSpineItems) {
    const int i0 = base + wv * 64 * kSpineItems + lane;
    uint32_t c[kSpineItems], inc[kSpineItems], s = 0;
#pragma unroll
    for (int k = 0; k < kSpineItems; ++k) c[k] = i0 + 64 * k < n ? pos[i0 + 64 * k] : 0u;
#pragma unroll
    for (int k = 0; k < kSpineItems; ++k) inc[k] = wave_incl_scan(c[k]);
#pragma unroll
    for (int k = 0; k < kSpineItems; ++k) {
      const uint32_t t = __shfl(inc[k], 63, 64);
      inc[k] += s;
      s += t;
    }
    if (lane == 0) s_w[wv] = s;
    __syncthreads();
    uint32_t before = carry, all = 0;
#pragma unroll
    for (int q = 0; q < kSpineThreads / 64; ++q) {
      const uint32_t t = s_w[q];
      before += q < wv ? t : 0u;
      all += t;
    }
#pragma unroll
    for (int k = 0; k < kSpineItems; ++k)
      if (i0 + 64 * k < n) pos[i0 + 64 * k] = before + inc[k] - c[k];
    carry += all;
    __syncthreads();  // s_w is rewritten by the next step
  }
}

// The block's first index-order position: `pos` holds the blocks' positions when
// `scanned`, else their pair counts, which every block adds up to its own: up to
// kSpineBlocks of them, 16 loads a thread from L2, that costs less than a launch
// of one block between the two kernels (10 us with it at 1M Gaussians, 2 without).  Every thread of the block
// must call it.
constexpr unsigned kSpineBlocks = 4096;

__device__ inline uint32_t block_first(const uint32_t* __restrict__ pos, int id, bool scanned) {
  if (scanned) return pos[id];
  __shared__ uint32_t s_p[kXT / 64];
  uint32_t acc = 0;
  for (unsigned j = threadIdx.x; int(j) < id; j += kXT) acc += pos[j];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) acc += uint32_t(__shfl_xor(int(acc), d, 64));
  if ((threadIdx.x & 63) == 0) s_p[threadIdx.x >> 6] = acc;
  __syncthreads();
  acc = 0;
#pragma unroll
  for (int w = 0; w < kXT / 64; ++w) acc += s_p[w];
  return acc;
}

// A block takes kXT * rounds consecutive items of a view.  It counts its pairs per
// tile in LDS first and issues one global atomic per touched tile when its pairs
// fall on at most kAggBins tiles that it can index:
//   - all tiles of the view (low resolutions, where
//     every tile collects thousands of pairs and same-counter atomics
//     serialise), bin = tile - first tile of the view; or
//   - the bounding rectangle of their footprints'
//     tiles (Gaussians stored close together in space, as the spatial order
//     stores them, cover few tiles), bin = row-major cell of that rectangle.
// Otherwise every pair goes to the global counters and ranks itself there.
struct BlockSpan : BlockItems {
  int32_t mode;      // 0: global counters, 1: the view's tiles, 2: the rectangle
  int32_t bx0, by0, bw, gw, base;  // mode 2: rectangle origin and width; view's grid
  int32_t span;      // bins in use
  __device__ int bin(uint32_t t, uint32_t xy) const {
    return mode == 1 ? int(t) - base
                     : (int(xy >> 16) - by0) * bw + (int(xy & 0xffffu) - bx0);
  }
  __device__ uint32_t tile_of(int b) const {
    if (mode == 1) return uint32_t(base + b);
    const int y = b / bw, x = b - y * bw;
    return uint32_t(base + (by0 + y) * gw + bx0 + x);
  }
};

// Loads the block's items (the thread's are it[0, rounds)) and decides its mode; every
// thread of the block must call it.
template <int R>
__device__ inline BlockSpan block_span(const Items& S, Item (&it)[R]) {
  BlockSpan b{};
  static_cast<BlockItems&>(b) = block_items(S);
#pragma unroll
  for (int r = 0; r < R; ++r)
    it[r] = r < S.rounds ? load_item(S, b.v, b.g0 + int64_t(r) * kXT + threadIdx.x)
                         : Item{kNoBox, 0u, 0u};
  b.gw = S.TI.gw[b.v];
  b.base = S.TI.tile_base[b.v];
  b.span = S.TI.tile_end[b.v] - b.base;
  b.mode = b.span <= kAggBins ? 1 : 0;
  if (b.mode == 1) return b;  // block-uniform
  // the tile rectangle of the block's footprints
  int x0 = 1 << 30, y0 = 1 << 30, x1 = -1, y1 = -1;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (it[r].visible()) {
      x0 = min(x0, box_x(it[r].lo) >> S.tile_log2);
      y0 = min(y0, box_y(it[r].lo) >> S.tile_log2);
      x1 = max(x1, box_x(it[r].hi) >> S.tile_log2);
      y1 = max(y1, box_y(it[r].hi) >> S.tile_log2);
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    x0 = min(x0, __shfl_xor(x0, d, 64));
    y0 = min(y0, __shfl_xor(y0, d, 64));
    x1 = max(x1, __shfl_xor(x1, d, 64));
    y1 = max(y1, __shfl_xor(y1, d, 64));
  }
  __shared__ int s_r[4][kXT / 64];
  if ((threadIdx.x & 63) == 0) {
    s_r[0][threadIdx.x >> 6] = x0;
    s_r[1][threadIdx.x >> 6] = y0;
    s_r[2][threadIdx.x >> 6] = x1;
    s_r[3][threadIdx.x >> 6] = y1;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kXT / 64; ++w) {
    x0 = min(x0, s_r[0][w]);
    y0 = min(y0, s_r[1][w]);
    x1 = max(x1, s_r[2][w]);
    y1 = max(y1, s_r[3][w]);
  }
  __syncthreads();  // s_r is rewritten by the next call
  if (x1 >= x0 && int64_t(x1 - x0 + 1) * (y1 - y0 + 1) <= kAggBins) {
    b.mode = 2;
    b.bx0 = x0;
    b.by0 = y0;
    b.bw = x1 - x0 + 1;
    b.span = b.bw * (y1 - y0 + 1);
  }
  return b;
}

// The counter an LDS-counting block reserves through for global tile t: with
// `copies` (launches of at most kAggBins tiles, where the same few hundred
// counters receive one atomic from nearly every block) one of kXcds copies,
// chosen by the block, so each copy sees an eighth of those atomics; else the
// tile's ranges[2t + 1].
__device__ __forceinline__ uint32_t* agg_counter(uint32_t* ranges, uint32_t* copies, uint32_t t) {
  return copies ? copies + (blockIdx.x % kXcds) * kAggBins + t : ranges + 2 * size_t(t) + 1;
}

// ---- what the passes do with a pair
struct CountLds {  // count it in the block's bins
  const BlockSpan& B;
  uint32_t* bins;
  __device__ uint32_t issue(uint32_t t, uint32_t, uint32_t xy) const {
    atomicAdd(&bins[B.bin(t, xy)], 1u);
    return 0u;
  }
  __device__ void commit(uint32_t, uint64_t, uint32_t) const {}
};
struct CountRank {  // the returned count is the pair's rank among its tile's ranked pairs
  uint32_t* ranges;
  uint32_t* rank;
  int64_t cap;
  __device__ uint32_t issue(uint32_t t, uint32_t, uint32_t) const {
    return atomicAdd(&ranges[2 * size_t(t)], 1u);
  }
  __device__ void commit(uint32_t got, uint64_t, uint32_t p) const {
    if (int64_t(p) < cap) rank[p] = got;
  }
};
struct PlaceLds {  // the next slot of the block's reservation
  const BlockSpan& B;
  uint32_t* bins;
  uint64_t* bucket;
  __device__ uint32_t issue(uint32_t t, uint32_t, uint32_t xy) const {
    return atomicAdd(&bins[B.bin(t, xy)], 1u);
  }
  __device__ void commit(uint32_t got, uint64_t key, uint32_t) const { bucket[got] = key; }
};
struct PlaceRank {
  const uint32_t* ranges;
  const uint32_t* rank;
  uint64_t* bucket;
  __device__ uint32_t issue(uint32_t t, uint32_t p, uint32_t) const {
    return ranges[2 * size_t(t)] + rank[p];
  }
  __device__ void commit(uint32_t got, uint64_t key, uint32_t) const { bucket[got] = key; }
};

template <int R>
__global__ __launch_bounds__(kXT) void k_tile_count(Items S,
                                                    const uint32_t* __restrict__ block_pos,
                                                    bool scanned, int64_t cap,
                                                    uint32_t* __restrict__ ranges,
                                                    uint32_t* __restrict__ rank,
                                                    uint32_t* __restrict__ copies) {
  extern __shared__ uint32_t s_bins[];
  Item it[R];
  const BlockSpan B = block_span(S, it);
  uint32_t pos = block_first(block_pos, B.id, scanned);  // for the items' pair offsets
  if (B.mode) {
    for (int b = threadIdx.x; b < B.span; b += kXT) s_bins[b] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < S.rounds)
        pos += for_each_pair(S, B.v, B.g0 + int64_t(r) * kXT, it[r], pos, CountLds{B, s_bins});
    for (int b = threadIdx.x; b < B.span; b += kXT)
      if (s_bins[b]) atomicAdd(agg_counter(ranges, copies, B.tile_of(b)), s_bins[b]);
  } else {
    // the returned count is the pair's rank among its tile's ranked pairs
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < S.rounds)
        pos += for_each_pair(S, B.v, B.g0 + int64_t(r) * kXT, it[r], pos,
                             CountRank{ranges, rank, cap});
  }
}

// Places every pair's key in its tile's bucket: a ranked pair at the tile's
// first slot plus its rank; with LDS bins the block first reserves one
// contiguous slot range per touched tile from the tile's cursor (which starts
// after the ranked pairs), then ranks its pairs inside it with LDS atomics.
template <int R>
__global__ __launch_bounds__(kXT) void k_bucket(Items S,
                                                const int64_t* __restrict__ n_eff,
                                                const uint32_t* __restrict__ block_pos,
                                                bool scanned,
                                                const uint32_t* __restrict__ rank,
                                                uint32_t* __restrict__ ranges,
                                                uint32_t* __restrict__ copies,
                                                uint64_t* __restrict__ bucket) {
  extern __shared__ uint32_t s_bins[];
  if (*n_eff == 0) return;  // capacity overflow (or no pairs): nothing to place
  Item it[R];
  const BlockSpan B = block_span(S, it);
  if (B.mode) {
    for (int b = threadIdx.x; b < B.span; b += kXT) s_bins[b] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < S.rounds)
        for_each_pair(S, B.v, B.g0 + int64_t(r) * kXT, it[r], 0u, CountLds{B, s_bins});
    // a thread's bins are b = t + u kXT, u < kAggBins / kXT: all their
    // reservation atomics are issued before the first result is used, so the
    // returns' latencies overlap
    constexpr int kU = kAggBins / kXT;
    uint32_t got[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int b = int(threadIdx.x) + u * kXT;
      const uint32_t k = b < B.span ? s_bins[b] : 0u;
      got[u] = k ? atomicAdd(agg_counter(ranges, copies, B.tile_of(b)), k) : 0u;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int b = int(threadIdx.x) + u * kXT;
      if (b < B.span && s_bins[b]) s_bins[b] = got[u];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < S.rounds)
        for_each_pair(S, B.v, B.g0 + int64_t(r) * kXT, it[r], 0u, PlaceLds{B, s_bins, bucket});
  } else {
    uint32_t pos = block_first(block_pos, B.id, scanned);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < S.rounds)
        pos += for_each_pair(S, B.v, B.g0 + int64_t(r) * kXT, it[r], pos,
                             PlaceRank{ranges, rank, bucket});
  }
}

// One block: with c_t = ranges[2t] (ranked pairs) + the pairs of LDS-counting
// blocks (ranges[2t+1], or the sum of the tile's kXcds counter copies),
// ranges[2t] = exclusive prefix of c (the tile's first slot) and ranges[2t+1]
// = that prefix plus the ranked pairs (where the LDS-counting blocks' cursor
// starts; with copies, copy x's cursor starts after copies 0..x-1's pairs);
// the pair total, and whether it fits the capacity.  Sums are 64-bit, so an
// overflowing total is always detected.
constexpr int kTS = 1024;

__device__ inline uint64_t wave_incl_scan64(uint64_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  return x;
}

// Bound by the latency of one block's steps: a wave takes 64 ITEMS tiles in a row, 64 a
// load (ITEMS 2, or 4 for more than 2 kTS tiles), and a step's loads run under the one
// before: 8 us at 950 tiles, 37 at 35768, 80 at 81600 (15, 56 and 138 with eight
// consecutive tiles a thread, one load per 64 cache lines).
template <int ITEMS>
__global__ __launch_bounds__(kTS) void k_tile_scan(uint32_t* __restrict__ ranges,
                                                   uint32_t* __restrict__ copies, int n_tiles,
                                                   int64_t* __restrict__ proj_total,
                                                   int64_t cap, int64_t* __restrict__ n_tot,
                                                   int64_t* __restrict__ n_eff,
                                                   int64_t* __restrict__ n_long,
                                                   int64_t* __restrict__ n_mid,
                                                   int64_t* __restrict__ n_pairs_user) {
  __shared__ uint64_t s_w[kTS / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t cr[ITEMS], ag[ITEMS];  // ranked pairs, LDS-counted pairs
  auto load = [&](int i0) {
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int i = i0 + 64 * k;
      cr[k] = ag[k] = 0u;
      if (i < n_tiles) {
        cr[k] = ranges[2 * size_t(i)];
        if (copies) {
#pragma unroll
          for (int x = 0; x < kXcds; ++x) ag[k] += copies[x * kAggBins + i];
        } else {
          ag[k] = ranges[2 * size_t(i) + 1];
        }
      }
    }
  };
  int i0 = wv * 64 * ITEMS + lane;
  load(i0);
  uint64_t carry = 0;
  for (int base = 0; base < n_tiles; base += kTS * ITEMS) {
    uint32_t r[ITEMS];
    uint64_t c[ITEMS], inc[ITEMS], s = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      r[k] = cr[k];
      c[k] = uint64_t(cr[k]) + ag[k];
      inc[k] = wave_incl_scan64(c[k]);
    }
    const int i = i0;
    i0 += kTS * ITEMS;
    if (base + kTS * ITEMS < n_tiles) load(i0);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const uint64_t t = __shfl(inc[k], 63, 64);
      inc[k] += s;
      s += t;
    }
    if (lane == 0) s_w[wv] = s;
    __syncthreads();
    uint64_t before = carry, tot = 0;
#pragma unroll
    for (int q = 0; q < kTS / 64; ++q) {
      const uint64_t t = s_w[q];
      before += (q < wv) ? t : 0u;
      tot += t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const int t = i + 64 * k;
      if (t < n_tiles) {
        const uint64_t ex = before + inc[k] - c[k];
        ranges[2 * size_t(t)] = uint32_t(ex);
        ranges[2 * size_t(t) + 1] = uint32_t(ex + r[k]);
        if (copies) {
          uint32_t cur = uint32_t(ex + r[k]);
#pragma unroll
          for (int x = 0; x < kXcds; ++x) {
            const uint32_t a = copies[x * kAggBins + t];
            copies[x * kAggBins + t] = cur;
            cur += a;
          }
        }
      }
    }
    carry += tot;
  }
  if (threadIdx.x == 0) {
    const int64_t t = int64_t(carry);
    *n_tot = t;
    if (proj_total) *proj_total = t;
    *n_eff = (t <= cap) ? t : 0;
    *n_pairs_user = t;
    *n_long = 0;  // set by the wave sort for lists it leaves to the larger tiers
    *n_mid = 0;
  }
}

// ---- bitonic network without directions: every step puts the smaller key at
// the lower index.  A merge of block size 2h starts with a mirror step
// (i, i ^ (2h - 1)) and continues with plain steps (i, i + d), d = h/2 .. 1.
// Keys at indices >= n act as +infinity: every step with a partner >= n would
// leave it in place, so they are neither stored nor compared.
__device__ inline void step_pair(uint32_t c, uint32_t h, bool mirror, uint32_t& i, uint32_t& l) {
  i = ((c & ~(h - 1)) << 1) | (c & (h - 1));
  l = mirror ? ((i | (2 * h - 1)) - (c & (h - 1))) : (i + h);
}

template <int THREADS>
__device__ inline void net_step(uint64_t* a, uint32_t n, uint32_t half_len, uint32_t h,
                                bool mirror) {
  for (uint32_t c = threadIdx.x; c < half_len; c += THREADS) {
    uint32_t i, l;
    step_pair(c, h, mirror, i, l);
    if (l < n) {
      const uint64_t x = a[i], y = a[l];
      if (y < x) {
        a[i] = y;
        a[l] = x;
      }
    }
  }
  __syncthreads();
}

// full sort of a[0, n) (n <= len, len a power of two) in LDS
template <int THREADS>
__device__ inline void lds_sort(uint64_t* a, uint32_t n, uint32_t len) {
  for (uint32_t h = 1; h < len; h <<= 1) {
    net_step<THREADS>(a, n, len / 2, h, true);
    for (uint32_t d = h >> 1; d > 0; d >>= 1) net_step<THREADS>(a, n, len / 2, d, false);
  }
}

__device__ inline uint32_t pow2_ceil(uint32_t x) {
  return x <= 1u ? 1u : (1u << (32 - __builtin_clz(x - 1u)));
}

template <int THREADS>
__device__ inline void write_sorted(const uint64_t* a, uint32_t n, uint32_t start, uint32_t t,
                                    uint32_t* __restrict__ vals, uint64_t* __restrict__ keys) {
  for (uint32_t i = threadIdx.x; i < n; i += THREADS) {
    const uint64_t k = a[i];
    vals[start + i] = uint32_t(k);
    if (keys) keys[start + i] = (uint64_t(t) << 32) | (k >> 32);
  }
}

// ---- the networks on the 64-bit keys, for lists that the words (below) do not put in
// order: at most kWaveKeys keys by one wave, 8 keys per lane in
// registers (element 8 lane + r in k[r]), padded with +infinity to a power of
// two; the same direction-free network with in-lane steps for strides below 8
// and lane shuffles above, so no LDS and no barriers.
constexpr int kWaveKeys = 512;
constexpr int kSmall = 2048;

__device__ __forceinline__ void cx(uint64_t& a, uint64_t& b) {
  const uint64_t x = a < b ? a : b, y = a < b ? b : a;
  a = x;
  b = y;
}

// lane l reads lane l ^ M.  Within a row of 16 lanes the exchange runs on the
// DPP path of the VALU (xor 1, 2, 3: quad permutes; 7, 15: half-row and row
// mirrors; 8: a rotation), within 32 lanes as a swizzle (xor 4, 16, 31), otherwise as a
// permute through the LDS crossbar
template <int M>
__device__ __forceinline__ uint32_t xor_lane(uint32_t x) {
  const int v = int(x);
  if constexpr (M == 1) return uint32_t(__builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true));
  else if constexpr (M == 2) return uint32_t(__builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true));
  else if constexpr (M == 3) return uint32_t(__builtin_amdgcn_update_dpp(0, v, 0x1B, 0xF, 0xF, true));
  else if constexpr (M == 7) return uint32_t(__builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true));
  else if constexpr (M == 8) return uint32_t(__builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true));
  else if constexpr (M == 15) return uint32_t(__builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true));
  else if constexpr (M < 32) return uint32_t(__builtin_amdgcn_ds_swizzle(v, (M << 10) | 0x1F));
  else return uint32_t(__shfl_xor(v, M, 64));
}

template <int M>
__device__ __forceinline__ uint64_t shfl_xor64(uint64_t x) {
  const uint32_t lo = xor_lane<M>(uint32_t(x));
  const uint32_t hi = xor_lane<M>(uint32_t(x >> 32));
  return (uint64_t(hi) << 32) | lo;
}

// lanes whose stride bit is clear hold the lower element and keep the minimum
template <int M>
__device__ __forceinline__ void cross_step_m(uint64_t (&k)[8], bool lower, bool mirror) {
  uint64_t p[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) p[r] = shfl_xor64<M>(k[mirror ? 7 - r : r]);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const bool lt = p[r] < k[r];
    k[r] = (lower == lt) ? p[r] : k[r];
  }
}

// the same step with a runtime mask, every exchange through the LDS crossbar
// (the block-wide network below measured faster with it than with the
// dispatch over exchange paths)
__device__ __forceinline__ void cross_step_perm(uint64_t (&k)[8], int mask, bool lower,
                                                bool mirror) {
  uint64_t p[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint64_t x = k[mirror ? 7 - r : r];
    const uint32_t lo = uint32_t(__shfl_xor(int(uint32_t(x)), mask, 64));
    const uint32_t hi = uint32_t(__shfl_xor(int(uint32_t(x >> 32)), mask, 64));
    p[r] = (uint64_t(hi) << 32) | lo;
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const bool lt = p[r] < k[r];
    k[r] = (lower == lt) ? p[r] : k[r];
  }
}

// the lane masks the networks use: 2^j for plain steps, 2^j - 1 for mirrors
__device__ __forceinline__ void cross_step(uint64_t (&k)[8], int mask, bool lower, bool mirror) {
  switch (mask) {  // wave-uniform
    case 1: cross_step_m<1>(k, lower, mirror); break;
    case 2: cross_step_m<2>(k, lower, mirror); break;
    case 3: cross_step_m<3>(k, lower, mirror); break;
    case 4: cross_step_m<4>(k, lower, mirror); break;
    case 7: cross_step_m<7>(k, lower, mirror); break;
    case 8: cross_step_m<8>(k, lower, mirror); break;
    case 15: cross_step_m<15>(k, lower, mirror); break;
    case 16: cross_step_m<16>(k, lower, mirror); break;
    case 31: cross_step_m<31>(k, lower, mirror); break;
    case 32: cross_step_m<32>(k, lower, mirror); break;
    default: cross_step_m<63>(k, lower, mirror); break;
  }
}

__device__ inline void wave_sort(uint64_t (&k)[8], uint32_t len) {
  const int lane = threadIdx.x & 63;
  for (uint32_t h = 1; h < len; h <<= 1) {
    if (h == 1) {
      cx(k[0], k[1]); cx(k[2], k[3]); cx(k[4], k[5]); cx(k[6], k[7]);
    } else if (h == 2) {
      cx(k[0], k[3]); cx(k[1], k[2]); cx(k[4], k[7]); cx(k[5], k[6]);
    } else if (h == 4) {
      cx(k[0], k[7]); cx(k[1], k[6]); cx(k[2], k[5]); cx(k[3], k[4]);
    } else {
      cross_step(k, int(2 * h / 8 - 1), (lane & int(h / 8)) == 0, true);
    }
    for (uint32_t d = h >> 1; d > 0; d >>= 1) {
      if (d >= 8) {
        cross_step(k, int(d / 8), (lane & int(d / 8)) == 0, false);
      } else if (d == 4) {
        cx(k[0], k[4]); cx(k[1], k[5]); cx(k[2], k[6]); cx(k[3], k[7]);
      } else if (d == 2) {
        cx(k[0], k[2]); cx(k[1], k[3]); cx(k[4], k[6]); cx(k[5], k[7]);
      } else {
        cx(k[0], k[1]); cx(k[2], k[3]); cx(k[4], k[5]); cx(k[6], k[7]);
      }
    }
  }
}

// The same network over W waves of a block, 8 keys per lane: element
// e = 512 w + 8 lane + r of the block's 512 W keys.  Strides below 8 run
// in-lane and strides below 512 by lane shuffles, as in wave_sort; longer
// ones exchange through LDS (s holds 512 W keys), two barriers each.  Every
// thread of the block must call it with the same len (a power of two, at most
// 512 W); keys at e >= len must be +infinity.
template <int W>
__device__ inline void block_reg_sort(uint64_t (&k)[8], uint32_t len, uint64_t* s) {
  const int lane = threadIdx.x & 63;
  const uint32_t e0 = 512u * uint32_t(threadIdx.x >> 6) + 8u * uint32_t(lane);
  // a wave whose keys all sit at e >= len holds only +infinity, which every
  // step leaves in place (partners of such keys are such keys): it only
  // keeps the barriers
  const bool idle = 512u * uint32_t(threadIdx.x >> 6) >= len;
  // partner e ^ m; the element whose bit hb is clear keeps the minimum
  auto lds_step = [&](uint32_t m, uint32_t hb) {
    if (!idle) {
#pragma unroll
      for (int r = 0; r < 8; ++r) s[e0 + r] = k[r];
    }
    __syncthreads();
    if (!idle) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const uint32_t e = e0 + uint32_t(r);
        const uint64_t p = s[e ^ m];
        const bool lower = (e & hb) == 0u;
        const bool lt = p < k[r];
        k[r] = (lower == lt) ? p : k[r];
      }
    }
    __syncthreads();
  };
  for (uint32_t h = 1; h < len; h <<= 1) {
    if (h >= 512u) {
      lds_step(2 * h - 1, h);
    } else if (!idle) {
      if (h == 1) {
        cx(k[0], k[1]); cx(k[2], k[3]); cx(k[4], k[5]); cx(k[6], k[7]);
      } else if (h == 2) {
        cx(k[0], k[3]); cx(k[1], k[2]); cx(k[4], k[7]); cx(k[5], k[6]);
      } else if (h == 4) {
        cx(k[0], k[7]); cx(k[1], k[6]); cx(k[2], k[5]); cx(k[3], k[4]);
      } else {
        cross_step_perm(k, int(2 * h / 8 - 1), (lane & int(h / 8)) == 0, true);
      }
    }
    for (uint32_t d = h >> 1; d > 0; d >>= 1) {
      if (d >= 512u) {
        lds_step(d, d);
      } else if (idle) {
      } else if (d >= 8u) {
        cross_step_perm(k, int(d / 8), (lane & int(d / 8)) == 0, false);
      } else if (d == 4) {
        cx(k[0], k[4]); cx(k[1], k[5]); cx(k[2], k[6]); cx(k[3], k[7]);
      } else if (d == 2) {
        cx(k[0], k[2]); cx(k[1], k[3]); cx(k[4], k[6]); cx(k[5], k[7]);
      } else {
        cx(k[0], k[1]); cx(k[2], k[3]); cx(k[4], k[5]); cx(k[6], k[7]);
      }
    }
  }
}

// ---- lists sorted as 32-bit words.  A comparator of 64-bit keys costs a compare and
// four selects, of words one v_med3 across lanes (the median with 0 is the smaller,
// with ~0 the larger) and a minimum and a maximum in a lane.  So the network sorts words:
// the key's depth above the list's least, shifted down to what the slot leaves of 32
// bits (23 for 512 keys: exact in a list whose depths lie within a factor of two), over
// the key's slot in the bucket.  Then the keys are fetched in that order, and what shared
// a word's depth is put right on the keys themselves: neighbours exchanged until none
// is out of order.  A list that is not done after kFixPasses (hundreds of equal
// depths) is sorted on its keys by the 64-bit networks instead; and one whose depths are
// seen to come in long runs at once: a quarter as many pairs as the network has places are
// compared as they lie in the bucket, of which about L / 4 are equal with runs of L equal
// depths; above kEqualPairs the runs are longer than the passes can put right.  1M Gaussians
// on one plane facing the camera, 1600x1064: sorts 205 us with the words tried first, 128 so,
// 116 with the 64-bit networks for every list; on two 262, 160 and 139; on 32, where the
// words mostly do, 96, 102 and 140 (pairs above 12: 114, above 8: 136); depths that all
// differ 58, 60 and 140.
constexpr int kFixPasses = 12;
constexpr int kEqualPairs = 16;

__device__ __forceinline__ uint32_t med3(uint32_t a, uint32_t b, uint32_t c) {
  return max(min(a, b), min(max(a, b), c));
}
__device__ __forceinline__ void cxw(uint32_t& a, uint32_t& b) {
  const uint32_t x = min(a, b), y = max(a, b);
  a = x;
  b = y;
}

// lane masks: bit[i] is ~0 in the lanes that keep the larger at stride 2^i
struct LaneBits {
  uint32_t bit[6];
  __device__ __forceinline__ explicit LaneBits(int lane) {
#pragma unroll
    for (int i = 0; i < 6; ++i) bit[i] = ((lane >> i) & 1) ? ~0u : 0u;
  }
};

template <int M, bool MIRROR>
__device__ __forceinline__ void cross_words(uint32_t (&k)[8], const LaneBits& B) {
  constexpr int kBit = MIRROR ? (M + 1) / 2 : M;
  const uint32_t bound = B.bit[__builtin_ctz(kBit)];
  uint32_t p[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) p[r] = xor_lane<M>(k[MIRROR ? 7 - r : r]);
#pragma unroll
  for (int r = 0; r < 8; ++r) k[r] = med3(k[r], p[r], bound);
}

// the plain steps of strides D, D / 2 .. 1 (in elements)
template <int D>
__device__ __forceinline__ void plain_words(uint32_t (&k)[8], const LaneBits& B) {
  if constexpr (D >= 8) {
    cross_words<D / 8, false>(k, B);
    plain_words<D / 2>(k, B);
  } else {
    if constexpr (D >= 4) { cxw(k[0], k[4]); cxw(k[1], k[5]); cxw(k[2], k[6]); cxw(k[3], k[7]); }
    if constexpr (D >= 2) { cxw(k[0], k[2]); cxw(k[1], k[3]); cxw(k[4], k[6]); cxw(k[5], k[7]); }
    cxw(k[0], k[1]); cxw(k[2], k[3]); cxw(k[4], k[5]); cxw(k[6], k[7]);
  }
}

// the stages H, 2 H .. 256 that a list of len needs: mirror step, then the plain ones
template <int H>
__device__ __forceinline__ void stages_words(uint32_t (&k)[8], uint32_t len, const LaneBits& B) {
  if constexpr (H < 512) {
    if (uint32_t(H) >= len) return;
    if constexpr (H == 1) {
      cxw(k[0], k[1]); cxw(k[2], k[3]); cxw(k[4], k[5]); cxw(k[6], k[7]);
    } else if constexpr (H == 2) {
      cxw(k[0], k[3]); cxw(k[1], k[2]); cxw(k[4], k[7]); cxw(k[5], k[6]);
    } else if constexpr (H == 4) {
      cxw(k[0], k[7]); cxw(k[1], k[6]); cxw(k[2], k[5]); cxw(k[3], k[4]);
    } else {
      cross_words<2 * H / 8 - 1, true>(k, B);
    }
    if constexpr (H > 1) plain_words<H / 2>(k, B);
    stages_words<2 * H>(k, len, B);
  }
}

// Sorts a list of n <= 512 W keys (n > 0) by W waves and writes it out; every thread of
// the W waves calls it.  s: 2 * 512 W words of LDS (W 1: the keys; else two buffers of
// words), edge: 2 W keys.  With IN_PLACE the sorted keys go back to the list instead.
// Returns false, with nothing written, if kFixPasses did not do or would not.
template <int W, bool IN_PLACE = false>
__device__ inline bool sort_list_words(uint64_t* list, uint32_t n, uint32_t start, uint32_t t,
                                       uint32_t* s, uint64_t* edge, uint32_t* __restrict__ vals,
                                       uint64_t* __restrict__ keys) {
  constexpr int kSlotBits = W == 1 ? 9 : W == 4 ? 11 : 13;
  static_assert((512 * W) == (1 << kSlotBits), "one slot per key");
  const int lane = threadIdx.x & 63;
  const int w = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  auto sync = [&]() {
    if constexpr (W == 1) __builtin_amdgcn_wave_barrier();
    else __syncthreads();
  };
  const uint32_t len = n <= 8u ? 8u : pow2_ceil(n);
  const uint32_t lanes = len / 8u, q = uint32_t(w * 64 + lane);  // lanes that hold keys
  const bool idle = uint32_t(w * 512) >= len;                    // wave-uniform
  const uint32_t e0 = 8u * q;  // the lane's elements of the sorted list
  uint64_t* s_keys = reinterpret_cast<uint64_t*>(s);
  // slots q, q + lanes ..: a load covers whole cache lines
  uint32_t k[8], dmin = ~0u, dmax = 0u;
  int equal = 0;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t slot = uint32_t(r) * lanes + q;
    const bool have = q < lanes && slot < n;
    const uint64_t key = have ? list[slot] : ~uint64_t(0);
    if (W == 1 && have) s_keys[slot] = key;
    k[r] = uint32_t(key >> 32);
    dmin = have ? min(dmin, k[r]) : dmin;
    dmax = have ? max(dmax, k[r]) : dmax;
    // (the slots of the lower half: every list has them)
    if (r == 1 || r == 3) equal += __builtin_popcountll(__ballot(have && k[r] == k[r > 0 ? r - 1 : 0]));
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    dmin = min(dmin, uint32_t(__shfl_xor(int(dmin), d, 64)));
    dmax = max(dmax, uint32_t(__shfl_xor(int(dmax), d, 64)));
  }
  if constexpr (W > 1) {
    if (lane == 0) {
      edge[w] = (uint64_t(dmin) << 32) | dmax;
      edge[W + w] = uint64_t(equal);
    }
    __syncthreads();
    dmin = uint32_t(edge[lane & (W - 1)] >> 32);
    dmax = uint32_t(edge[lane & (W - 1)]);
    equal = int(edge[W + (lane & (W - 1))]);
#pragma unroll
    for (int d = W / 2; d >= 1; d >>= 1) {
      dmin = min(dmin, uint32_t(__shfl_xor(int(dmin), d, 64)));
      dmax = max(dmax, uint32_t(__shfl_xor(int(dmax), d, 64)));
      equal += __shfl_xor(equal, d, 64);
    }
    equal = __builtin_amdgcn_readfirstlane(equal);
    __syncthreads();
  }
  if (equal > kEqualPairs) return false;
  const uint32_t range = dmax - dmin;
  const int bits = range ? 32 - __builtin_clz(range) : 0;
  const int shift = max(bits - (32 - kSlotBits), 0);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t slot = uint32_t(r) * lanes + q;
    k[r] = (q < lanes && slot < n) ? (((k[r] - dmin) >> shift) << kSlotBits) | slot : ~0u;
  }
  const LaneBits B(lane);
  if (!idle) stages_words<1>(k, len, B);
  if constexpr (W > 1) {
    int buf = 0;
    // partner e ^ m, whose bit hb (a wave's) is the other's; the lower keeps the minimum
    auto lds_step = [&](uint32_t m, uint32_t hb) {
      uint4* mine = reinterpret_cast<uint4*>(s + buf * 512 * W + e0);
      if (!idle) {
        mine[0] = make_uint4(k[0], k[1], k[2], k[3]);
        mine[1] = make_uint4(k[4], k[5], k[6], k[7]);
      }
      __syncthreads();
      if (!idle) {
        const uint4* o = reinterpret_cast<const uint4*>(s + buf * 512 * W + (e0 ^ (m & ~7u)));
        const uint4 a = o[0], b = o[1];
        uint32_t p[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        const bool mirror = m & 1u, lower = (uint32_t(w * 512) & hb) == 0u;  // uniform
        if (mirror) {
          const uint32_t f[8] = {p[7], p[6], p[5], p[4], p[3], p[2], p[1], p[0]};
#pragma unroll
          for (int r = 0; r < 8; ++r) k[r] = lower ? min(k[r], f[r]) : max(k[r], f[r]);
        } else {
#pragma unroll
          for (int r = 0; r < 8; ++r) k[r] = lower ? min(k[r], p[r]) : max(k[r], p[r]);
        }
      }
      buf ^= 1;
    };
    for (uint32_t h = 512; h < len; h <<= 1) {
      lds_step(2 * h - 1, h);
      for (uint32_t d = h >> 1; d >= 512u; d >>= 1) lds_step(d, d);
      if (!idle) plain_words<256>(k, B);
    }
  } else {
    __builtin_amdgcn_wave_barrier();
  }
  // the keys in that order
  uint64_t x[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t slot = k[r] & ((1u << kSlotBits) - 1u);
    x[r] = e0 + uint32_t(r) < n ? (W == 1 ? s_keys[slot] : list[slot]) : ~uint64_t(0);
  }
  auto out_of_order = [&]() {
    uint64_t next = __shfl_down(x[0], 1, 64);
    bool bad = lane < 63 && next < x[7];
#pragma unroll
    for (int r = 0; r < 7; ++r) bad |= x[r + 1] < x[r];
    if constexpr (W > 1) {
      if (lane == 0) edge[2 * w] = x[0];
      if (lane == 63) edge[2 * w + 1] = x[7];
      __syncthreads();
      if (lane == 63 && w + 1 < W) bad |= edge[2 * w + 2] < x[7];
      return __syncthreads_or(bad) != 0;
    } else {
      return __ballot(bad) != 0ull;
    }
  };
  int pass = 0;
  while (out_of_order()) {
    if (++pass > kFixPasses) return false;
    cx(x[0], x[1]); cx(x[2], x[3]); cx(x[4], x[5]); cx(x[6], x[7]);
    cx(x[1], x[2]); cx(x[3], x[4]); cx(x[5], x[6]);
    uint64_t up = __shfl_down(x[0], 1, 64), dn = __shfl_up(x[7], 1, 64);
    if constexpr (W > 1) {
      if (lane == 0) edge[2 * w] = x[0];
      if (lane == 63) edge[2 * w + 1] = x[7];
      __syncthreads();
      if (lane == 63) up = w + 1 < W ? edge[2 * w + 2] : ~uint64_t(0);
      if (lane == 0) dn = w > 0 ? edge[2 * w - 1] : 0ull;
      __syncthreads();
    } else {
      if (lane == 63) up = ~uint64_t(0);
      if (lane == 0) dn = 0ull;
    }
    x[7] = up < x[7] ? up : x[7];
    x[0] = dn > x[0] ? dn : x[0];
  }
  sync();  // every key is fetched
  if constexpr (IN_PLACE) {
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (e0 + uint32_t(r) < n) list[e0 + uint32_t(r)] = x[r];
    sync();
    return true;
  }
  // out through LDS, 64 values in a row a store
  uint32_t* s_out = s;
#pragma unroll
  for (int r = 0; r < 8; ++r)
    if (e0 + uint32_t(r) < n) s_out[e0 + uint32_t(r)] = uint32_t(x[r]);
  sync();
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t i = uint32_t(r * 64 * W) + q;
    if (i < n) vals[start + i] = s_out[i];
  }
  if (keys) {
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (e0 + uint32_t(r) < n)
        keys[start + e0 + uint32_t(r)] = (uint64_t(t) << 32) | (x[r] >> 32);
  }
  sync();  // s is reused by the caller
  return true;
}

// A tile's list of n <= 512 W keys sorted by block_reg_sort and written out.
template <int W>
__device__ inline void sort_list_regs(const uint64_t* __restrict__ bucket, uint32_t start,
                                      uint32_t n, uint32_t t, uint64_t* s,
                                      uint32_t* __restrict__ vals, uint64_t* __restrict__ keys) {
  const uint32_t e0 = 512u * uint32_t(threadIdx.x >> 6) + 8u * uint32_t(threadIdx.x & 63);
  uint64_t k[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t e = e0 + uint32_t(r);
    k[r] = (e < n) ? bucket[start + e] : ~uint64_t(0);
  }
  block_reg_sort<W>(k, pow2_ceil(n), s);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t e = e0 + uint32_t(r);
    if (e < n) {
      vals[start + e] = uint32_t(k[r]);
      if (keys) keys[start + e] = (uint64_t(t) << 32) | (k[r] >> 32);
    }
  }
}

// One wave per tile, four tiles per block: 1M Gaussians at 1600x1064, 6700 lists of 335
// keys, 17 us; 35 with the network on the 64-bit keys.  Also writes every tile's range end
// (or [0,0) everywhere after a capacity overflow) and flags the presence of
// lists for the two larger tiers.
__global__ __launch_bounds__(256) void k_tile_sort_wave(
    int n_tiles, const int64_t* __restrict__ n_tot, const int64_t* __restrict__ n_eff,
    int64_t* __restrict__ n_mid, int64_t* __restrict__ n_long,
    uint64_t* __restrict__ bucket, uint32_t* __restrict__ vals,
    uint64_t* __restrict__ keys, uint32_t* __restrict__ ranges) {
  __shared__ __align__(16) uint32_t s_words[4][2 * kWaveKeys];
  const int lane = threadIdx.x & 63;
  const uint32_t t = blockIdx.x * 4u + (threadIdx.x >> 6);
  if (t >= uint32_t(n_tiles)) return;  // wave-uniform; no block barrier below
  if (*n_eff == 0) {
    if (lane == 0) {
      ranges[2 * size_t(t)] = 0u;
      ranges[2 * size_t(t) + 1] = 0u;
    }
    return;
  }
  // each wave writes only its own range end (the cursor has counted down to the
  // first slot); the next tile's first slot stays
  const uint32_t start = ranges[2 * size_t(t)];
  const uint32_t end = (t + 1 < uint32_t(n_tiles)) ? ranges[2 * size_t(t) + 2] : uint32_t(*n_tot);
  if (lane == 0) ranges[2 * size_t(t) + 1] = end;
  const uint32_t n = end - start;
  if (n > uint32_t(kWaveKeys)) {
    if (lane == 0) *(n > uint32_t(kSmall) ? n_long : n_mid) = 1;
    return;
  }
  if (n == 0) return;
  if (sort_list_words<1>(bucket + start, n, start, t, s_words[threadIdx.x >> 6], nullptr, vals, keys))
    return;
  uint64_t k[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t i = 8u * lane + r;
    k[r] = (i < n) ? bucket[start + i] : ~uint64_t(0);
  }
  wave_sort(k, n <= 8u ? 8u : pow2_ceil(n));
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t i = 8u * lane + r;
    if (i < n) {
      vals[start + i] = uint32_t(k[r]);
      if (keys) keys[start + i] = (uint64_t(t) << 32) | (k[r] >> 32);
    }
  }
}

// Lists of kWaveKeys+1 .. kSmall keys: 256-thread blocks striding over the
// tiles, 8 words per lane in registers, LDS only for the
// strides that cross waves (1M Gaussians, 200x133, tile 8: 12 us, 29 as 64-bit keys in
// registers, 46 in LDS; 36 thousand such lists of 16 views of 4M: 320 against 971).
// Up to 2048 blocks: at 400x266 (1700 tiles)
// every tile then has its own block (binning 161 -> 153 us against 1024 blocks).
constexpr int kMidThreads = 256;
constexpr int kMidBlocks = 2048;

__global__ __launch_bounds__(kMidThreads) void k_tile_sort_mid(
    int n_tiles, const int64_t* __restrict__ n_eff, const int64_t* __restrict__ n_mid,
    uint64_t* __restrict__ bucket, uint32_t* __restrict__ vals,
    uint64_t* __restrict__ keys, const uint32_t* __restrict__ ranges) {
  __shared__ __align__(16) uint64_t s[kSmall];
  __shared__ uint64_t s_edge[2 * kMidThreads / 64];
  if (*n_eff == 0 || *n_mid == 0) return;
  for (uint32_t t = blockIdx.x; t < uint32_t(n_tiles); t += gridDim.x) {
    const uint32_t start = ranges[2 * size_t(t)];
    const uint32_t n = ranges[2 * size_t(t) + 1] - start;
    if (n <= uint32_t(kWaveKeys) || n > uint32_t(kSmall)) continue;  // block-uniform
    if (!sort_list_words<kMidThreads / 64>(bucket + start, n, start, t,
                                           reinterpret_cast<uint32_t*>(s), s_edge, vals, keys))
      sort_list_regs<kMidThreads / 64>(bucket, start, n, t, s, vals, keys);
  }
}

// Longer lists: 1024-thread blocks, each striding over the tiles (a block
// needs much of a CU's LDS, so one block per tile would serialise on empty
// tiles), with LDS chunks of kChunk keys.  A list of at most kChunk keys is
// sorted as words (30 us at 1M Gaussians, 200x133, tile 8; 46 as 64-bit keys in LDS).
// A longer one is sorted in place in the bucket: each chunk as words,
// then for every further merge size the strides >= kChunk run on
// global memory and the shorter ones per chunk in LDS (16 views of mixed sizes, 102
// lists of up to 11 thousand keys: 280 us, 242 with only the shorter lists as words, 154
// with the chunks too, 127 with the tiles looked up together).  (All waves of a block
// share one CU, whose L1 keeps the block's global writes coherent across the
// barriers.)  The 64 KB chunk lets two blocks share a CU, so 512 blocks take
// all of a low-resolution view's long lists at once; with 16384-key chunks one
// block held a CU, and the 425 lists of 1M Gaussians at 200x133 (tile 8) took
// two rounds of 256 blocks (sorts 96 -> 80 us, the same keys).
constexpr int kChunk = 8192;
constexpr int kBigThreads = 1024;
constexpr int kBigBlocks = 512;

__device__ inline void sort_long(uint64_t* s, uint64_t* edge, uint64_t* a, uint32_t n) {
  const uint32_t len = pow2_ceil(n);
  auto load = [&](uint32_t c0, uint32_t m) {
    for (uint32_t i = threadIdx.x; i < m; i += kBigThreads) s[i] = a[c0 + i];
    __syncthreads();
  };
  auto store = [&](uint32_t c0, uint32_t m) {
    for (uint32_t i = threadIdx.x; i < m; i += kBigThreads) a[c0 + i] = s[i];
    __syncthreads();
  };
  // every chunk sorted on its own (chunks are aligned blocks of the network)
  for (uint32_t c0 = 0; c0 < n; c0 += kChunk) {
    const uint32_t m = (n - c0 < uint32_t(kChunk)) ? n - c0 : uint32_t(kChunk);
    if (sort_list_words<kBigThreads / 64, true>(a + c0, m, 0u, 0u, reinterpret_cast<uint32_t*>(s),
                                                edge, nullptr, nullptr))
      continue;
    load(c0, m);
    lds_sort<kBigThreads>(s, m, kChunk);
    store(c0, m);
  }
  for (uint32_t h = kChunk; h < len; h <<= 1) {
    net_step<kBigThreads>(a, n, len / 2, h, true);
    for (uint32_t d = h >> 1; d >= uint32_t(kChunk); d >>= 1)
      net_step<kBigThreads>(a, n, len / 2, d, false);
    for (uint32_t c0 = 0; c0 < n; c0 += kChunk) {
      const uint32_t m = (n - c0 < uint32_t(kChunk)) ? n - c0 : uint32_t(kChunk);
      load(c0, m);
      for (uint32_t d = kChunk / 2; d > 0; d >>= 1)
        net_step<kBigThreads>(s, m, kChunk / 2, d, false);
      store(c0, m);
    }
  }
}

// Calls f(tile, first slot, length) for the block's tiles (blockIdx.x, + gridDim.x, ..)
// whose list has more than `lo` keys, and sets the ranges of its empty tiles to [0, 0):
// the thread that looks a tile up is the only one of the launch that touches an empty
// tile's range, so no other reads it half written.  THREADS tiles are looked up at a time: one
// after the other, each a round trip to memory, cost 512 blocks on 81600 tiles 100 us.
// Every thread of the block calls it, and f with block-uniform arguments.
template <int THREADS, class F>
__device__ inline void for_each_list(int n_tiles, uint32_t* ranges, uint32_t lo, F&& f) {
  __shared__ uint32_t s_t[THREADS];
  __shared__ int s_n;
  for (int64_t base = blockIdx.x; base < n_tiles; base += int64_t(gridDim.x) * THREADS) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const int64_t mine = base + int64_t(threadIdx.x) * gridDim.x;
    if (mine < n_tiles) {
      const uint32_t n = ranges[2 * mine + 1] - ranges[2 * mine];
      if (n == 0u) ranges[2 * mine] = ranges[2 * mine + 1] = 0u;
      else if (n > lo) s_t[atomicAdd(&s_n, 1)] = uint32_t(mine);
    }
    __syncthreads();
    const int count = s_n;
    for (int i = 0; i < count; ++i) {
      const uint32_t t = s_t[i], start = ranges[2 * size_t(t)];
      f(t, start, ranges[2 * size_t(t) + 1] - start);
      __syncthreads();  // f's LDS is reused by the next list
    }
  }
}

__global__ __launch_bounds__(kBigThreads) void k_tile_sort_big(
    int n_tiles, const int64_t* __restrict__ n_eff, const int64_t* __restrict__ n_long,
    uint64_t* __restrict__ bucket,
    uint32_t* __restrict__ vals, uint64_t* __restrict__ keys,
    uint32_t* __restrict__ ranges) {
  __shared__ __align__(16) uint64_t s[kChunk];
  __shared__ uint64_t s_edge[2 * kBigThreads / 64];
  if (*n_eff == 0) return;  // every range is [0, 0) already
  // empty tiles read [0, 0): the wave tier leaves them at [p, p) because a
  // tile's end is its neighbour's start, which must stay until every wave has
  // read it.  Without long lists they are set here, in whole cache lines; else
  // by the lookup below, which deals the tiles to the blocks in another order.
  if (*n_long == 0) {
    for (uint32_t t = blockIdx.x * kBigThreads + threadIdx.x; t < uint32_t(n_tiles);
         t += gridDim.x * kBigThreads)
      if (ranges[2 * size_t(t)] == ranges[2 * size_t(t) + 1])
        ranges[2 * size_t(t)] = ranges[2 * size_t(t) + 1] = 0u;
    return;
  }
  for_each_list<kBigThreads>(
      n_tiles, ranges, kSmall, [&](uint32_t t, uint32_t start, uint32_t n) {
        if (n > uint32_t(kChunk)) {
          sort_long(s, s_edge, bucket + start, n);
          write_sorted<kBigThreads>(bucket + start, n, start, t, vals, keys);
        } else if (!sort_list_words<kBigThreads / 64>(bucket + start, n, start, t,
                                                      reinterpret_cast<uint32_t*>(s), s_edge, vals,
                                                      keys)) {
          for (uint32_t i = threadIdx.x; i < n; i += kBigThreads) s[i] = bucket[start + i];
          __syncthreads();
          lds_sort<kBigThreads>(s, n, pow2_ceil(n));
          write_sorted<kBigThreads>(s, n, start, t, vals, keys);
        }
      });
}

// ---- small launches in one kernel: few Gaussians and few tiles, where seven launches of
// a few blocks each are mostly launches.  Block t < n_tiles goes over all items: those
// whose box holds its tile make its list, in LDS, and what every box has of the tiles
// before it gives the list's first slot, without asking another block.  One more block
// writes the items' pair offsets and the totals.
// Against the general passes: 4096 Gaussians, 48 tiles: 11 us against 33; 8192 and 192:
// 16 against 39; 1024 and 2048: 26 against 94.  A block's loop is items / 1024 steps
// and 512 blocks run at a time, so the gain ends with tiles times items: 8192 and 1024
// 35 against 54, 8 views of 2048 and 384 tiles 25 against 29; there is the line.  The
// items of a view are bounded by the keys that fit the LDS.
constexpr int kDirectThreads = 1024;
constexpr int kDirectKeys = kChunk;          // items of a view
constexpr int64_t kDirectItems = 16384;      // items of the launch
constexpr int64_t kDirectWork = 1 << 23;     // tiles x items

// the sum of x over the block; s_w holds 16 words, every thread calls it
__device__ inline uint32_t block_sum1024(uint32_t x, uint32_t* s_w) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x += uint32_t(__shfl_xor(int(x), d, 64));
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = x;
  __syncthreads();
  uint32_t all = 0;
#pragma unroll
  for (int w = 0; w < kDirectThreads / 64; ++w) all += s_w[w];
  __syncthreads();
  return all;
}

__global__ __launch_bounds__(kDirectThreads) void k_bin_direct(
    Items S, int n_views, int n_tiles, int64_t cap, uint64_t* __restrict__ bucket,
    uint32_t* __restrict__ vals, uint64_t* __restrict__ keys, uint32_t* __restrict__ ranges,
    int64_t* __restrict__ proj_total, int64_t* __restrict__ n_pairs_user) {
  __shared__ __align__(16) uint64_t s[kDirectKeys];
  __shared__ uint64_t s_edge[2 * kDirectThreads / 64];
  __shared__ uint32_t s_w[kDirectThreads / 64];
  __shared__ uint32_t s_n;
  const int tid = threadIdx.x, lane = tid & 63, m = n_views * S.n;
  auto tt_of = [&](int v, int g) {
    return reinterpret_cast<const uint32_t*>(S.proj + size_t(v) * S.stride + S.tt_off)[g];
  };
  if (int(blockIdx.x) == n_tiles) {  // the items' pair offsets
    uint32_t carry = 0;
    for (int base = 0; base < m; base += kDirectThreads) {
      const int i = base + tid, v = i / S.n, g = i - v * S.n;
      const uint32_t tt = i < m ? tt_of(v, g) : 0u;
      const uint32_t inc = wave_incl_scan(tt);
      if (lane == 63) s_w[tid >> 6] = inc;
      __syncthreads();
      uint32_t before = carry;
#pragma unroll
      for (int w = 0; w < kDirectThreads / 64; ++w) {
        const uint32_t x = s_w[w];
        before += w < (tid >> 6) ? x : 0u;
        carry += x;
      }
      if (i < m)
        reinterpret_cast<uint32_t*>(S.goff_proj + size_t(v) * S.stride + S.goff_off)[g] =
            before + inc - tt;
      __syncthreads();  // s_w is rewritten by the next step
    }
    if (tid == 0) {
      *proj_total = int64_t(carry);
      *n_pairs_user = int64_t(carry);
    }
    return;
  }
  const uint32_t t = blockIdx.x;
  int v = 0;
  for (int k = 1; k < n_views; ++k) v = S.TI.tile_base[k] <= int(t) ? k : v;
  const int lt = int(t) - S.TI.tile_base[v];
  const int ty = lt / S.TI.gw[v], tx = lt - ty * S.TI.gw[v];
  if (tid == 0) s_n = 0u;
  __syncthreads();
  uint32_t all = 0, before = 0;
  for (int base = 0; base < m; base += kDirectThreads) {
    const int i = base + tid, u = i / S.n, g = i - u * S.n;
    const uint32_t tt = i < m ? tt_of(u, g) : 0u;
    all += tt;
    if (u < v) before += tt;
    if (tt > 0u && u == v) {
      const float4 r2 =
          reinterpret_cast<const float4*>(S.proj + size_t(v) * S.stride)[3 * size_t(g) + 2];
      const uint32_t lo = __float_as_uint(r2.z), hi = __float_as_uint(r2.w);
      const int x0 = box_x(lo) >> S.tile_log2, y0 = box_y(lo) >> S.tile_log2;
      const int x1 = box_x(hi) >> S.tile_log2, y1 = box_y(hi) >> S.tile_log2;
      // the box's tiles before (tx, ty): its rows above, and of this row those to the left
      const int w = x1 - x0 + 1;
      before += uint32_t(w * max(min(y1 + 1, ty) - y0, 0));
      if (ty >= y0 && ty <= y1) {
        before += uint32_t(min(max(tx - x0, 0), w));
        if (tx >= x0 && tx <= x1)
          s[atomicAdd(&s_n, 1u)] = (uint64_t(__float_as_uint(r2.y)) << 32) | uint32_t(g);
      }
    }
  }
  all = block_sum1024(all, s_w);
  before = block_sum1024(before, s_w);  // (its barriers: the list is whole)
  const uint32_t n = s_n;
  const bool fits = int64_t(all) <= cap;  // block-uniform, and the same in every block
  if (tid == 0) {
    ranges[2 * size_t(t)] = fits && n ? before : 0u;
    ranges[2 * size_t(t) + 1] = fits && n ? before + n : 0u;
  }
  if (!fits || n == 0u) return;
  if (n <= uint32_t(kWaveKeys)) {
    if (tid >= 64) return;  // no block barrier below
    if (sort_list_words<1>(s, n, before, t, reinterpret_cast<uint32_t*>(s + kWaveKeys), nullptr,
                           vals, keys))
      return;
    uint64_t k[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) k[r] = 8u * lane + r < n ? s[8 * lane + r] : ~uint64_t(0);
    wave_sort(k, n <= 8u ? 8u : pow2_ceil(n));
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t i = 8u * lane + r;
      if (i < n) {
        vals[before + i] = uint32_t(k[r]);
        if (keys) keys[before + i] = (uint64_t(t) << 32) | (k[r] >> 32);
      }
    }
    return;
  }
  for (uint32_t i = tid; i < n; i += kDirectThreads) bucket[before + i] = s[i];
  __syncthreads();
  if (!sort_list_words<kDirectThreads / 64>(bucket + before, n, before, t,
                                            reinterpret_cast<uint32_t*>(s), s_edge, vals, keys)) {
    for (uint32_t i = tid; i < n; i += kDirectThreads) s[i] = bucket[before + i];
    __syncthreads();
    lds_sort<kDirectThreads>(s, n, pow2_ceil(n));
    write_sorted<kDirectThreads>(s, n, before, t, vals, keys);
  }
}

struct WsLayout {
  size_t cnt, copies, bucket, rank, bpos, total;
  WsLayout(int64_t n_views, int64_t n, int64_t cap) {
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t r = o; o += align256(bytes); return r; };
    cnt = take(8 * 4);
    copies = take(4 * size_t(kXcds) * kAggBins);
    bucket = take(8 * size_t(cap));
    rank = take(4 * size_t(cap));
    // per expansion block: at most one more a view than the items fill, whatever the views,
    // so that a workspace for as many items of fewer views holds too
    bpos = take(4 * (size_t((n_views * n + kXT - 1) / kXT) + GS_MAX_VIEWS));
    total = o;
  }
};

// ---- the no-allocation form (gs_bin_sort_noalloc): the workspace of a call
// of at most GS_BIN_SORT_NOALLOC_MAX_PAIRS pairs of capacity lives in this
// file-scope device array, one copy per GPU.  Host code never passes the
// array's name to a kernel (on the host it only names the symbol): the
// device address comes from hipGetSymbolAddress, once per device.
constexpr size_t align256c(size_t x) { return (x + 255) & ~size_t(255); }
constexpr size_t kNoAllocBytes =
    256 + align256c(4 * size_t(kXcds) * kAggBins) + align256c(8 * size_t(GS_BIN_SORT_NOALLOC_MAX_PAIRS)) +
    align256c(4 * size_t(GS_BIN_SORT_NOALLOC_MAX_PAIRS)) +
    align256c(4 * (size_t(GS_BIN_SORT_NOALLOC_MAX_ITEMS + kXT - 1) / kXT + GS_MAX_VIEWS + 1));
static __device__ __align__(256) char scratch[kNoAllocBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

// The current device's copy of `scratch`, looked up on the first call on that
// device (with it current) and kept until the process ends.
hipError_t scratch_address(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_dev[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return hipSuccess;
}

}  // namespace

size_t bin_sort_ws_bytes(int n_views, int n, int64_t cap) {
  return WsLayout(n_views, n, cap).total;
}

hipError_t launch_bin_sort_noalloc(const Views& V, int n, char* proj, int64_t cap,
                                   uint64_t* keys, uint32_t* vals, uint32_t* ranges,
                                   int64_t* n_pairs_dev, hipStream_t st) {
  const int64_t m = int64_t(V.n_views) * n;
  if (cap < 0 || cap > GS_BIN_SORT_NOALLOC_MAX_PAIRS || m > GS_BIN_SORT_NOALLOC_MAX_ITEMS ||
      WsLayout(V.n_views, n, cap).total > kNoAllocBytes)
    return hipErrorInvalidValue;  // the caller rejects this first
  void* ws = nullptr;
  const hipError_t e = scratch_address(&ws);
  if (e != hipSuccess) return e;
  // every call writes each scratch byte it reads before reading it (the counts
  // in the tile scan, the block offsets in the reduce pass, the ranks in the
  // count pass, the bucket slots [0, pairs) in the bucket pass), so nothing is
  // cleared
  return launch_bin_sort(V, n, proj, cap, ws, keys, vals, ranges, n_pairs_dev, st);
}

hipError_t launch_bin_sort(const Views& V, int n, char* proj, int64_t cap, void* ws_,
                           uint64_t* keys, uint32_t* vals, uint32_t* ranges,
                           int64_t* n_pairs_dev, hipStream_t st) {
  const WsLayout W(V.n_views, n, cap);
  char* ws = static_cast<char*>(ws_);
  int64_t* counts = reinterpret_cast<int64_t*>(ws + W.cnt);
  int64_t* n_tot = counts + 0;
  int64_t* n_eff = counts + 1;
  int64_t* n_long = counts + 2;
  int64_t* n_mid = counts + 3;
  uint64_t* bucket = reinterpret_cast<uint64_t*>(ws + W.bucket);
  uint32_t* rank = reinterpret_cast<uint32_t*>(ws + W.rank);
  uint32_t* bpos = reinterpret_cast<uint32_t*>(ws + W.bpos);
  uint32_t* copies_ws = reinterpret_cast<uint32_t*>(ws + W.copies);
  const ProjLayout L(n);
  Items S{};
  int min_view_tiles = 1 << 30;
  for (int v = 0; v < V.n_views; ++v) {
    S.TI.tile_base[v] = V.v[v].tile_base;
    S.TI.tile_end[v] = V.v[v].tile_base + V.v[v].gw * V.v[v].gh;
    S.TI.gw[v] = V.v[v].gw;
    min_view_tiles = std::min(min_view_tiles, V.v[v].gw * V.v[v].gh);
  }
  S.proj = proj;
  S.stride = L.stride;
  S.tt_off = L.tt;
  S.goff_proj = proj;  // the count pass records the items' pair offsets
  S.goff_off = L.goff;
  S.n = n;
  S.tile_log2 = V.tile == 8 ? 3 : V.tile == 16 ? 4 : 5;
  const int T = V.total_tiles;
  const int64_t nr = 2 * int64_t(T);
  // LDS aggregation pays where views have few tiles; blocks then take more
  // items (fewer global atomics), as long as the grid still fills the chip:
  // a small scene keeps one round per block
  const bool any_agg = min_view_tiles <= kAggBins;
  S.rounds = 1;
  const int64_t m = int64_t(V.n_views) * n;
  int64_t* proj_total = proj ? reinterpret_cast<int64_t*>(proj + L.total) : nullptr;
  if (n > 0 && n <= kDirectKeys && m <= kDirectItems && m * T <= kDirectWork) {
    GS_LAUNCH("k_bin_direct", k_bin_direct, dim3(unsigned(T) + 1u), dim3(kDirectThreads), 0, st, S,
              V.n_views, T, cap, bucket, vals, keys, ranges, proj_total, n_pairs_dev);
    return hipGetLastError();
  }
  if (any_agg) {
    const int64_t want = (m + int64_t(kXT) * kAggBlocks - 1) / (int64_t(kXT) * kAggBlocks);
    S.rounds = int(std::min<int64_t>(std::max<int64_t>(want, 1), kAggRounds));
  }
  S.bpv = int((int64_t(n) + int64_t(kXT) * S.rounds - 1) / (int64_t(kXT) * S.rounds));
  for (int v = 0; v < V.n_views; ++v) S.order[v] = v;
  std::stable_sort(S.order, S.order + V.n_views, [&](int a, int b) {
    return V.v[a].gw * V.v[a].gh > V.v[b].gw * V.v[b].gh;
  });
  const size_t agg_lds = sizeof(uint32_t) * kAggBins;
  const unsigned xb = unsigned(S.bpv) * unsigned(V.n_views);

  // launches of at most kAggBins tiles spread the LDS-counting blocks'
  // reservation atomics over kXcds counter copies
  uint32_t* copies = (T <= kAggBins) ? copies_ws : nullptr;
  const int64_t nc = copies ? int64_t(kXcds) * kAggBins : 0;
  // every block's first index-order position: ranked pairs store
  // their ranks there, and every item's pair offset (recorded in proj for
  // the backward) follows from them
  GS_LAUNCH("k_tile_reduce", k_tile_reduce, dim3(xb > 0 ? xb : 1u), dim3(kXT), 0, st, S, bpos,
            ranges, nr, copies, nc);
  const bool scanned = xb > kSpineBlocks;
  if (scanned)
    GS_LAUNCH("k_tile_spine", k_tile_spine, dim3(1), dim3(kSpineThreads), 0, st, bpos, int(xb));
  if (xb > 0)
    GS_LAUNCH("k_tile_count", (S.rounds == 1 ? k_tile_count<1> : k_tile_count<kAggRounds>), dim3(xb),
              dim3(kXT), agg_lds, st, S, bpos, scanned, cap, ranges, rank,
              copies);
  GS_LAUNCH("k_tile_scan", (T <= 2 * kTS ? k_tile_scan<2> : k_tile_scan<4>), dim3(1), dim3(kTS), 0,
            st, ranges, copies, T, proj_total, cap, n_tot, n_eff, n_long, n_mid, n_pairs_dev);
  Items Sb = S;
  Sb.goff_proj = nullptr;
  if (xb > 0)
    GS_LAUNCH("k_bucket", (S.rounds == 1 ? k_bucket<1> : k_bucket<kAggRounds>), dim3(xb), dim3(kXT),
              agg_lds, st, Sb, n_eff, bpos, scanned, rank, ranges, copies,
              bucket);
  GS_LAUNCH("k_tile_sort_wave", k_tile_sort_wave, dim3(unsigned((T + 3) / 4)), dim3(256), 0, st,
            T, n_tot, n_eff, n_mid, n_long, bucket, vals, keys, ranges);
  GS_LAUNCH("k_tile_sort_mid", k_tile_sort_mid, dim3(unsigned(T < kMidBlocks ? T : kMidBlocks)),
            dim3(kMidThreads), 0, st, T, n_eff, n_mid, bucket, vals, keys, ranges);
  GS_LAUNCH("k_tile_sort_big", k_tile_sort_big, dim3(unsigned(T < kBigBlocks ? T : kBigBlocks)),
            dim3(kBigThreads), 0, st, T, n_eff, n_long, bucket, vals, keys, ranges);
  return hipGetLastError();
}

}  // namespace gsk

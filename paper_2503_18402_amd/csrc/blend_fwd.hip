// Forward blend (Eq. 1): one workgroup per tile walks the tile's depth-sorted
// list front to back.  Batches of Gaussian records are staged in LDS by the
// whole workgroup; each 64-lane wave owns an 8x8 (or 16x16) square of the
// tile and walks the entries whose footprint box touches its square, from a
// ballot, on the scalar unit.  (The backward runs one wave per tile instead;
// both share the float32 evaluation of alpha, so their decisions agree.)  A
// pixel stops at the first Gaussian that would take its transmittance below
// 1e-4; a wave leaves the list when all its pixels have stopped, the workgroup
// when all waves have.
//
// k_blend_fwd is bound by instruction issue: about 20 vector instructions per
// (entry, pixel) whose box is touched, of which a third of the entries reach no
// pixel of the square, and an entry's record has to arrive from LDS first.  So
// the colour's part runs under the mask of the pixels reached and is branched
// over when there is none; a stopped pixel is a raised threshold, not a test; the
// record is one 48-byte piece, read at one address while the one before is
// blended; and the walk itself takes few scalar instructions, which bound the kernel
// as much as the vector ones did.  1M Gaussians at 1600x1064, 16-pixel tiles: 246 us
// with every lane selecting its updates and records read as used, 186 with the mask, 180
// with the record read ahead, 160 with 9 scalar instructions an entry for 13 (16 views
// of mixed sizes 1455, 1103 with the record read ahead, 940; tiles of 8 435, 379; of 32
// 467, 240).
#include <type_traits>

#include "blend_common.hpp"

namespace gsk {
namespace {

// The L1 gradient of one pixel's three channels (elements e, e + plane,
// e + 2 plane), from the values just stored in the image; returns sum |d|.
__device__ __forceinline__ float l1_pixel(const L1Fuse& l1, int64_t e, int64_t plane, float c0,
                                          float c1, float c2) {
  const float* tgt = l1.index ? l1.target + int64_t(*l1.index) * l1.stride : l1.target;
  const float d0 = c0 - tgt[e], d1 = c1 - tgt[e + plane], d2 = c2 - tgt[e + 2 * plane];
  l1.dL[e] = l1_sign(d0, l1.scale);
  l1.dL[e + plane] = l1_sign(d1, l1.scale);
  l1.dL[e + 2 * plane] = l1_sign(d2, l1.scale);
  return (fabsf(d0) + fabsf(d1)) + fabsf(d2);
}

// scale * (the workgroup's sum of x) added to the loss with one atomic; every
// thread of the NW-wave workgroup calls it
template <int NW>
__device__ __forceinline__ void l1_block_add(const L1Fuse& l1, float x) {
  __shared__ float s_part[NW];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += s_part[w];
    atomicAdd(l1.loss, l1.scale * t);
  }
}

// A staged list entry: the record in the tile's frame.
struct FwdRec {
  float4 r0;         // mx, my, A, B
  float4 r1;         // C, log2 opacity, r, g
  float b;
  uint32_t pos;      // list position, from 1
  uint32_t mask;     // bit w: the box touches wave w's square; kNotPlain
  uint32_t pad;      // 48 bytes: 16-byte aligned float4s (64: bank conflicts, 164 us)
};

constexpr uint32_t kNotPlain = 1u << 31;
struct FwdEnt {  // the part of it that a pixel needs, in registers
  float4 r0, r1;
  float b;
  uint32_t pos;
};

// One pixel's front-to-back state.  thr is the exponent a splat has to reach:
// log2(1/255), or +inf once the pixel has stopped (or lies outside the view),
// so that stopping costs the evaluation no test of its own.
struct FwdPix {
  float T, C0, C1, C2, thr;
  uint32_t last;
};

// Blends an entry into a pixel, under the mask of the pixels reached.  PLAIN:
// the entry is a plain_record.  STOP: the pixel stops at kTMin (else T is a product).
template <bool PLAIN, bool STOP>
__device__ __forceinline__ void fwd_blend(FwdPix& P, const FwdEnt& e, float px, float py) {
  const Exponent x = exponent_at(e.r0, e.r1.x, e.r1.y, px, py);
  if (__builtin_expect(falls_off<PLAIN>(x) & reaches(x, P.thr), 1)) {
    const float raw = __builtin_amdgcn_exp2f(x.q);
    const float a = alpha_of<PLAIN>(raw);
    const float aT = a * P.T;
    // T (1 - alpha), reusing the weight's product where the pixel may stop
    const float Tn = STOP ? P.T - aT : P.T * (1.0f - a);
    const bool stop = STOP && Tn < kTMin;  // stops without blending the entry
    const float w = stop ? 0.0f : aT;
    P.C0 = fmaf(w, e.r1.z, P.C0);
    P.C1 = fmaf(w, e.r1.w, P.C1);
    P.C2 = fmaf(w, e.b, P.C2);
    P.T = stop ? P.T : Tn;
    P.last = stop ? P.last : e.pos;
    P.thr = stop ? INFINITY : P.thr;
  }
}

// Walks the entries of `todo` among the 64 at rec, on the scalar unit: the next
// entry's record is read while the current one is blended (past the last one, the
// record before the 64 is read and not used).  The scalar instructions are as many as
// the vector ones leave time for, so there are few: the lowest bit is found and
// cleared, and its record's place added to a base that the lanes hold.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <class Blend>
__device__ __forceinline__ void fwd_walk(const FwdRec* rec, uint64_t todo, Blend&& blend) {
  typedef __attribute__((address_space(3))) const char lds_char;
  uint32_t base = uint32_t(reinterpret_cast<uintptr_t>((lds_char*)rec));
  asm("" : "+v"(base));
  auto fetch = [&](FwdEnt& e) {
    int k;  // -1 when none is left
    asm("s_ff1_i32_b64 %0, %1" : "=s"(k) : "s"(todo));
    asm("s_bitset0_b64 %0, %1" : "+s"(todo) : "s"(k));
    lds_char* r = (lds_char*)(uintptr_t)(base + uint32_t(k * int(sizeof(FwdRec))));
    const f32x4 r0 = *(__attribute__((address_space(3))) const f32x4*)r;
    const f32x4 r1 = *(__attribute__((address_space(3))) const f32x4*)(r + 16);
    const u32x2 r2 = *(__attribute__((address_space(3))) const u32x2*)(r + 32);
    e.r0 = make_float4(r0.x, r0.y, r0.z, r0.w);
    e.r1 = make_float4(r1.x, r1.y, r1.z, r1.w);
    e.b = __uint_as_float(r2.x);
    e.pos = r2.y;
  };
  int left = __builtin_popcountll(todo);
  if (left == 0) return;
  FwdEnt ea, eb;
  fetch(ea);
  while (true) {
    fetch(eb);
    blend(ea);
    if (left == 1) break;
    fetch(ea);
    blend(eb);
    if (left == 2) break;
    left -= 2;
  }
}

template <int TILE, int BATCH>
__global__ __launch_bounds__(WaveShape<TILE>::kThreads) void k_blend_fwd(
    RViews RV, const char* __restrict__ proj, size_t stride, const uint32_t* __restrict__ ranges,
    const uint32_t* __restrict__ vals, float* __restrict__ image, float* __restrict__ final_T,
    uint32_t* __restrict__ last_contrib, float bg0, float bg1, float bg2, L1Fuse l1) {
  using S = WaveShape<TILE>;
  constexpr int NT = S::kThreads, NW = S::kWaves, R = S::kRegion, SUB = S::kSub, P = S::kPix;
  __shared__ FwdRec s_all[1 + BATCH];  // (one to read past a walk's last)
  FwdRec* const s_rec = s_all + 1;

  const int t = xcd_tile(blockIdx.x, RV);
  const int v = view_of_tile(RV, t);
  const int lt = t - RV.tile_base[v];
  const int gw = RV.gw[v], W = RV.W[v], H = RV.H[v];
  const int tx = lt % gw, ty = lt / gw;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wx = (NW == 1) ? 0 : (w & 1), wy = (NW == 1) ? 0 : (w >> 1);
  const int rx0 = tx * TILE + wx * R, ry0 = ty * TILE + wy * R;
  const int lx = lane & 7, ly = lane >> 3;

  // pixel centres in the tile's frame
  const float px0 = float(wx * R + lx) + 0.5f, py0 = float(wy * R + ly) + 0.5f;
  FwdPix X[P];
#pragma unroll
  for (int j = 0; j < SUB; ++j)
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      const bool in = (rx0 + i * 8 + lx < W) & (ry0 + j * 8 + ly < H);
      X[j * SUB + i] = FwdPix{1.0f, 0.0f, 0.0f, 0.0f, in ? kLog2AlphaMin : INFINITY, 0u};
    }
  auto alive = [&]() {
    bool any = false;
#pragma unroll
    for (int p = 0; p < P; ++p) any |= X[p].thr < INFINITY;
    return any;
  };

  const uint32_t start = ranges[2 * t], end = ranges[2 * t + 1];
  const float4* rec = reinterpret_cast<const float4*>(proj + size_t(v) * stride);

  for (uint32_t bstart = start; bstart < end; bstart += BATCH) {
    if (__syncthreads_count(alive()) == 0) break;
    const int nb = int((end - bstart < uint32_t(BATCH)) ? (end - bstart) : uint32_t(BATCH));
    for (int k = tid; k < nb; k += NT) {
      const uint32_t g = vals[bstart + k];
      const float4 r0 = rec[3 * size_t(g)];
      const float4 r1 = rec[3 * size_t(g) + 1];
      const float4 r2 = rec[3 * size_t(g) + 2];
      const uint32_t lo = __float_as_uint(r2.z), hi = __float_as_uint(r2.w);
      uint32_t msk = 0;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) {
        const int x0 = tx * TILE + ((NW == 1) ? 0 : (ww & 1) * R);
        const int y0 = ty * TILE + ((NW == 1) ? 0 : (ww >> 1) * R);
        msk |= box_overlaps(lo, hi, x0, y0, x0 + R - 1, y0 + R - 1) ? (1u << ww) : 0u;
      }
      s_rec[k].r0 = to_tile_frame<TILE>(r0, lo, tx, ty);
      s_rec[k].r1 = r1;
      s_rec[k].b = r2.x;
      s_rec[k].pos = bstart - start + uint32_t(k) + 1u;
      s_rec[k].mask = msk | (plain_record(r0, r1.x, r1.y) ? 0u : kNotPlain);
    }
    __syncthreads();
    for (int c = 0; c < nb; c += 64) {
      if (__ballot(alive()) == 0ull) break;
      // the entries of these 64 whose box touches this wave's square, walked on the scalar unit
      const uint32_t msk = c + lane < nb ? s_rec[(c + lane) % BATCH].mask : 0u;
      uint64_t todo = __ballot((msk >> w) & 1u);
      auto walk = [&](auto is_plain) {
        fwd_walk(s_rec + c, todo, [&](const FwdEnt& e) {
#pragma unroll
          for (int p = 0; p < P; ++p)
            fwd_blend<decltype(is_plain)::value, true>(X[p], e, px0 + float((p % SUB) * 8),
                                                       py0 + float((p / SUB) * 8));
        });
      };
      if ((__ballot((msk & kNotPlain) != 0u) & todo) == 0ull) walk(std::true_type{});
      else walk(std::false_type{});
    }
  }

  const int64_t pb = RV.pix_base[v];
  const int64_t plane = int64_t(W) * H;
  float l1_abs = 0.0f;
#pragma unroll
  for (int j = 0; j < SUB; ++j)
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      const int p = j * SUB + i;
      const int x = rx0 + i * 8 + lx, y = ry0 + j * 8 + ly;
      if (x < W && y < H) {
        const int64_t o = int64_t(y) * W + x;
        const float c0 = fmaf(X[p].T, bg0, X[p].C0), c1 = fmaf(X[p].T, bg1, X[p].C1),
                    c2 = fmaf(X[p].T, bg2, X[p].C2);
        image[3 * pb + o] = c0;
        image[3 * pb + plane + o] = c1;
        image[3 * pb + 2 * plane + o] = c2;
        final_T[pb + o] = X[p].T;
        last_contrib[pb + o] = X[p].last;
        if (l1.target) l1_abs += l1_pixel(l1, 3 * pb + o, plane, c0, c1, c2);
      }
    }
  if (l1.loss) l1_block_add<NW>(l1, l1_abs);
}

// ---- launches with few tiles (low resolutions: up to thousands of entries per
// list): NW waves per 8x8 group of a tile, lane l at pixel
// (l % 8, l / 8).  The list is cut into up to kFMaxChunks chunks and walked in rounds
// of NW, one per wave, until no pixel is left.  Transmittance only decreases along the list, so a pixel
// stops inside a chunk exactly when T entering it times the product of (1 - alpha)
// over its entries falls below 1e-4:
//   A. per chunk, with no stopping: the product, the colour (T = 1 at the
//      chunk's start) and the last entry with alpha >= 1/255;
//   B. in every wave, from all chunks: the chunk where the pixel stops, and T and
//      colour entering it (or, if none, after the round);
//   C. from that chunk on, its wave walks the pixel's list until it stops.
// A list of up to kFWalk entries is only walked (C).
//
// Up to kFFew8 or kFFew16 tiles (of 8 or 16 pixels): a block of kFWaves waves per
// group; the groups of a short list are a wave each of the tile's first block.  More tiles:
// a block of kFMoreWaves waves per tile, at tiles of 16 a wave per group (NW 1, no
// barriers).  There a wave per group or so fills the chip, the waves and LDS of more
// lie idle in short lists, and blocks cost: each adds its loss with one atomic on
// one address, 14 ns apiece whatever else runs.  2000 tiles of 16, lists of 10 / 48 / 100 /
// 300 entries on average: 35 / 40 / 47 / 84 us against 110 / 115 / 117 / 141 with 8 waves per
// group (13 / 21 / 32 / 81 and 37 / 57 / 61 / 130 without the loss; as two launches with
// the short lists in k_blend_fwd, 52 / 96 / 94 / 298).  2000 of 8 without the loss, 10 / 100 /
// 300: 12 / 22 / 48 against 16 / 24 / 53.  The lines: 600 tiles of 16 with 1000 entries take 91
// us with a wave per group and 82 with eight, 770 the same; 770 of 8 56 with four waves
// and 51 with eight, 1000 62 and 66.
//
// Bound by one wave's issue rate and by the rounds, each a gather, a walk and a
// barrier.  A 128x96 view of 48 tiles of 16: 16 us, against 51 with one block per tile
// and a second launch for its short lists; 425 tiles of up to 3152 entries, where no
// pixel needs more than 1205 and half the pixels 530: 56 against 139 with the whole list
// evaluated; 950 tiles of 180: 21 against 38.  (With chunks of up to 48 entries in rounds
// of their own, 4 waves took 18, 76 and 20 us, 8 waves 15, 58 and 22, 16 waves 16, 68
// and 40: but the chunks' bounds decide how T is rounded, an image that differs in its
// last bits flips the sign of an L1 gradient now and then, and with it a Gaussian's
// step, so the chunks stay where they were.)
constexpr int kFWaves = 8;
constexpr int kFMaxChunks = 16;
constexpr uint32_t kFMinChunk = 32;
constexpr uint32_t kFWalk = 48;
constexpr int kFFew8 = 960, kFFew16 = 768;
constexpr int kFMoreWaves = 4;

// NW: waves per group; GPB: groups per block, one or all of the tile's
template <int TILE, int NW, int GPB>
__global__ __launch_bounds__(64 * NW * GPB) void k_blend_fwd_long(
    RViews RV, const char* __restrict__ proj, size_t stride, const uint32_t* __restrict__ ranges,
    const uint32_t* __restrict__ vals, float* __restrict__ image, float* __restrict__ final_T,
    uint32_t* __restrict__ last_contrib, float bg0, float bg1, float bg2, L1Fuse l1) {
  constexpr int GX = TileShape<TILE>::kGroupsX, Q = TileShape<TILE>::kGroups;
  static_assert(GPB == 1 || (GPB == Q && NW == 1), "a group's waves share barriers");
  __shared__ FwdRec s_rec[NW * GPB][1 + 64];  // (one to read past a walk's last)
  __shared__ float4 s_ch[2][NW > 1 ? NW : 1][64];    // A: (product, colour); rounds alternate
  __shared__ uint32_t s_lp[2][NW > 1 ? NW : 1][64];  // A: last entry with alpha >= 1/255
  // the blocks of a tile run on one XCD
  constexpr int kBlocks = Q / GPB;
  const int xcd = blockIdx.x % kXcds, bq = (blockIdx.x / kXcds) % kBlocks;
  const int block = int(blockIdx.x / (kXcds * kBlocks)) * kXcds + xcd;
  if (block >= RV.total_tiles) return;
  const int t = xcd_tile(block, RV);
  const int v = view_of_tile(RV, t);
  const int lt = t - RV.tile_base[v];
  const int gw = RV.gw[v], W = RV.W[v], H = RV.H[v];
  const int tx = lt % gw, ty = lt / gw;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const uint32_t start = ranges[2 * t], len = ranges[2 * t + 1] - start;
  const bool only_walk = len <= kFWalk;
  const bool own_group = GPB > 1 || only_walk;
  if (GPB == 1 && only_walk && bq != 0) return;
  const int q = own_group ? min(wave, Q - 1) : bq;
  const int wv = own_group ? 0 : wave;  // among the group's waves
  const int gx0 = tx * TILE + (q % GX) * 8, gy0 = ty * TILE + (q / GX) * 8;
  const int x = gx0 + (lane & 7), y = gy0 + (lane >> 3);
  // pixel centre in the tile's frame
  const float px = float((q % GX) * 8 + (lane & 7)) + 0.5f;
  const float py = float((q / GX) * 8 + (lane >> 3)) + 0.5f;
  const float4* rec = reinterpret_cast<const float4*>(proj + size_t(v) * stride);
  FwdRec* const my = s_rec[wave] + 1;

  const int64_t pb = RV.pix_base[v];
  const int64_t plane = int64_t(W) * H;
  float l1_abs = 0.0f;
  auto write = [&](float T, float C0, float C1, float C2, uint32_t last) {
    const int64_t o = int64_t(y) * W + x;
    const float c0 = fmaf(T, bg0, C0), c1 = fmaf(T, bg1, C1), c2 = fmaf(T, bg2, C2);
    image[3 * pb + o] = c0;
    image[3 * pb + plane + o] = c1;
    image[3 * pb + 2 * plane + o] = c2;
    final_T[pb + o] = T;
    last_contrib[pb + o] = last;
    if (l1.target) l1_abs += l1_pixel(l1, 3 * pb + o, plane, c0, c1, c2);
  };

  // entries [i0, min(i0 + 64, i1)) into this wave's LDS: those that touch the group
  uint64_t todo = 0ull, general = 0ull;
  auto index = [&](uint32_t i0, uint32_t i1) {
    return i0 + uint32_t(lane) < i1 ? vals[start + i0 + uint32_t(lane)] : 0u;
  };
  auto stage = [&](uint32_t i0, uint32_t i1, uint32_t g) {
    __builtin_amdgcn_wave_barrier();
    const uint32_t i = i0 + uint32_t(lane);
    bool touch = false, plain = true;
    if (i < i1) {
      const float4 r0 = rec[3 * size_t(g)];
      const float4 r1 = rec[3 * size_t(g) + 1];
      const float4 r2 = rec[3 * size_t(g) + 2];
      const uint32_t lo = __float_as_uint(r2.z), hi = __float_as_uint(r2.w);
      touch = box_overlaps(lo, hi, gx0, gy0, gx0 + 7, gy0 + 7);
      plain = plain_record(r0, r1.x, r1.y);
      my[lane].r0 = to_tile_frame<TILE>(r0, lo, tx, ty);
      my[lane].r1 = r1;
      my[lane].b = r2.x;
      my[lane].pos = i + 1u;
    }
    todo = __ballot(touch);
    general = todo & __ballot(!plain);
    __builtin_amdgcn_wave_barrier();
  };
  FwdPix X;
  auto walk = [&](auto stops) {
    if (general == 0ull)
      fwd_walk(my, todo,
               [&](const FwdEnt& e) { fwd_blend<true, decltype(stops)::value>(X, e, px, py); });
    else
      fwd_walk(my, todo,
               [&](const FwdEnt& e) { fwd_blend<false, decltype(stops)::value>(X, e, px, py); });
  };

  const bool in = (x < W) & (y < H);
  bool alive = in & (!own_group | (wave < Q));
  float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
  uint32_t last = 0u;
  const uint32_t chunks = min((len + kFMinChunk - 1u) / kFMinChunk, uint32_t(kFMaxChunks));
  const uint32_t ch = only_walk ? kFWalk : (len + chunks - 1u) / chunks;
  // (the next round's indices are read ahead)
  uint32_t g = index(uint32_t(wv) * ch, min(uint32_t(wv + 1) * ch, len));
  int par = 0;
  for (uint32_t r0 = 0; r0 < len && __ballot(alive) != 0ull; r0 += NW * ch, par ^= 1) {
    const uint32_t c0 = r0 + uint32_t(wv) * ch, c1 = min(c0 + ch, len);
    const int nch = int(min((len - r0 + ch - 1u) / ch, uint32_t(NW)));
    bool mine = false;
    if (wv < nch) stage(c0, c1, g);
    g = index(c0 + NW * ch, min(c0 + (NW + 1u) * ch, len));
    uint32_t at = c0;  // the staged entries
    if (only_walk) {
      mine = alive;
      alive = false;
    } else {
      // A
      if (wv < nch) {
        X = FwdPix{1.0f, 0.0f, 0.0f, 0.0f, alive ? kLog2AlphaMin : INFINITY, 0u};
        walk(std::false_type{});
        while (at + 64u < c1) {
          at += 64u;
          stage(at, c1, index(at, c1));
          walk(std::false_type{});
        }
        if (NW > 1) {
          s_ch[par][wv][lane] = make_float4(X.T, X.C0, X.C1, X.C2);
          s_lp[par][wv][lane] = X.last;
        }
      }
      if (NW > 1) __syncthreads();
      // B
      for (int c = 0; c < nch; ++c) {
        const float4 pc = NW > 1 ? s_ch[par][c][lane] : make_float4(X.T, X.C0, X.C1, X.C2);
        const uint32_t lp = NW > 1 ? s_lp[par][c][lane] : X.last;
        const float Tn = T * pc.x;
        const bool stop = alive & (Tn < kTMin);
        mine |= stop & (c == wv);
        alive &= !stop;
        if (alive) {
          C0 = fmaf(T, pc.y, C0);
          C1 = fmaf(T, pc.z, C1);
          C2 = fmaf(T, pc.w, C2);
          T = Tn;
          last = lp ? lp : last;
        }
      }
    }
    // C
    if (__ballot(mine) != 0ull) {
      X = FwdPix{T, C0, C1, C2, mine ? kLog2AlphaMin : INFINITY, last};
      if (at != c0) stage(c0, c1, index(c0, c1));
      for (uint32_t i = c0, end = c1;;) {
        walk(std::true_type{});
        i = min(i + 64u, end);
        // (a product rounded below kTMin where the walk stays above: on past the chunk)
        if (i >= len || __ballot(X.thr < INFINITY) == 0ull) break;
        if (i >= end) end = len;
        stage(i, end, index(i, end));
      }
      if (mine) write(X.T, X.C0, X.C1, X.C2, X.last);
    }
  }
  if (wv == 0 && alive) write(T, C0, C1, C2, last);  // the pixels that never stopped
  if (l1.loss) l1_block_add<NW * GPB>(l1, l1_abs);
}

template <int TILE>
hipError_t launch_tile(int batch, const RViews& RV, const char* proj, size_t stride,
                       const uint32_t* ranges, const uint32_t* vals, float* image,
                       float* final_T, uint32_t* last_contrib, const float* bg, const L1Fuse& l1,
                       hipStream_t st) {
  if (few_tiles(RV, TILE)) {
    constexpr int T = TILE <= 16 ? TILE : 16;
    constexpr int Q = TileShape<T>::kGroups;
    const bool few = RV.total_tiles <= (T == 8 ? kFFew8 : kFFew16);
    const unsigned nb = unsigned((RV.total_tiles + kXcds - 1) / kXcds * kXcds) * (few ? Q : 1);
    auto* const kern = few ? k_blend_fwd_long<T, kFWaves, 1> : k_blend_fwd_long<T, kFMoreWaves / Q, Q>;
    GS_LAUNCH("k_blend_fwd_long", kern, dim3(nb), dim3(64 * (few ? kFWaves : kFMoreWaves)), 0, st, RV,
              proj, stride, ranges, vals, image, final_T, last_contrib, bg[0], bg[1], bg[2], l1);
    return hipGetLastError();
  }
  const dim3 grid(unsigned(RV.total_tiles)), block(WaveShape<TILE>::kThreads);
  switch (batch) {
    case 128:
      GS_LAUNCH("k_blend_fwd", HIP_KERNEL_NAME(k_blend_fwd<TILE, 128>), grid, block, 0, st, RV, proj,
                         stride, ranges, vals, image, final_T, last_contrib, bg[0], bg[1], bg[2],
                         l1);
      break;
    case 256:
      GS_LAUNCH("k_blend_fwd", HIP_KERNEL_NAME(k_blend_fwd<TILE, 256>), grid, block, 0, st, RV, proj,
                         stride, ranges, vals, image, final_T, last_contrib, bg[0], bg[1], bg[2],
                         l1);
      break;
    default:
      GS_LAUNCH("k_blend_fwd", HIP_KERNEL_NAME(k_blend_fwd<TILE, 512>), grid, block, 0, st, RV, proj,
                         stride, ranges, vals, image, final_T, last_contrib, bg[0], bg[1], bg[2],
                         l1);
      break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_render_fwd(const Views& V, int n, const gs_raster_cfg& cfg, const char* proj,
                             const uint32_t* ranges, const uint32_t* vals, float* image,
                             float* final_T, uint32_t* last_contrib, const L1Fuse& l1,
                             hipStream_t st) {
  if (V.total_tiles == 0) return hipSuccess;
  const RViews RV = make_rviews(V);
  const size_t stride = ProjLayout(n).stride;
  switch (cfg.tile) {
    case 8:
      return launch_tile<8>(cfg.lds_batch, RV, proj, stride, ranges, vals, image, final_T,
                            last_contrib, cfg.bg, l1, st);
    case 16:
      return launch_tile<16>(cfg.lds_batch, RV, proj, stride, ranges, vals, image, final_T,
                             last_contrib, cfg.bg, l1, st);
    default:
      return launch_tile<32>(cfg.lds_batch, RV, proj, stride, ranges, vals, image, final_T,
                             last_contrib, cfg.bg, l1, st);
  }
}

}  // namespace gsk

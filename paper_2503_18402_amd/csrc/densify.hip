// Densification under the primitive schedule (Sec. 4.3; supplementary,
// "Densification of DashGaussian"): prune, then clone or split the candidates
// with the top k densification scores, where k follows Eq. 4 with the budget
// of Eq. 5 (both host arithmetic, in abi.cpp).
//
// Score of a Gaussian: the mean, over the iterations it was seen, of the norm
// of its 2D-mean gradient (accumulated by k_densify_stats).  Candidates:
// unpruned Gaussians whose score reaches the threshold.  The top k are found
// without sorting: a radix select over the score's float bits (positive floats
// order like their bits) in digits of 11, 11 and 10 bits yields the k-th largest
// key and how many of its ties to take; ties go to the lowest indices.
// Such a step is short passes over a few bytes per Gaussian, bound by the number of
// launches.  The first digit is counted while classifying, every later kernel's
// blocks read off the digit that the one before counted, and one pair of passes
// ranks the ties, counts the outputs and names each output row's source: 6 launches
// before the rows are written, 19 with digits of 8 bits, a kernel to pick each and two
// scans (272k Gaussians: 53 us of kernels now, 186 so).
// The output keeps index order: a pruned Gaussian writes nothing, a kept one
// itself, a cloned one itself then its copy, a split one its two children at
// mu + R(q) diag(s) z_j with scales s / 1.6 (z given by the caller).  Moments
// are copied for originals and zero for copies and children.
#include <algorithm>
#include <cmath>

#include "scan.hpp"

namespace gsk {
namespace {

constexpr uint32_t kPrune = 1u, kCand = 2u;
constexpr uint32_t kNoKey = 0xffffffffu;  // not a candidate (above every float's bits)
constexpr int kBins = 2048;               // 11 bits of key
constexpr int kShift1 = 21, kShift2 = 10;

__global__ __launch_bounds__(256) void k_densify_stats(int n, int n_views, const char* __restrict__ proj,
                                                       size_t stride, size_t tt_off,
                                                       const float* __restrict__ mean2d_abs,
                                                       float scale, float* __restrict__ accum,
                                                       float* __restrict__ count) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  int seen = 0;
  for (int v = 0; v < n_views; ++v)
    seen += reinterpret_cast<const uint32_t*>(proj + size_t(v) * stride + tt_off)[g] > 0u ? 1 : 0;
  if (seen) {
    accum[g] += scale * mean2d_abs[g];
    count[g] += float(seen);
  }
}

__global__ __launch_bounds__(256) void k_densify_clear(unsigned long long* __restrict__ counts,
                                                       uint32_t* __restrict__ hist1,
                                                       uint32_t* __restrict__ hist2) {
  if (threadIdx.x < 2) counts[threadIdx.x] = 0ull;
  for (int i = threadIdx.x; i < kBins; i += 256) hist1[i] = hist2[i] = 0u;
}

// the block's bins added to the launch's
__device__ __forceinline__ void add_bins(const uint32_t* s_h, uint32_t* __restrict__ hist) {
  for (int i = threadIdx.x; i < kBins; i += 256)
    if (s_h[i]) atomicAdd(&hist[i], s_h[i]);
}

// At most kClassBlocks blocks: every block adds to the same two counters and to the
// few bins that the scores share (272k Gaussians: 21 us with a block per 256).
constexpr int kClassBlocks = 256;

__global__ __launch_bounds__(256) void k_densify_classify(int n, const float* __restrict__ accum,
                                                          const float* __restrict__ count,
                                                          const float* __restrict__ opacity_logits,
                                                          float thr, float min_opacity,
                                                          uint32_t* __restrict__ keys,
                                                          uint32_t* __restrict__ flags,
                                                          uint32_t* __restrict__ hist1,
                                                          unsigned long long* __restrict__ counts) {
  __shared__ uint32_t s_c[2];
  __shared__ uint32_t s_h[kBins];
  if (threadIdx.x < 2) s_c[threadIdx.x] = 0u;
  for (int i = threadIdx.x; i < kBins; i += 256) s_h[i] = 0u;
  __syncthreads();
  const int64_t step = int64_t(gridDim.x) * 256;
  for (int64_t g = int64_t(blockIdx.x) * 256 + threadIdx.x; g < n; g += step) {
    const float c = count[g];
    const float score = c > 0.0f ? accum[g] / c : 0.0f;
    const float o = 1.0f / (1.0f + expf(-opacity_logits[g]));
    const bool prune = o < min_opacity;
    const bool cand = !prune && c > 0.0f && score >= thr;
    const uint32_t key = cand ? __float_as_uint(score) & 0x7fffffffu : kNoKey;
    keys[g] = key;
    flags[g] = (prune ? kPrune : 0u) | (cand ? kCand : 0u);
    if (prune) atomicAdd(&s_c[0], 1u);
    if (cand) {
      atomicAdd(&s_c[1], 1u);
      atomicAdd(&s_h[key >> kShift1], 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 && s_c[threadIdx.x])
    atomicAdd(&counts[threadIdx.x], (unsigned long long)s_c[threadIdx.x]);
  add_bins(s_h, hist1);
}

// what the select has found: the k-th key's digits so far, and how many of the keys
// with these digits are still to be taken
struct SelState {
  uint32_t prefix, k_rem;
};

// The next digit: the bin of the k_rem-th largest among the keys that hist counts.
// All 256 threads of the block call it.
__device__ inline SelState pick(const SelState s, const uint32_t* __restrict__ hist, int shift) {
  __shared__ uint32_t s_tmp[4];
  __shared__ SelState s_out;
  constexpr int kPer = kBins / 256;
  const int top = kBins - 1 - int(threadIdx.x) * kPer;  // a thread's bins, from the top
  uint32_t h[kPer], sum = 0, all;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    h[i] = hist[top - i];
    sum += h[i];
  }
  uint32_t above = block_excl_scan256(sum, all, s_tmp);
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (above < s.k_rem && s.k_rem <= above + h[i])
      s_out = SelState{s.prefix | (uint32_t(top - i) << shift), s.k_rem - above};
    above += h[i];
  }
  // (fewer keys than the caller said: all of them)
  if (threadIdx.x == 255 && s.k_rem > all)
    s_out = SelState{s.prefix, s.k_rem - (all - h[kPer - 1])};
  __syncthreads();
  return s_out;
}

// Counts the second (LAST false) or third digit of the keys that share the digits
// before.  st[0] is what was found before hist_in; block 0 leaves what hist_in adds to
// it in st[1], and clears the bins that the next kernel counts in.
template <bool LAST>
__global__ __launch_bounds__(256) void k_sel_hist(int n, uint32_t k,
                                                  const uint32_t* __restrict__ keys,
                                                  SelState* __restrict__ st,
                                                  const uint32_t* __restrict__ hist_in,
                                                  uint32_t* __restrict__ hist_out,
                                                  uint32_t* __restrict__ hist_clear) {
  __shared__ uint32_t s_h[kBins];
  for (int i = threadIdx.x; i < kBins; i += 256) s_h[i] = 0u;
  const SelState s = pick(LAST ? st[0] : SelState{0u, k}, hist_in, LAST ? kShift2 : kShift1);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) st[LAST ? 1 : 0] = s;
    if (hist_clear)
      for (int i = threadIdx.x; i < kBins; i += 256) hist_clear[i] = 0u;
  }
  const int64_t step = int64_t(gridDim.x) * 256;
  for (int64_t g = int64_t(blockIdx.x) * 256 + threadIdx.x; g < n; g += step) {
    const uint32_t key = keys[g];
    if (LAST ? (key >> kShift2) == (s.prefix >> kShift2) : (key >> kShift1) == (s.prefix >> kShift1))
      atomicAdd(&s_h[LAST ? key & ((1u << kShift2) - 1u) : (key >> kShift2) & (kBins - 1u)], 1u);
  }
  __syncthreads();
  add_bins(s_h, hist_out);
}

// What a Gaussian contributes to the output rows before the ties are dealt with: 1
// unless pruned, 1 more if selected for a key above the k-th (mode 0), as any
// candidate (mode 1), never (mode 2); and whether it ties with the k-th key.  The rows
// before a Gaussian are then the sum of these plus the first k_rem ties.
struct Out {
  uint32_t rows, tie;
};
__device__ __forceinline__ Out out_of(int mode, uint32_t flag, uint32_t key, const SelState s) {
  const bool cand = flag & kCand;
  const bool sel = cand & (mode == 1 || (mode == 0 && key > s.prefix));
  return Out{((flag & kPrune) ? 0u : 1u) + (sel ? 1u : 0u),
             (cand && mode == 0 && key == s.prefix) ? 1u : 0u};
}

constexpr int kPlanItems = 4;
constexpr int kPlanTile = 256 * kPlanItems;

__global__ __launch_bounds__(256) void k_plan_reduce(int n, int mode,
                                                     const uint32_t* __restrict__ keys,
                                                     const uint32_t* __restrict__ flags,
                                                     SelState* __restrict__ st,
                                                     const uint32_t* __restrict__ hist3,
                                                     uint32_t* __restrict__ hist_clear,
                                                     uint2* __restrict__ sums) {
  __shared__ uint32_t s_tmp[4];
  SelState s{0u, 0u};
  if (mode == 0) {
    s = pick(st[1], hist3, 0);
    if (blockIdx.x == 0) {
      if (threadIdx.x == 0) st[2] = s;
      for (int i = threadIdx.x; i < kBins; i += 256) hist_clear[i] = 0u;
    }
  }
  const int64_t base = int64_t(blockIdx.x) * kPlanTile;
  uint32_t rows = 0, ties = 0, all_rows, all_ties;
#pragma unroll
  for (int i = 0; i < kPlanItems; ++i) {
    const int64_t g = base + i * 256 + threadIdx.x;
    if (g < n) {
      const Out o = out_of(mode, flags[g], keys[g], s);
      rows += o.rows;
      ties += o.tie;
    }
  }
  block_excl_scan256(rows, all_rows, s_tmp);
  block_excl_scan256(ties, all_ties, s_tmp);
  if (threadIdx.x == 0) sums[blockIdx.x] = make_uint2(all_rows, all_ties);
}

// Output row o -> (source Gaussian g, kind), packed as g << 2 | kind:
// kind 0 the Gaussian itself (moments copied), 1 a clone's copy (fresh
// moments), 2 + j split child j (fresh moments).  The last block leaves the row
// count for the apply call and the caller.
__global__ __launch_bounds__(256) void k_plan_rows(int n, int mode,
                                                   const uint32_t* __restrict__ keys,
                                                   const uint32_t* __restrict__ flags,
                                                   const SelState* __restrict__ st,
                                                   const uint2* __restrict__ sums,
                                                   const float* __restrict__ log_scales,
                                                   float max_scale, uint32_t* __restrict__ src,
                                                   uint32_t* __restrict__ total,
                                                   int64_t* __restrict__ n_new) {
  __shared__ uint32_t s_tmp[4];
  const SelState s = mode == 0 ? st[2] : SelState{0u, 0u};
  uint32_t rows = 0, ties = 0, rows0, ties0;
  for (unsigned b = threadIdx.x; b < blockIdx.x; b += 256) {
    const uint2 x = sums[b];
    rows += x.x;
    ties += x.y;
  }
  block_excl_scan256(rows, rows0, s_tmp);
  block_excl_scan256(ties, ties0, s_tmp);
#pragma unroll
  for (int i = 0; i < kPlanItems; ++i) {
    const int64_t g = int64_t(blockIdx.x) * kPlanTile + i * 256 + threadIdx.x;
    const uint32_t f = g < n ? flags[g] : kPrune;
    const uint32_t key = g < n ? keys[g] : kNoKey;
    const Out o = out_of(mode, f, key, s);
    uint32_t all_rows, all_ties;
    const uint32_t r = rows0 + block_excl_scan256(o.rows, all_rows, s_tmp);
    const uint32_t t = ties0 + block_excl_scan256(o.tie, all_ties, s_tmp);
    rows0 += all_rows;
    ties0 += all_ties;
    if (f & kPrune) continue;
    const uint32_t at = r + min(t, s.k_rem), base = uint32_t(g) << 2;
    if (o.rows == 2u || (o.tie && t < s.k_rem)) {  // selected
      const float smax = fmaxf(expf(log_scales[3 * g]),
                               fmaxf(expf(log_scales[3 * g + 1]), expf(log_scales[3 * g + 2])));
      const bool split = smax > max_scale;
      src[at] = base | (split ? 2u : 0u);
      src[at + 1] = base | (split ? 3u : 1u);
    } else {
      src[at] = base;
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    const uint32_t all = rows0 + min(ties0, s.k_rem);
    *total = all;
    *n_new = int64_t(all);
  }
}

struct DensifyIO {
  const float* p[5];
  const float* m[5];
  const float* v[5];
  float* po[5];
  float* mo[5];
  float* vo[5];
};

// One group of the new arrays, one thread per output element (consecutive
// threads write consecutive floats of p, m and v).
template <int G, int W>
__device__ __forceinline__ void apply_group(const DensifyIO& io, const float* __restrict__ z,
                                            const uint32_t* __restrict__ src, uint32_t total) {
  const int64_t E = int64_t(total) * W;
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < E; e += stride) {
    const int64_t o = e / W;
    const int k = int(e - o * W);
    const uint32_t sk = src[o];
    const size_t g = sk >> 2;
    const uint32_t kind = sk & 3u;
    const size_t i = g * W + k;
    float pv;
    if (G == 0 && kind >= 2u) {  // child mean: mu + R(q) diag(s) z_j, row k of R
      const float* q = io.p[2] + 4 * g;
      const float qinv = 1.0f / sqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
      const float qw = q[0] * qinv, qx = q[1] * qinv, qy = q[2] * qinv, qz = q[3] * qinv;
      float r0, r1, r2;
      if (k == 0) {
        r0 = 1.0f - 2.0f * (qy * qy + qz * qz);
        r1 = 2.0f * (qx * qy - qw * qz);
        r2 = 2.0f * (qx * qz + qw * qy);
      } else if (k == 1) {
        r0 = 2.0f * (qx * qy + qw * qz);
        r1 = 1.0f - 2.0f * (qx * qx + qz * qz);
        r2 = 2.0f * (qy * qz - qw * qx);
      } else {
        r0 = 2.0f * (qx * qz - qw * qy);
        r1 = 2.0f * (qy * qz + qw * qx);
        r2 = 1.0f - 2.0f * (qx * qx + qy * qy);
      }
      const float* ls = io.p[1] + 3 * g;
      const float* zz = z + 6 * g + 3 * (kind - 2u);
      const float d0 = expf(ls[0]) * zz[0], d1 = expf(ls[1]) * zz[1], d2 = expf(ls[2]) * zz[2];
      pv = io.p[0][i] + (r0 * d0 + r1 * d1 + r2 * d2);
    } else if (G == 1 && kind >= 2u) {
      pv = io.p[1][i] - logf(1.6f);
    } else {
      pv = io.p[G][i];
    }
    io.po[G][e] = pv;
    io.mo[G][e] = kind == 0u ? io.m[G][i] : 0.0f;
    io.vo[G][e] = kind == 0u ? io.v[G][i] : 0.0f;
  }
}

// The rows of a group that are copied whole as float4s (V of them; the arrays are
// 16-byte aligned): one thread per float4 of p, m and v.
template <int G, int V>
__device__ __forceinline__ void copy_group(const DensifyIO& io, const uint32_t* __restrict__ src,
                                           uint32_t total) {
  const int64_t E = int64_t(total) * V;
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  const float4* p = reinterpret_cast<const float4*>(io.p[G]);
  const float4* m = reinterpret_cast<const float4*>(io.m[G]);
  const float4* v = reinterpret_cast<const float4*>(io.v[G]);
  float4* po = reinterpret_cast<float4*>(io.po[G]);
  float4* mo = reinterpret_cast<float4*>(io.mo[G]);
  float4* vo = reinterpret_cast<float4*>(io.vo[G]);
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < E; e += stride) {
    const int64_t o = e / V;
    const uint32_t sk = src[o];
    const size_t i = size_t(sk >> 2) * V + size_t(e - o * V);
    const bool keep = (sk & 3u) == 0u;
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const float4 a = p[i], b = keep ? m[i] : zero, c = keep ? v[i] : zero;
    po[e] = a;
    mo[e] = b;
    vo[e] = c;
  }
}

// blockIdx.y selects the group, the largest first; the row count is the plan's.
// Bound by its copies: 272k Gaussians 144 us with a float a thread, 92 (4.2 TB/s) with
// float4s where the arrays allow (bit g of vec).
__global__ __launch_bounds__(256) void k_densify_apply(DensifyIO io, const float* __restrict__ z,
                                                       const uint32_t* __restrict__ src,
                                                       const uint32_t* __restrict__ total_dev,
                                                       uint32_t vec) {
  const uint32_t total = *total_dev;
  switch (blockIdx.y) {
    case 0:
      if (vec & 16u) copy_group<4, 12>(io, src, total);
      else apply_group<4, 48>(io, z, src, total);
      break;
    case 1:
      if (vec & 4u) copy_group<2, 1>(io, src, total);
      else apply_group<2, 4>(io, z, src, total);
      break;
    case 2: apply_group<0, 3>(io, z, src, total); break;
    case 3: apply_group<1, 3>(io, z, src, total); break;
    default: apply_group<3, 1>(io, z, src, total); break;
  }
}

struct DWs {
  size_t keys, flags, src, sums, hist, st, total, bytes;
  explicit DWs(int64_t n) {
    size_t o = 0;
    auto take = [&](size_t b) { size_t r = o; o += align256(b); return r; };
    keys = take(4 * size_t(n));
    flags = take(4 * size_t(n));
    src = take(8 * size_t(n));  // up to two output rows per Gaussian
    sums = take(8 * (size_t(n + kPlanTile - 1) / kPlanTile + 1));
    hist = take(3 * 4 * kBins);
    st = take(3 * sizeof(SelState));
    total = take(4);
    bytes = o;
  }
};

}  // namespace

size_t densify_ws_bytes(int n) { return DWs(n).bytes; }

hipError_t launch_densify_stats(int n_views, int n, const char* proj, const float* mean2d_abs,
                                float scale, float* accum, float* count, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const ProjLayout L(n);
  GS_LAUNCH("k_densify_stats", k_densify_stats, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st,
            n, n_views, proj, L.stride, L.tt, mean2d_abs, scale, accum, count);
  return hipGetLastError();
}

hipError_t launch_densify_classify(int n, const float* accum, const float* count,
                                   const float* opacity_logits, float thr, float min_opacity,
                                   void* ws_, int64_t* counts_out, hipStream_t st) {
  const DWs W(n);
  char* ws = static_cast<char*>(ws_);
  unsigned long long* cnt = reinterpret_cast<unsigned long long*>(counts_out);
  uint32_t* hist = reinterpret_cast<uint32_t*>(ws + W.hist);
  GS_LAUNCH("k_densify_clear", k_densify_clear, dim3(1), dim3(256), 0, st, cnt, hist,
            hist + kBins);
  if (n > 0)
    GS_LAUNCH("k_densify_classify", k_densify_classify,
              dim3(unsigned(std::min<int64_t>((int64_t(n) + 255) / 256, kClassBlocks))), dim3(256),
              0, st, n, accum, count, opacity_logits, thr, min_opacity,
              reinterpret_cast<uint32_t*>(ws + W.keys), reinterpret_cast<uint32_t*>(ws + W.flags),
              hist, cnt);
  return hipGetLastError();
}

hipError_t launch_densify_plan(int n, int64_t k, int64_t n_cand, const float* log_scales,
                               float max_scale, void* ws_, int64_t* n_new, hipStream_t st) {
  const DWs W(n);
  char* ws = static_cast<char*>(ws_);
  uint32_t* keys = reinterpret_cast<uint32_t*>(ws + W.keys);
  uint32_t* flags = reinterpret_cast<uint32_t*>(ws + W.flags);
  uint32_t* hist1 = reinterpret_cast<uint32_t*>(ws + W.hist);
  uint32_t *hist2 = hist1 + kBins, *hist3 = hist2 + kBins;
  SelState* sst = reinterpret_cast<SelState*>(ws + W.st);
  uint2* sums = reinterpret_cast<uint2*>(ws + W.sums);
  const uint32_t kk = uint32_t(k > 0 ? (k < n_cand ? k : n_cand) : 0);
  const int mode = kk == 0 ? 2 : (k >= n_cand ? 1 : 0);
  // the bins: classify counted the first digit and cleared hist2; each kernel here
  // clears what the next one, or the next plan, counts in
  if (mode == 0 && n > 0) {
    const unsigned hb = unsigned(std::min<int64_t>((int64_t(n) + 255) / 256, kClassBlocks));
    GS_LAUNCH("k_sel_hist", k_sel_hist<false>, dim3(hb), dim3(256), 0, st, n, kk, keys, sst, hist1,
              hist2, hist3);
    GS_LAUNCH("k_sel_hist", k_sel_hist<true>, dim3(hb), dim3(256), 0, st, n, kk, keys, sst, hist2,
              hist3, static_cast<uint32_t*>(nullptr));
  }
  const unsigned nb = unsigned(std::max<int64_t>((int64_t(n) + kPlanTile - 1) / kPlanTile, 1));
  GS_LAUNCH("k_plan_reduce", k_plan_reduce, dim3(nb), dim3(256), 0, st, n, mode, keys, flags, sst,
            hist3, hist2, sums);
  GS_LAUNCH("k_plan_rows", k_plan_rows, dim3(nb), dim3(256), 0, st, n, mode, keys, flags, sst,
            sums, log_scales, max_scale, reinterpret_cast<uint32_t*>(ws + W.src),
            reinterpret_cast<uint32_t*>(ws + W.total), n_new);
  return hipGetLastError();
}

hipError_t launch_densify_apply(int n, const float* const* p, const float* const* m,
                                const float* const* v, const float* z, const void* ws_,
                                float* const* po, float* const* mo, float* const* vo,
                                hipStream_t st) {
  if (n == 0) return hipSuccess;
  const DWs W(n);
  const char* ws = static_cast<const char*>(ws_);
  DensifyIO io{};
  for (int t = 0; t < 5; ++t) {
    io.p[t] = p[t];
    io.m[t] = m[t];
    io.v[t] = v[t];
    io.po[t] = po[t];
    io.mo[t] = mo[t];
    io.vo[t] = vo[t];
  }
  const uint32_t* src = reinterpret_cast<const uint32_t*>(ws + W.src);
  // groups whose six arrays are 16-byte aligned
  uint32_t vec = 0;
  for (int t = 0; t < 5; ++t) {
    uintptr_t a = 0;
    for (const void* q : {static_cast<const void*>(p[t]), static_cast<const void*>(m[t]),
                          static_cast<const void*>(v[t]), static_cast<const void*>(po[t]),
                          static_cast<const void*>(mo[t]), static_cast<const void*>(vo[t])})
      a |= reinterpret_cast<uintptr_t>(q);
    vec |= (a & 15u) ? 0u : 1u << t;
  }
  // enough blocks for the largest group (48 floats per row, up to 2n rows); the
  // smaller groups' extra blocks find no element and exit
  const unsigned gx = unsigned(std::min<int64_t>((int64_t(n) * 96 + 255) / 256, 8192));
  GS_LAUNCH("k_densify_apply", k_densify_apply, dim3(gx, 5), dim3(256), 0, st, io, z, src,
            reinterpret_cast<const uint32_t*>(ws + W.total), vec);
  return hipGetLastError();
}

}  // namespace gsk

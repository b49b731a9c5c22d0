// The frequency-guided resolution schedule (Sec. 4.2, Eq. 2; supplementary
// Eq. 6-7) and the anti-aliased downsampling of the ground-truth views
// (supplementary, "Ground Truth Downsampling").
//
// Frequency map: M(i,j) = (1/N) sum_n ||F^n(i,j)||_2 with F^n the
// unnormalised 2D DFT of view n and the norm taken over the colour channels.
// It is computed once per scene, in FP64, by fast Fourier transforms in LDS: a
// row pass on the real image (two rows per transform, only the non-negative
// column frequencies: the rest follow by conjugate symmetry) and a column pass
// over the three channels, which takes the norm over channels.  A 1200x800 view
// takes 0.05 ms (16 us rows, 30 us columns: rounds of LDS and L2 latency; the
// 54 MB that it moves would take 10 us), against 1.49 ms for a direct DFT of
// HW(H + W) terms, which is bound by FP64 arithmetic; small views take the direct sums.
// Views are added in order, so the map is deterministic.  H and W are at most
// kDftMax (a line, or its Bluestein padding of at most 8192 values, fits in LDS).
//
// Schedule: from the map, X(F_r) is the sum of M over the centred crop
// |k_y| <= H/(2r), |k_x| <= W/(2r) (the spectrum of the ideal downsample by r),
// scaled by 1/r^2 (Eq. 2 with unnormalised DFTs) or by 1/(H W) (each view's
// DFT normalised by its pixel count); r_m solves X(F_r) = X(F)/a, the knots X_1..X_{m-1} are
// spaced linearly between X(F) and X(F_{r_m}) and solved for r_i by
// bisection, and Eq. 7 places them at s_{r_i} = S ln(X_i/X_m) / ln(X_F/X_m).
// This part is host code over a summed-area table of the map.
//
// Downsampling: separable anti-aliased linear resampling; output sample i is
// centred at input coordinate (i + 0.5) * in/out and weighs the inputs with a
// triangle of half-width max(1, in/out), normalised to sum 1.
#include <algorithm>
#include <cmath>
#include <vector>

#include "gs_internal.hpp"

namespace gsk {
namespace {

// ---- a block-wide FFT in LDS, FP64.  One Stockham stage per factor of the
// length: radices 8, 4, 2, 3, 5, 7 as register butterflies, a prime of 11 to
// kMaxPrime as a direct sum of that many terms; the values of a stage are held
// in registers across the barrier, so one LDS buffer is enough.  A length with
// a larger prime factor p goes through Bluestein's chirp convolution: two
// transforms of a 7-smooth length >= 2n - 1 instead of p terms per value.
constexpr int kMaxStages = 13;   // 2^13 is the longest length
// The largest prime with a stage of its own, one value at a time, p terms each: lines of up
// to kMidLine values are faster through a chirp from 41 on (400x610 = 61 x 10, four views
// 192 and 145 us; 752x1128 = 47 x 16, 24, one 171 and 157; 41: 400x615 157 and 149; 37: 185x259
// 41 and 34, but 592x888 88 and 97), longer ones, whose chirps fill the LDS, are not (848x1272
// = 53 x 16, 24: 211 and 235; 944x944 200 and 197).
constexpr int kMidLine = 800, kMaxPrimeMid = 37, kMaxPrime = 61;

struct FftPlan {
  int n;       // the transform's length
  int len;     // the length run through the stages: n, or Bluestein's m
  int stages;
  int radix[kMaxStages];
  uint32_t magic_ns[kMaxStages];  // x / ns and x / (len / radix) as multiplications
  uint32_t magic_m[kMaxStages];
  uint32_t magic_len;
  // complex tables: len roots of unity; with Bluestein n chirps and the len
  // values of the chirp filter's transform, scaled by 1 / len
  __host__ __device__ bool blue() const { return len != n; }
  __host__ __device__ size_t table() const { return size_t(len) + (blue() ? size_t(n) + len : 0u); }
};

// x / d for x d < 2^32 with magic = ceil(2^32 / d) (0 for d = 1)
__device__ __forceinline__ uint32_t div_magic(uint32_t x, uint32_t magic) {
  return magic ? __umulhi(x, magic) : x;
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) {
  return make_double2(a.x + b.x, a.y + b.y);
}
__device__ __forceinline__ double2 csub(double2 a, double2 b) {
  return make_double2(a.x - b.x, a.y - b.y);
}
__device__ __forceinline__ double2 mul_mi(double2 a) { return make_double2(a.y, -a.x); }  // -i a

template <int R>
struct OddRoots;  // cos and sin of 2 pi k / R, k = 1 .. (R - 1) / 2
template <>
struct OddRoots<3> {
  static constexpr double c[1] = {-0.5}, s[1] = {0.86602540378443864676};
};
template <>
struct OddRoots<5> {
  static constexpr double c[2] = {0.30901699437494742410, -0.80901699437494742410};
  static constexpr double s[2] = {0.95105651629515357212, 0.58778525229247312917};
};
template <>
struct OddRoots<7> {
  static constexpr double c[3] = {0.62348980185873353053, -0.22252093395631440429,
                                  -0.90096886790241912624};
  static constexpr double s[3] = {0.78183148246802980871, 0.97492791218182360702,
                                  0.43388373911755812048};
};

// y_k = sum_q v_q e^{-2 pi i q k / R} in place
template <int R>
__device__ __forceinline__ void dft_small(double2 (&v)[R]) {
  if constexpr (R == 2) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 4) {
    const double2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
    const double2 c = cadd(v[1], v[3]), d = mul_mi(csub(v[1], v[3]));
    v[0] = cadd(a, c);
    v[1] = cadd(b, d);
    v[2] = csub(a, c);
    v[3] = csub(b, d);
  } else if constexpr (R == 8) {
    double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft_small<4>(e);
    dft_small<4>(o);
    constexpr double h = 0.70710678118654752440;
    o[1] = make_double2(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));
    o[2] = mul_mi(o[2]);
    o[3] = make_double2(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = cadd(e[k], o[k]);
      v[k + 4] = csub(e[k], o[k]);
    }
  } else {  // odd prime: pairs q, R - q share their cosine and sine sums
    constexpr int H = (R - 1) / 2;
    double2 p[H], m[H];
    double2 sum = v[0];
#pragma unroll
    for (int q = 1; q <= H; ++q) {
      p[q - 1] = cadd(v[q], v[R - q]);
      m[q - 1] = csub(v[q], v[R - q]);
      sum = cadd(sum, p[q - 1]);
    }
    double2 out[R];
    out[0] = sum;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      double2 re = v[0], im = make_double2(0.0, 0.0);
#pragma unroll
      for (int q = 1; q <= H; ++q) {
        const int r = (q * k) % R, f = r <= H ? r : R - r;
        const double c = OddRoots<R>::c[f - 1], s = r <= H ? OddRoots<R>::s[f - 1]
                                                           : -OddRoots<R>::s[f - 1];
        re = make_double2(fma(c, p[q - 1].x, re.x), fma(c, p[q - 1].y, re.y));
        im = make_double2(fma(s, m[q - 1].x, im.x), fma(s, m[q - 1].y, im.y));
      }
      const double2 t = mul_mi(im);
      out[k] = cadd(re, t);
      out[R - k] = csub(re, t);
    }
#pragma unroll
    for (int k = 0; k < R; ++k) v[k] = out[k];
  }
}

// One Stockham stage of radix R over nseq sequences of P.len values in s
// (sequence after sequence), ns the product of the radices before it.
template <int T, int E, int R>
__device__ __forceinline__ void fft_stage(double2* s, const FftPlan& P, int st, uint32_t ns,
                                          uint32_t nseq, const double2* __restrict__ tw) {
  constexpr int B = (E + R - 1) / R;  // butterflies per thread
  const uint32_t len = uint32_t(P.len), m = len / R, total = m * nseq, tstep = m / ns;
  double2 v[B][R];
  uint32_t to[B];
#pragma unroll
  for (int u = 0; u < B; ++u) {
    const uint32_t b = threadIdx.x + uint32_t(u * T);
    if (b < total) {
      const uint32_t seq = div_magic(b, P.magic_m[st]), j = b - seq * m;
      const uint32_t d = div_magic(j, P.magic_ns[st]), k = j - d * ns;
      const double2* src = s + seq * len + j;
#pragma unroll
      for (int q = 0; q < R; ++q) v[u][q] = src[q * m];
      if (ns > 1u) {
#pragma unroll
        for (int q = 1; q < R; ++q) v[u][q] = cmul(v[u][q], tw[uint32_t(q) * k * tstep]);
      }
      dft_small<R>(v[u]);
      to[u] = seq * len + d * ns * R + k;
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < B; ++u) {
    if (threadIdx.x + uint32_t(u * T) < total) {
#pragma unroll
      for (int q = 0; q < R; ++q) s[to[u] + uint32_t(q) * ns] = v[u][q];
    }
  }
  __syncthreads();
}

// The same for a prime radix p: one output value at a time, p terms each.
template <int T, int E>
__device__ __forceinline__ void fft_stage_prime(double2* s, const FftPlan& P, int st, uint32_t ns,
                                                uint32_t nseq, const double2* __restrict__ tw) {
  const uint32_t len = uint32_t(P.len), p = uint32_t(P.radix[st]), m = len / p,
                 total = len * nseq, tstep = m / ns;
  double2 v[E];
  uint32_t to[E];
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const uint32_t o = threadIdx.x + uint32_t(u * T);
    if (o < total) {
      const uint32_t seq = div_magic(o, P.magic_len), r = o - seq * len;
      const uint32_t y = div_magic(r, P.magic_m[st]), j = r - y * m;
      const uint32_t d = div_magic(j, P.magic_ns[st]), k = j - d * ns;
      uint32_t step = k * tstep + y * m, at = 0;
      if (step >= len) step -= len;
      const double2* src = s + seq * len + j;
      double2 acc = make_double2(0.0, 0.0);
      for (uint32_t q = 0; q < p; ++q) {
        const double2 a = src[q * m], w = tw[at];
        acc.x = fma(a.x, w.x, fma(-a.y, w.y, acc.x));
        acc.y = fma(a.x, w.y, fma(a.y, w.x, acc.y));
        at += step;
        if (at >= len) at -= len;
      }
      v[u] = acc;
      to[u] = seq * len + d * ns * p + k + y * ns;
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < E; ++u)
    if (threadIdx.x + uint32_t(u * T) < total) s[to[u]] = v[u];
  __syncthreads();
}

// The transform of nseq sequences in s (P.len values each, at most E T in
// all); every thread of the block calls it, with a barrier on either side.
// Plain lengths: s holds the values, then the spectra.  Bluestein: s holds
// x_k chirp_k padded with zeros to P.len; afterwards conj(s[k]) chirp_k is the
// spectrum at k < n.  `convolve` false: the stages alone.
template <int T, int E>
__device__ __forceinline__ void fft_block(double2* s, const FftPlan& P, uint32_t nseq,
                                          const double2* __restrict__ tab, bool convolve) {
  for (int pass = 0;; ++pass) {
    uint32_t ns = 1;
    for (int st = 0; st < P.stages; ++st) {
      switch (P.radix[st]) {
        case 2: fft_stage<T, E, 2>(s, P, st, ns, nseq, tab); break;
        case 3: fft_stage<T, E, 3>(s, P, st, ns, nseq, tab); break;
        case 4: fft_stage<T, E, 4>(s, P, st, ns, nseq, tab); break;
        case 5: fft_stage<T, E, 5>(s, P, st, ns, nseq, tab); break;
        case 7: fft_stage<T, E, 7>(s, P, st, ns, nseq, tab); break;
        case 8: fft_stage<T, E, 8>(s, P, st, ns, nseq, tab); break;
        default: fft_stage_prime<T, E>(s, P, st, ns, nseq, tab); break;
      }
      ns *= uint32_t(P.radix[st]);
    }
    if (!convolve || pass) return;
    const double2* filter = tab + P.len + P.n;
    const uint32_t len = uint32_t(P.len);
    for (uint32_t i = threadIdx.x; i < len * nseq; i += T) {
      const uint32_t seq = div_magic(i, P.magic_len);
      const double2 a = cmul(s[i], filter[i - seq * len]);
      s[i] = make_double2(a.x, -a.y);  // the inverse transform as a conjugated forward one
    }
    __syncthreads();
  }
}

// The tables of the row plan (blockIdx.y 0) and the column plan (1): roots
// e^{-2 pi i k / len}; for Bluestein also the chirps e^{-pi i k^2 / n}.
constexpr int kTabThreads = 256;
__global__ __launch_bounds__(kTabThreads) void k_fft_tables(FftPlan row, FftPlan col,
                                                            double2* __restrict__ row_tab,
                                                            double2* __restrict__ col_tab) {
  const FftPlan& P = blockIdx.y == 0 ? row : col;
  double2* tab = blockIdx.y == 0 ? row_tab : col_tab;
  const int k = int(blockIdx.x * kTabThreads + threadIdx.x);
  double s, c;
  if (k < P.len) {
    sincospi(2.0 * double(k) / double(P.len), &s, &c);
    tab[k] = make_double2(c, -s);
  }
  if (P.blue() && k < P.n) {
    sincospi(double((k * k) % (2 * P.n)) / double(P.n), &s, &c);
    tab[P.len + k] = make_double2(c, -s);
  }
}

// a + b, the rounding error added to e
__device__ __forceinline__ double add_exact(double a, double b, double& e) {
  const double s = a + b, t = s - a;
  e += (a - (s - t)) + (b - t);
  return s;
}

// The transform of the chirp filter conj(chirp_|k|), |k| < n, scaled by 1 / len.  It goes
// into every line of every image, so that its error stays where others average out: taken
// by a transform in FP64, it made the map of four images of 71x211 1.8e-16 off, 1.4 so.
// It is even, so a wave sums the n cosine terms of one value, with the roundings of
// products and sums carried along (and all waves of the chip do, where one block ran the
// transform: one image of 211x263 48 us, 36 so).  blockIdx.y as above.
__global__ __launch_bounds__(kTabThreads) void k_chirp_filter(FftPlan row, FftPlan col,
                                                              double2* __restrict__ row_tab,
                                                              double2* __restrict__ col_tab) {
  const FftPlan& P = blockIdx.y == 0 ? row : col;
  double2* tab = blockIdx.y == 0 ? row_tab : col_tab;
  const uint32_t len = uint32_t(P.len), n = uint32_t(P.n), lane = threadIdx.x & 63u;
  const uint32_t k = blockIdx.x * (kTabThreads / 64) + (threadIdx.x >> 6);
  if (!P.blue() || k > len / 2u) return;  // wave-uniform
  const double2* chirp = tab + len;
  const uint32_t x = lane * k, step = 64u * k - div_magic(64u * k, P.magic_len) * len;
  uint32_t at = x - div_magic(x, P.magic_len) * len;  // j k mod len
  double2 s = make_double2(0.0, 0.0), e = s;
  for (uint32_t j = lane; j < n; j += 64u) {
    const double2 h = chirp[j];
    const double c = j ? 2.0 * tab[at].x : 1.0;
    const double re = h.x * c, im = -h.y * c;
    e.x += fma(h.x, c, -re);
    e.y += fma(-h.y, c, -im);
    s.x = add_exact(s.x, re, e.x);
    s.y = add_exact(s.y, im, e.y);
    at += step;
    if (at >= len) at -= len;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const double sx = __shfl_xor(s.x, d, 64), sy = __shfl_xor(s.y, d, 64);
    const double ex = __shfl_xor(e.x, d, 64), ey = __shfl_xor(e.y, d, 64);
    s.x = add_exact(s.x, sx, e.x);
    s.y = add_exact(s.y, sy, e.y);
    e.x += ex;
    e.y += ey;
  }
  if (lane == 0) {
    const double scale = 1.0 / double(len);
    const double2 f = make_double2((s.x + e.x) * scale, (s.y + e.y) * scale);
    double2* filter = tab + len + n;
    filter[k] = f;
    if (k > 0) filter[len - k] = f;
  }
}

// A chirp convolution runs about twice as many stages as a plain transform, and its error is a few
// roundings of the size of what goes in.  So the mean of each row, and of the column of
// frequency 0, goes round it: rounded to float32, so that the differences of a row's
// values are exact, as is its product with the length, which is what it adds to frequency 0.
// Error of the map of an image in [0, 1), of its 2-norm: 607x809 1.7e-16, and 3.7e-16
// without this, 3.5e-16 with direct sums; 211x263 1.3, 4.0 and 2.1.
template <int T>
__device__ __forceinline__ double block_sum(double x, double* s_part) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = x;
  __syncthreads();
  x = 0.0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) x += s_part[w];
  __syncthreads();  // s_part is rewritten by the next call
  return x;
}

// Row pass: one block per two rows of a channel, transformed together as the
// real and imaginary part of one sequence; outputs the non-negative column
// frequencies kx = 0 .. W/2 of both rows.
template <int T, int E>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(T < 1024 ? 5 : 4))) void k_fft_rows(FftPlan P, int H, int W,
                                                const float* __restrict__ img,
                                                const double2* __restrict__ tab,
                                                double2* __restrict__ rows) {
  extern __shared__ double2 s_fft[];
  const int y = 2 * int(blockIdx.x), c = blockIdx.y;
  const bool two = y + 1 < H;
  const float* src = img + (size_t(c) * H + y) * W;
  const double2* chirp = tab + P.len;
  __shared__ double s_part[T / 64], s_mean[2];
  if (P.blue()) {  // block-uniform
    double2 sum = make_double2(0.0, 0.0);
    for (int x = threadIdx.x; x < W; x += T) {
      sum.x += double(src[x]);
      sum.y += two ? double(src[x + W]) : 0.0;
    }
    sum.x = block_sum<T>(sum.x, s_part);
    sum.y = block_sum<T>(sum.y, s_part);
    if (threadIdx.x == 0) {
      s_mean[0] = double(float(sum.x / double(W)));
      s_mean[1] = double(float(sum.y / double(W)));
    }
    __syncthreads();
  }
  for (int x = threadIdx.x; x < P.len; x += T) {
    double2 a = make_double2(0.0, 0.0);
    if (x < W) {
      a = make_double2(double(src[x]), two ? double(src[x + W]) : 0.0);
      if (P.blue()) a = cmul(make_double2(a.x - s_mean[0], a.y - s_mean[1]), chirp[x]);
    }
    s_fft[x] = a;
  }
  __syncthreads();
  fft_block<T, E>(s_fft, P, 1u, tab, P.blue());
  const int nk = W / 2 + 1;
  double2* dst = rows + (size_t(c) * H + y) * nk;
  for (int k = threadIdx.x; k < nk; k += T) {
    const int j = k == 0 ? 0 : W - k;
    double2 a = s_fft[k], b = s_fft[j];
    if (P.blue()) {
      a = cmul(make_double2(a.x, -a.y), chirp[k]);
      b = cmul(make_double2(b.x, -b.y), chirp[j]);
      if (k == 0) {
        a = make_double2(fma(double(W), s_mean[0], a.x), fma(double(W), s_mean[1], a.y));
        b = a;
      }
    }
    dst[k] = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
    if (two) dst[k + nk] = make_double2(0.5 * (a.y + b.y), 0.5 * (b.x - a.x));
  }
}

// Column pass: one block per C column frequencies, CH channels of them at a
// time, summing |F_c|^2 over the channels (a chirp of modulus 1 changes no
// norm).  Writes M(ky, kx) and, by conjugate symmetry, M(-ky, -kx); the image's
// norm is added to the running mean (first image: overwrite).  Blocks are
// dealt so that an XCD's columns are neighbours: their 16-byte pieces of the
// row spectra and the map then meet in one L2.
template <int T, int E, int CH>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4))) void k_fft_cols(FftPlan P, int H, int W, int C,
                                                const double2* __restrict__ rows,
                                                const double2* __restrict__ tab, double inv_n,
                                                int first, double* __restrict__ mag) {
  extern __shared__ double2 s_fft[];
  const int nk = W / 2 + 1, groups = (nk + C - 1) / C;
  const int per = (groups + kXcds - 1) / kXcds;
  const int grp = int(blockIdx.x % kXcds) * per + int(blockIdx.x / kXcds);
  if (int(blockIdx.x / kXcds) >= per || grp >= groups) return;  // block-uniform
  const int kx0 = grp * C, cols = min(C, nk - kx0);
  const double2* chirp = tab + P.len;
  // consecutive threads take the C columns (a power of two) of one row, then the next row
  const int cc = int(threadIdx.x) & (C - 1), yt = int(threadIdx.x) / C, dy = T / C;
  const bool in = cc < cols;
  const int kx = kx0 + cc, mx = (W - kx) % W;
  const bool mirror = in && mx != kx && mx >= nk;  // (-ky, -kx) is another column
  const bool centre = P.blue() && kx0 == 0;  // block-uniform: the block has frequency 0
  __shared__ double s_part[T / 64], s_mean[CH];
  double acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.0;
  for (int c0 = 0; c0 < 3; c0 += CH) {
    if (c0 > 0) __syncthreads();  // the previous channel's spectra are consumed
    if (centre) {
      for (int ch = 0; ch < CH; ++ch) {
        double sum = 0.0;
        for (int y = threadIdx.x; y < H; y += T) sum += rows[(size_t(c0 + ch) * H + y) * nk].x;
        sum = block_sum<T>(sum, s_part);
        if (threadIdx.x == 0) s_mean[ch] = double(float(sum / double(H)));
      }
      __syncthreads();
    }
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const double2* src = rows + size_t(c0 + ch) * H * nk + kx;
      double2* col = s_fft + (ch * C + cc) * P.len;
      for (int y = yt; y < P.len; y += dy) {
        double2 a = make_double2(0.0, 0.0);
        if (y < H && in) {
          a = src[size_t(y) * nk];
          if (centre && cc == 0) a.x -= s_mean[ch];
          if (P.blue()) a = cmul(a, chirp[y]);
        }
        col[y] = a;
      }
    }
    __syncthreads();
    fft_block<T, E>(s_fft, P, uint32_t(C * CH), tab, P.blue());
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int ky = yt + e * dy;
      if (ky < H) {
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
          double2 f = s_fft[(ch * C + cc) * P.len + ky];
          if (centre && cc + ky == 0) f.x = fma(double(H), s_mean[ch], f.x);  // (chirp 0 is 1)
          acc[e] = fma(f.x, f.x, fma(f.y, f.y, acc[e]));
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int ky = yt + e * dy;
    if (ky < H && in) {
      const double v = sqrt(acc[e]) * inv_n;
      const size_t o = size_t(ky) * W + kx, om = size_t(ky ? H - ky : 0) * W + mx;
      mag[o] = first ? v : mag[o] + v;
      if (mirror) mag[om] = first ? v : mag[om] + v;
    }
  }
}

// Small views: the sums themselves, a thread per frequency and one root per term, for
// lines of up to kDirect values together, kDirectChirp where one of them would need a
// chirp.  Both ways are chains of latency: the transforms' stages and barriers a fixed
// one, the sums' one step per term.  Four views, the sums and the transforms: 64x32 35 and
// 55 us, 80x48 40 and 56, 128x96 63 and 57, 200x132 121 and 66; with chirps 211x71 66 and
// 94, 250x67 71 and 76, 199x134 126 and 106; one view 20 and 31, 21 and 25, 35 and 34.
constexpr int kDirect = 144, kDirectChirp = 320;
constexpr int kDirectThreads = 128;
__global__ __launch_bounds__(256) void k_roots(int W, int H, double2* __restrict__ row_tab,
                                               double2* __restrict__ col_tab) {
  const int i = int(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= W + H) return;
  const int k = i < W ? i : i - W, n = i < W ? W : H;
  double s, c;
  sincospi(2.0 * double(k) / double(n), &s, &c);
  (i < W ? row_tab : col_tab)[k] = make_double2(c, -s);
}
// one block per row of a channel: its non-negative column frequencies
__global__ __launch_bounds__(kDirectThreads) void k_dft_rows(int H, int W,
                                                             const float* __restrict__ img,
                                                             const double2* __restrict__ tab,
                                                             double2* __restrict__ rows) {
  extern __shared__ double2 s_root[];  // W roots, then the row
  double* s_row = reinterpret_cast<double*>(s_root + W);
  const int y = blockIdx.x, c = blockIdx.y, nk = W / 2 + 1;
  const float* src = img + (size_t(c) * H + y) * W;
  for (int x = threadIdx.x; x < W; x += kDirectThreads) s_row[x] = double(src[x]), s_root[x] = tab[x];
  __syncthreads();
  for (int k = threadIdx.x; k < nk; k += kDirectThreads) {
    double re = 0.0, im = 0.0;
    int i = 0;  // x k mod W
#pragma unroll 8
    for (int x = 0; x < W; ++x) {
      const double2 w = s_root[i];
      re = fma(s_row[x], w.x, re);
      im = fma(s_row[x], w.y, im);
      i += k;
      i -= i >= W ? W : 0;
    }
    rows[(size_t(c) * H + y) * nk + k] = make_double2(re, im);
  }
}
// one block per column frequency, the three channels side by side; M as in k_fft_cols
__global__ __launch_bounds__(kDirectThreads) void k_dft_cols(int H, int W,
                                                             const double2* __restrict__ rows,
                                                             const double2* __restrict__ tab,
                                                             double inv_n, int first,
                                                             double* __restrict__ mag) {
  extern __shared__ double2 s_root[];  // H roots, then the three columns
  double2* s_col = s_root + H;
  const int kx = blockIdx.x, nk = W / 2 + 1, mx = (W - kx) % W;
  const bool mirror = mx != kx && mx >= nk;  // (-ky, -kx) is another column
  for (int y = threadIdx.x; y < H; y += kDirectThreads) {
    s_root[y] = tab[y];
#pragma unroll
    for (int c = 0; c < 3; ++c) s_col[c * H + y] = rows[(size_t(c) * H + y) * nk + kx];
  }
  __syncthreads();
  for (int ky = threadIdx.x; ky < H; ky += kDirectThreads) {
    double re[3] = {}, im[3] = {};
    int i = 0;  // y ky mod H
#pragma unroll 4
    for (int y = 0; y < H; ++y) {
      const double2 w = s_root[i];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double2 a = s_col[c * H + y];
        re[c] = fma(a.x, w.x, fma(-a.y, w.y, re[c]));
        im[c] = fma(a.x, w.y, fma(a.y, w.x, im[c]));
      }
      i += ky;
      i -= i >= H ? H : 0;
    }
    double sum = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) sum = fma(re[c], re[c], fma(im[c], im[c], sum));
    const double v = sqrt(sum) * inv_n;
    const size_t o = size_t(ky) * W + kx, om = size_t(ky ? H - ky : 0) * W + mx;
    mag[o] = first ? v : mag[o] + v;
    if (mirror) mag[om] = first ? v : mag[om] + v;
  }
}

// Anti-aliased downsampling of [n][C][H][W] to [n][C][h][w].  Output sample i
// weighs the inputs of its window with a triangle around (i + 0.5) in / out.
// Coordinates, weights and sums are FP64: in FP32 the tap centre
// (i + 0.5) H / h carries an error of 1e-4 px near H = 1000, which moves
// non-integer-factor weights.

// Downsampling by factors of 1 or more on both axes.  A block streams down a
// strip of input rows for up to kDsRows output rows: with its centres at least
// one input apart, an input row y weighs on two output rows only, the last one
// centred at or before it and the next, so every thread keeps two running sums
// per input column and each input is loaded once (plus one window per strip).
// When an output row is complete its column sums go through LDS and the threads
// sum their output columns' windows.  Row weights sit in LDS, formed once per
// block; a thread holds four input columns (one 16-byte load per row when the
// rows are 16-byte aligned) and the next kDsBatch rows are in flight while the
// current ones are summed.  64 views of 1200x800 to 300x200: 179 us, 4.4 TB/s of
// the 783 MB in and out (224 with 8 output rows a strip, room for four output columns
// a thread where one is used, and the column sums in one plane), against 882 us for one
// thread per output, which loads each input for the 4 outputs around it and forms every
// weight again.  Batches of 3 or 6 rows 187 and 182, of 8 275; strips of 25 rows 190.
constexpr int kDsRows = 16;      // output rows per block, or fewer where that leaves few blocks
constexpr int kDsBlocks = 1024, kDsFew = 256;
constexpr int kDsTable = 256;    // input rows a block may walk
constexpr int kDsBatch = 4;
constexpr int kDsThreads = 512;  // at most; 4 input columns per thread

// NU: output columns per thread, at most.  VEC: 16-byte loads.  PLANES: the columns'
// place in LDS.  Neighbouring outputs read a factor apart: where that is an even number
// of columns, or one, a thread's four columns go to four planes, so that such taps lie
// next to each other or nearly; at odd ones they spread over the banks as they are
// (factor 4: 212 us in one plane, 179 in four; factor 3, 16 views to 400x266: 80 and 85).
template <bool VEC, int NU, int PLANES>
__global__ __launch_bounds__(kDsThreads) void k_downsample_strip(
    int H, int W, int h, int w, int rows_out, int tile_w, int tiles_x, int groups_y,
    const float* __restrict__ src, float* __restrict__ dst) {
  extern __shared__ double s_col[];  // two buffers of 4 x blockDim.x column sums
  __shared__ double2 s_wy[kDsTable];
  __shared__ int s_low[kDsTable];
  __shared__ double s_ry[kDsRows];
  const int T = blockDim.x, tid = threadIdx.x;
  const unsigned tx = blockIdx.x % unsigned(tiles_x), r = blockIdx.x / unsigned(tiles_x);
  const int64_t plane = r / unsigned(groups_y);
  const int i0 = int(r % unsigned(groups_y)) * rows_out, i1 = min(h, i0 + rows_out);
  const int j0 = int(tx) * tile_w, j1 = min(w, j0 + tile_w);
  const double sy = double(H) / double(h), sx = double(W) / double(w);
  const double iy = 1.0 / sy, ix = 1.0 / sx;
  auto centre = [](int i, double s) { return (double(i) + 0.5) * s; };
  // inputs with |(p + 0.5) - c| < s lie in (c - s - 0.5, c + s - 0.5)
  auto first = [](double c, double s) { return max(0, int(floor(c - s - 0.5))); };
  auto last = [](double c, double s, int n) { return min(n - 1, int(ceil(c + s - 0.5))); };
  // exactly zero from one window's half-width on, whatever inv = 1 / half rounds to
  auto tri = [](double d, double half, double inv) {
    return fabs(d) < half ? fma(-fabs(d), inv, 1.0) : 0.0;
  };
  auto weight = [&](int p, double c, double half, double inv) {
    return tri(double(p) + 0.5 - c, half, inv);
  };
  int y0 = first(centre(i0, sy), sy), y1 = last(centre(i1 - 1, sy), sy, H);
  // rows of weight zero at the strip's ends are left out (0 x Inf is not 0)
  while (y0 < y1 && weight(y0, centre(i0, sy), sy, iy) == 0.0) ++y0;
  while (y0 < y1 && weight(y1, centre(i1 - 1, sy), sy, iy) == 0.0) --y1;
  const int ny = y1 - y0 + 1;  // at most kDsTable (the host's rows_out)
  for (int k = tid; k < ny; k += T) {
    const int y = y0 + k, lo = int(floor((double(y) + 0.5) * iy - 0.5));
    s_low[k] = lo;
    s_wy[k] = make_double2(weight(y, centre(lo, sy), sy, iy),
                           weight(y, centre(lo + 1, sy), sy, iy));
  }
  if (tid < i1 - i0) {
    const double c = centre(i0 + tid, sy);
    double sum = 0.0;
    for (int y = first(c, sy); y <= last(c, sy, H); ++y) sum += weight(y, c, sy, iy);
    s_ry[tid] = 1.0 / sum;
  }
  // input columns [x0, x0 + 4 T), the thread's: x0 + 4 tid + u, or x0 + tid + u T
  const int xa = first(centre(j0, sx), sx), x0 = VEC ? xa & ~3 : xa;
  const int span = last(centre(j1 - 1, sx), sx, W) - x0 + 1;  // at most 4 T (the host's tile_w)
  const float* s = src + plane * int64_t(H) * W;
  int at[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) at[u] = VEC ? 4 * tid + u : tid + u * T;
  const bool any = at[0] < span;
  auto load = [&](int k, float (&v)[4]) {
    const float* row = s + int64_t(y0 + min(k, ny - 1)) * W + x0;
    if (VEC) {
      const float4 q = *reinterpret_cast<const float4*>(row + (any ? at[0] : 0));
      v[0] = q.x, v[1] = q.y, v[2] = q.z, v[3] = q.w;
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = row[at[u] < span ? at[u] : 0];
    }
  };
  // the thread's output columns j0 + tid + u T: window, centre, 1 / weight sum
  double cx[NU], rx[NU];
  int xs[NU], xn[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int j = j0 + tid + u * T;
    xs[u] = xn[u] = 0;
    cx[u] = rx[u] = 0.0;
    if (j < j1) {
      const double c = centre(j, sx);
      const int a = first(c, sx), b = last(c, sx, W);
      double sum = 0.0;
      for (int x = a; x <= b; ++x) sum += weight(x, c, sx, ix);
      rx[u] = 1.0 / sum;
      xs[u] = a - x0;
      xn[u] = b - a + 1;
      cx[u] = double(a) + 0.5 - c;  // the window's first offset from the centre
    }
  }
  double acc0[4] = {0.0, 0.0, 0.0, 0.0}, acc1[4] = {0.0, 0.0, 0.0, 0.0};
  float cur[kDsBatch][4], nxt[kDsBatch][4];
#pragma unroll
  for (int b = 0; b < kDsBatch; ++b) load(b, cur[b]);
  __syncthreads();
  int i_cur = __builtin_amdgcn_readfirstlane(s_low[0]);
  auto place = [&](int c) { return PLANES == 4 ? (c & 3) * T + (c >> 2) : c; };
  auto emit = [&]() {  // output row i_cur is complete in acc0
    if (i_cur >= i0 && i_cur < i1) {
      double* buf = s_col + (i_cur & 1) * 4 * T;
#pragma unroll
      for (int u = 0; u < 4; ++u) buf[VEC && PLANES == 4 ? u * T + tid : place(at[u])] = acc0[u];
      __syncthreads();  // the other buffer is rewritten only after the next barrier
      const double ry = s_ry[i_cur - i0];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int j = j0 + tid + u * T;
        if (j < j1) {
          double row = 0.0, d = cx[u];
          for (int k = 0; k < xn[u]; ++k, d += 1.0)
            row = fma(tri(d, sx, ix), buf[place(xs[u] + k)], row);
          dst[(plane * h + i_cur) * int64_t(w) + j] = float(row * (rx[u] * ry));
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc0[u] = acc1[u], acc1[u] = 0.0;
    ++i_cur;
  };
  for (int k0 = 0; k0 < ny; k0 += kDsBatch) {
#pragma unroll
    for (int b = 0; b < kDsBatch; ++b) load(k0 + kDsBatch + b, nxt[b]);
#pragma unroll
    for (int b = 0; b < kDsBatch; ++b) {
      const int k = k0 + b;
      if (k < ny) {
        const int lo = __builtin_amdgcn_readfirstlane(s_low[k]);
        while (i_cur < lo) emit();
        const double2 wy = s_wy[k];
        // block-uniform: a row of weight zero is left out (0 x Inf is not 0)
        if (wy.x != 0.0) {
#pragma unroll
          for (int u = 0; u < 4; ++u) acc0[u] = fma(wy.x, double(cur[b][u]), acc0[u]);
        }
        if (wy.y != 0.0) {
#pragma unroll
          for (int u = 0; u < 4; ++u) acc1[u] = fma(wy.y, double(cur[b][u]), acc1[u]);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < kDsBatch; ++b)
#pragma unroll
      for (int u = 0; u < 4; ++u) cur[b][u] = nxt[b][u];
  }
  while (i_cur < i1) emit();
}

// Enlarging on an axis (two or three taps per output), or windows too long for
// the strips' tables (factors above about 100): one thread per output.
__global__ __launch_bounds__(256) void k_downsample(int64_t total, int H, int W, int h, int w,
                                                    const float* __restrict__ src,
                                                    float* __restrict__ dst) {
  const int64_t o = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (o >= total) return;
  const int j = int(o % w), i = int((o / w) % h);
  const int64_t plane = o / (int64_t(w) * h);
  const float* s = src + plane * int64_t(H) * W;
  const double sy = double(H) / double(h), sx = double(W) / double(w);
  const double hy = fmax(sy, 1.0), hx = fmax(sx, 1.0);
  const double cy = (double(i) + 0.5) * sy, cx = (double(j) + 0.5) * sx;
  // inputs with |(p + 0.5) - c| < half lie in (c - half - 0.5, c + half - 0.5)
  const int y0 = max(0, int(floor(cy - hy - 0.5))), y1 = min(H - 1, int(ceil(cy + hy - 0.5)));
  const int x0 = max(0, int(floor(cx - hx - 0.5))), x1 = min(W - 1, int(ceil(cx + hx - 0.5)));
  double wsum_x = 0.0;
  for (int x = x0; x <= x1; ++x) wsum_x += fmax(0.0, 1.0 - fabs((double(x) + 0.5 - cx) / hx));
  double acc = 0.0, wsum_y = 0.0;
  for (int y = y0; y <= y1; ++y) {
    const double wy = fmax(0.0, 1.0 - fabs((double(y) + 0.5 - cy) / hy));
    if (wy == 0.0) continue;
    wsum_y += wy;
    double row = 0.0;
    const float* sr = s + int64_t(y) * W;
    for (int x = x0; x <= x1; ++x)
      row = fma(fmax(0.0, 1.0 - fabs((double(x) + 0.5 - cx) / hx)), double(sr[x]), row);
    acc = fma(wy, row, acc);
  }
  dst[o] = float(acc / (wsum_x * wsum_y));
}

}  // namespace

namespace {

// appends n's factors to P (false when a prime factor is too large for a stage)
bool plan_stages(FftPlan& P, int n) {
  const int most = n <= kMidLine ? kMaxPrimeMid : kMaxPrime;
  P.stages = 0;
  auto add = [&](int r) { P.radix[P.stages++] = r; };
  int twos = 0;
  while (n % 2 == 0) n /= 2, ++twos;
  for (; twos >= 5 || twos == 3; twos -= 3) add(8);  // 2^4 as 4 x 4
  for (; twos >= 2; twos -= 2) add(4);
  if (twos) add(2);
  for (int p = 3; p <= most && n > 1; p += 2)
    while (n % p == 0) add(p), n /= p;
  return n == 1;
}

int pow2_from(int x) {
  int m = 1;
  while (m < x) m *= 2;
  return m;
}

// The stages of the chirp convolution for n go into P: of the 7-smooth lengths from 2 n - 1 on, up
// to 8 / 7 of it and to the power of two there, the one of fewest stages, each a barrier and
// a rounding (n = 211: 448 = 8 x 8 x 7 rather than 432 = 4 x 4 x 3 x 3 x 3).
void plan_chirp(FftPlan& P, int n) {
  const int least = 2 * n - 1, most = pow2_from(least);  // at most 8192 for n <= 4096
  int best = most, stages = kMaxStages + 1;
  for (int m = least; m <= most && (m - least) * 7 <= least; ++m) {
    int rest = m;
    for (int p : {2, 3, 5, 7})
      while (rest % p == 0) rest /= p;
    if (rest != 1) continue;
    plan_stages(P, m);
    if (P.stages < stages) best = m, stages = P.stages;
  }
  P.len = best;
  plan_stages(P, best);
}

FftPlan make_plan(int n) {
  FftPlan P{};
  P.n = P.len = n;
  if (!plan_stages(P, n)) plan_chirp(P, n);
  auto magic = [](uint32_t d) { return d == 1u ? 0u : uint32_t(((uint64_t(1) << 32) + d - 1) / d); };
  uint32_t ns = 1;
  for (int k = 0; k < P.stages; ++k) {
    P.magic_ns[k] = magic(ns);
    P.magic_m[k] = magic(uint32_t(P.len / P.radix[k]));
    ns *= uint32_t(P.radix[k]);
  }
  P.magic_len = magic(uint32_t(P.len));
  return P;
}

}  // namespace

// Room for either kind of tables whatever the factors, so that a workspace for an image holds for
// every smaller one (at most 0.6 MB beyond what the plans take).
size_t frequency_map_ws_bytes(int H, int W) {
  auto tables = [](int n) { return align256((2 * size_t(pow2_from(2 * n - 1)) + n) * sizeof(double2)); };
  return align256(size_t(3) * H * (W / 2 + 1) * sizeof(double2)) + tables(W) + tables(H);
}

hipError_t launch_frequency_map(int n_images, int H, int W, const float* images, double* mag,
                                void* ws, hipStream_t st) {
  const FftPlan row = make_plan(W), col = make_plan(H);
  char* p = static_cast<char*>(ws);
  double2* rows = reinterpret_cast<double2*>(p);
  p += align256(size_t(3) * H * (W / 2 + 1) * sizeof(double2));
  double2* row_tab = reinterpret_cast<double2*>(p);
  p += align256(row.table() * sizeof(double2));
  double2* col_tab = reinterpret_cast<double2*>(p);
  const double inv_n = 1.0 / double(n_images);
  if (W + H <= (row.blue() || col.blue() ? kDirectChirp : kDirect)) {
    GS_LAUNCH("k_roots", k_roots, dim3(unsigned((W + H + 255) / 256)), dim3(256), 0, st, W, H,
              row_tab, col_tab);
    for (int k = 0; k < n_images; ++k) {
      GS_LAUNCH("k_dft_rows", k_dft_rows, dim3(unsigned(H), 3u), dim3(kDirectThreads),
                size_t(W) * (sizeof(double2) + sizeof(double)), st, H, W,
                images + size_t(k) * 3 * H * W, row_tab, rows);
      GS_LAUNCH("k_dft_cols", k_dft_cols, dim3(unsigned(W / 2 + 1)), dim3(kDirectThreads),
                size_t(4) * H * sizeof(double2), st, H, W, rows, col_tab, inv_n, k == 0 ? 1 : 0,
                mag);
    }
    return hipGetLastError();
  }
  const int most = std::max(row.len, col.len);
  GS_LAUNCH("k_fft_tables", k_fft_tables, dim3(unsigned((most + kTabThreads - 1) / kTabThreads), 2u),
            dim3(kTabThreads), 0, st, row, col, row_tab, col_tab);
  const int chirps = std::max(row.blue() ? row.len : 0, col.blue() ? col.len : 0);
  if (chirps)
    GS_LAUNCH("k_chirp_filter", k_chirp_filter,
              dim3(unsigned((chirps / 2 + kTabThreads / 64) / (kTabThreads / 64)), 2u),
              dim3(kTabThreads), 0, st, row, col, row_tab, col_tab);
  // columns per block: up to 4 (64-byte pieces of the row spectra) while the
  // three channels' columns fit the register budget and 512 blocks remain, two
  // per CU (four 1200x800 views: 216 us with one column per block, 601 blocks,
  // against 222 with two); longer columns take one channel after the other
  int C = 4, CH = 3;
  while (C > 1 && (col.len * C * CH > 1024 * 5 || (W / 2 + C) / C < 512)) C /= 2;
  if (col.len * C * CH > 1024 * 5) CH = 1;
  const int nc = col.len * C * CH, groups = (W / 2 + C) / C;
  const dim3 rgrid(unsigned((H + 1) / 2), 3u);
  const dim3 cgrid(unsigned((groups + kXcds - 1) / kXcds * kXcds));
  const size_t rlds = size_t(row.len) * sizeof(double2), clds = size_t(nc) * sizeof(double2);
#define GS_FFT_ROWS(T, E)                                                                      \
  GS_LAUNCH("k_fft_rows", HIP_KERNEL_NAME(k_fft_rows<T, E>), rgrid, dim3(T), rlds, st, row, H, W, img, row_tab, \
            rows)
#define GS_FFT_COLS(T, E, CH)                                                                         \
  GS_LAUNCH("k_fft_cols", HIP_KERNEL_NAME(k_fft_cols<T, E, CH>), cgrid, dim3(T), clds, st, col, H, W, C, rows,         \
            col_tab, inv_n, k == 0 ? 1 : 0, mag)
  for (int k = 0; k < n_images; ++k) {
    const float* img = images + size_t(k) * 3 * H * W;
    if (row.len <= 64 * 5) GS_FFT_ROWS(64, 5);
    else if (row.len <= 256 * 5) GS_FFT_ROWS(256, 5);
    else if (row.len <= 512 * 5) GS_FFT_ROWS(512, 5);
    else GS_FFT_ROWS(1024, 8);
    if (CH == 3 && nc <= 256 * 5) GS_FFT_COLS(256, 5, 3);
    else if (CH == 3 && nc <= 512 * 5) GS_FFT_COLS(512, 5, 3);
    else if (CH == 3) GS_FFT_COLS(1024, 5, 3);
    else GS_FFT_COLS(1024, 8, 1);
  }
#undef GS_FFT_ROWS
#undef GS_FFT_COLS
  return hipGetLastError();
}

hipError_t launch_downsample(int n_planes, int H, int W, int h, int w, const float* src, float* dst,
                             hipStream_t st) {
  const int64_t total = int64_t(n_planes) * h * w;
  if (total == 0) return hipSuccess;
  const double sx = double(W) / double(w), sy = double(H) / double(h);
  if (sx >= 1.0 && sy >= 1.0) {
    // rows per strip: (rows + 1) sy + 3 input rows at most; columns per block:
    // (tile_w + 1) sx + 6 input columns at most, four per thread
    int rows_out = std::min(kDsRows, int((kDsTable - 3) / sy) - 1);
    const int most = int((4 * kDsThreads - 6) / sx) - 1;
    if (rows_out >= 1 && most >= 1) {
      const int tiles_x = (w + most - 1) / most, tile_w = (w + tiles_x - 1) / tiles_x;
      // A strip reads two output rows' window again, but few blocks leave CUs idle, and one
      // strip's rows are a chain: fewer rows a strip below kDsBlocks blocks, one below
      // kDsFew.  1 view of 400x264 to half 14.5 us in strips of 8, 9.4 of 4, 7.7 of 2, 7.8 of
      // 1 (a thread per output 7.9); 1 of 64x42 to an eighth 16.7, 15.0, 10.7, 8.3 (31.7);
      // 8 of 800x528 to a half 24, 25, 28, 37 (73).
      while (rows_out > 1 && int64_t(n_planes) * ((h + rows_out - 1) / rows_out) * tiles_x <
                                 (rows_out > 2 ? kDsBlocks : kDsFew))
        rows_out = (rows_out + 1) / 2;
      const int groups_y = (h + rows_out - 1) / rows_out;
      const int64_t blocks = int64_t(n_planes) * groups_y * tiles_x;
      const int span = std::min(W + 3, int((tile_w + 1) * sx) + 7);
      const int T = std::min(kDsThreads, ((span + 3) / 4 + 63) / 64 * 64);
      const bool vec = W % 4 == 0 && (reinterpret_cast<uintptr_t>(src) & 15u) == 0;
      const size_t lds = size_t(8) * T * sizeof(double);
      if (blocks < (int64_t(1) << 31)) {
        const int factor = int(sx + 0.5);
        const bool planes = vec && (factor == 1 || factor % 2 == 0), one = tile_w <= T;
        auto* const strip =
            planes ? (one ? k_downsample_strip<true, 1, 4> : k_downsample_strip<true, 4, 4>)
            : vec  ? (one ? k_downsample_strip<true, 1, 1> : k_downsample_strip<true, 4, 1>)
                   : (one ? k_downsample_strip<false, 1, 1> : k_downsample_strip<false, 4, 1>);
        GS_LAUNCH("k_downsample_strip", strip, dim3(unsigned(blocks)), dim3(unsigned(T)), lds, st,
                  H, W, h, w, rows_out, tile_w, tiles_x, groups_y, src, dst);
        return hipGetLastError();
      }
    }
  }
  GS_LAUNCH("k_downsample", k_downsample, dim3(unsigned((total + 255) / 256)), dim3(256), 0, st,
            total, H, W, h, w, src, dst);
  return hipGetLastError();
}

// ---- host: crop significance over a summed-area table of the centred map
struct CropTable {
  int H, W;
  std::vector<double> sat;  // (H+1) x (W+1) prefix sums of the map with DC at (H/2, W/2)
  CropTable(const double* mag, int H_, int W_) : H(H_), W(W_), sat(size_t(H_ + 1) * (W_ + 1), 0.0) {
    for (int j = 0; j < H; ++j) {
      const int ky = (j + H - H / 2) % H;  // centred row j holds frequency j - H/2
      double run = 0.0;
      for (int i = 0; i < W; ++i) {
        const int kx = (i + W - W / 2) % W;
        run += mag[size_t(ky) * W + kx];
        sat[size_t(j + 1) * (W + 1) + (i + 1)] = sat[size_t(j) * (W + 1) + (i + 1)] + run;
      }
    }
  }
  // sum of the map over |f_y| <= H/(2r), |f_x| <= W/(2r), times 1/r^2 or 1/(H W)
  bool per_pixel = false;
  double significance(double r) const {
    const int by = int(std::floor(double(H) / (2.0 * r))), bx = int(std::floor(double(W) / (2.0 * r)));
    const int y0 = std::max(0, H / 2 - by), y1 = std::min(H - 1, H / 2 + by);
    const int x0 = std::max(0, W / 2 - bx), x1 = std::min(W - 1, W / 2 + bx);
    const double s = sat[size_t(y1 + 1) * (W + 1) + (x1 + 1)] - sat[size_t(y0) * (W + 1) + (x1 + 1)] -
                     sat[size_t(y1 + 1) * (W + 1) + x0] + sat[size_t(y0) * (W + 1) + x0];
    return per_pixel ? s / (double(H) * double(W)) : s / (r * r);
  }
  // largest r in [1, r_max] with significance(r) >= target (bisection)
  double solve(double target, double r_max) const {
    if (significance(r_max) >= target) return r_max;
    double lo = 1.0, hi = r_max;
    for (int it = 0; it < 60; ++it) {
      const double mid = 0.5 * (lo + hi);
      if (significance(mid) >= target)
        lo = mid;
      else
        hi = mid;
    }
    return lo;
  }
};

void resolution_schedule(const double* mag, int H, int W, double S, double a, int m, double r_max,
                         int per_pixel, double* r_knots, double* s_knots, double* x_knots) {
  CropTable T(mag, H, W);
  T.per_pixel = per_pixel != 0;
  const double XF = T.significance(1.0), Xm = XF / a;
  for (int i = 0; i <= m; ++i) {
    const double Xi = XF - (XF - Xm) * double(i) / double(m);
    r_knots[i] = (i == 0) ? 1.0 : T.solve(Xi, r_max);
    s_knots[i] = S * std::log(Xi / Xm) / std::log(XF / Xm);
    if (x_knots) x_knots[i] = Xi;
  }
}

}  // namespace gsk

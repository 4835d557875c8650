// Discrete Fourier transform by Cooley-Tukey on the tensor unit (Section
// 4.5, Theorem 7): y[k] = sum_j x[j] exp(-2 pi i j k / n), for a batch of
// complex vectors (binary32 real and imaginary parts, interleaved).
//
// The section arranges x as an s x (n/s) matrix, replaces every column by
// its DFT -- the tall product X^T W_s, n/s rows through the unit -- scales
// entry (r, c) by the twiddle w_n^(r c), transposes, and recurses on the s
// rows (a last level of radix n/s^(L-1) <= s).  A level reads the whole array
// and writes it reordered (a Stockham ordering: the digits of k already
// produced are kept as the fastest-varying index), so the last level leaves y
// in natural order with no separate transpose.  With n = R_1 ... R_L,
// P_t = R_1 ... R_(t-1) and N_t = n / P_t:
//   level t reads  a[j] = src[j (n/R_t) + c],           c = J P_t + K,
//   and writes     dst[(J R_t + k) P_t + K] = f(J, k) sum_j a[j] w_(R_t)^(j k)
// for every transform c < n/R_t (J < N_t/R_t, K < P_t) and k < R_t, with the
// twiddle f(J, k) = w_(N_t)^(J k) (1 on the last level).
// Two consecutive full-radix levels t, t+1 form a pair, and their twiddles
// are regrouped: with N' = N_t / S and J = J' + j' (N'/S),
//   w_(N_t)^(J k) = w_(N_t)^(J' k) w_(S^2)^(j' k),
// and the first factor does not depend on j', the index level t+1 (transform
// J', K + k P_t) sums over; so level t multiplies by w_(S^2)^(j' k), a table of
// S^2 entries, and level t+1 by w_(N_t)^(J' (k + S k')), which costs what its
// own twiddle does and nothing on the last level, where J' = 0.
//
// One launch holds as many levels as it can:
//   * vectors of up to 2^13 elements: all of them, in LDS (dft_local_kernel;
//     few long ones in more launches, see local_fits);
//   * else pairs of full-radix levels, through LDS (dft_pair_kernel), and
//     single levels (dft_level_kernel).
// Every kernel forms a value by the same operations, so the results do not
// depend on how the levels are divided into launches, bit for bit.
//
// On the unit: 16 columns per wave step, S contracted elements and S outputs
// each; the weights operand is W_S (rows = output frequency k, contracted index
// j), formed once per wave.  A last level of radix R < S takes S/R transforms
// per column, its weights S/R diagonal blocks W_R (a column of one transform
// would leave S - R of its elements empty).  The zeros between the blocks keep
// the transforms of a column apart only while every word is finite (0 x Inf is
// NaN), so an element that is not is replaced by zero and every output of its
// transform by NaN, what the products with its words would give
// (dft_set_apart): an infinite or NaN value, or one past bfloat16's range,
// reaches its own transform alone.  Complex products are real products
// on the bf16 matrix cores: Re = Wr Xr - Wi Xi, Im = Wi Xr + Wr Xi.  The data
// and W each enter as the sum of two bf16 words (hi + lo), and every real
// product is formed as hi*hi + hi*lo + lo*hi into binary32 accumulators, about
// 2^-16 relative accuracy (one bf16 rounding would cost 2^-9 per level).  The
// twiddles are computed in the kernel: w_N^m for N <= 2^20 as the product of
// two entries of per-workgroup LDS tables (each the sincospi of an exact
// angle), above that as one sincospi of the exactly reduced angle; nothing is
// stored between launches.
#include <mutex>

#include "tcu_device.h"
#include "tcu_split.h"
#include "tcu_launch.h"

namespace tcu {
namespace {

constexpr int kDftThreads = 256;

typedef float f32x2 __attribute__((ext_vector_type(2)));

// exp(-2 pi i m / N) for 0 <= m < N, N a power of two: (cos, -sin) of pi x,
// x = 2m/N formed exactly (N is a power of two).
__device__ __forceinline__ f32x2 twiddle(int64_t m, int64_t N) {
  const float x = (float)m * (2.0f / (float)N);
  float s, c;
  sincospif(x, &s, &c);
  return f32x2{c, -s};
}

// Complex product of two (re, im) pairs (the roundings written out, so that
// every kernel takes the same ones).
__device__ __forceinline__ f32x2 cmul(f32x2 a, f32x2 b) {
  return f32x2{__builtin_fmaf(a[0], b[0], -(a[1] * b[1])),
               __builtin_fmaf(a[0], b[1], a[1] * b[0])};
}

// Twiddles of one level, N = 2^L: for L <= kTabLg,
//   w_N^m = T_hi[m >> b] * T_lo[m mod 2^b],   b = ceil(L / 2),
// T_lo[i] = w_N^i (i < 2^b) and T_hi[i] = w_N^(i 2^b) (i < 2^(L-b)), built
// in LDS by the workgroup (2^b + 2^(L-b) <= 2048 sincospi evaluations, in
// place of about three per lane and transform step); above kTabLg every
// twiddle is one sincospi.  The choice depends on L alone.
constexpr int kTabLg = 20;
__host__ __device__ constexpr int tab_entries(int L) {
  return L <= kTabLg ? (1 << ((L + 1) / 2)) + (1 << (L / 2)) : 0;
}
struct TwTab {
  const f32x2 *lo = nullptr;   // LDS; null: no table
  const f32x2 *hi = nullptr;
  int b = 0;
  int lg = 0;                  // L
};
// Fill pool[0 .. tab_entries(L)) (threads tid < nthreads share the work);
// the caller synchronises the workgroup before the first lookup.
__device__ __forceinline__ TwTab build_tab(f32x2 *pool, int L, int tid, int nthreads) {
  TwTab t;
  t.lg = L;
  if (L > kTabLg) return t;
  t.b = (L + 1) / 2;
  const int nlo = 1 << t.b, nhi = 1 << (L - t.b);
  const int64_t N = (int64_t)1 << L;
  for (int i = tid; i < nlo + nhi; i += nthreads)
    pool[i] = i < nlo ? twiddle(i, N) : twiddle((int64_t)(i - nlo) << t.b, N);
  t.lo = pool;
  t.hi = pool + nlo;
  return t;
}
// w_N^(m mod N).
__device__ __forceinline__ f32x2 tw(const TwTab &t, int64_t m) {
  const int64_t mm = m & (((int64_t)1 << t.lg) - 1);
  if (t.lo == nullptr) return twiddle(mm, (int64_t)1 << t.lg);
  return cmul(t.hi[mm >> t.b], t.lo[mm & ((1 << t.b) - 1)]);
}

// The first twiddles of a pair, w_(S^2)^(j' k) at S j' + k: S^2 sincospi
// evaluations per workgroup, read four at a time.
template <int S>
__device__ __forceinline__ void build_pair_tab(f32x2 *v, int tid, int nthreads) {
  for (int i = tid; i < S * S; i += nthreads) v[i] = twiddle((i / S) * (i % S), S * S);
}

// Shapes of a radix-S step on the unit: a lane holds kRun consecutive
// contracted elements, and the S output frequencies come in kH halves of 16.
template <int S>
struct DftShape {
  static constexpr int kRun = S == 32 ? 8 : 4;   // contracted elements per lane
  static constexpr int kH = S / 16;              // 16-frequency halves
  static constexpr int kWords = kRun / 2;
  typedef typename std::conditional<kRun == 8, u32x4, u32x2>::type Run;
};

// The weights operand as hi/lo words: S/R diagonal blocks W_R (R <= S), row
// 16h + r of the unit operand = block u = row / R, frequency k = row mod R, and
// contracted run kRun g + e likewise; -Wi for the real part.  wtab[m] = w_R^m.
template <int S>
struct DftWeights {
  typedef typename DftShape<S>::Run Run;
  Run wr_h[DftShape<S>::kH], wr_l[DftShape<S>::kH], wi_h[DftShape<S>::kH],
      wi_l[DftShape<S>::kH], ni_h[DftShape<S>::kH], ni_l[DftShape<S>::kH];
};
template <int S>
__device__ __forceinline__ void dft_weights(DftWeights<S> &W, const f32x2 *wtab, int lg_r, int r,
                                            int g, SplitConsts sc) {
  constexpr int kRun = DftShape<S>::kRun, kH = DftShape<S>::kH, kWords = DftShape<S>::kWords;
#pragma unroll
  for (int h = 0; h < kH; ++h) {
    float cr[kRun], ci[kRun];
    const int k = 16 * h + r;
#pragma unroll
    for (int e = 0; e < kRun; ++e) {
      const int j = kRun * g + e;   // (j k mod R does not see the blocks' bits)
      const f32x2 w = j >> lg_r == k >> lg_r ? wtab[(j * k) & ((1 << lg_r) - 1)] : f32x2{0.f, 0.f};
      cr[e] = w[0];
      ci[e] = w[1];
    }
#pragma unroll
    for (int q = 0; q < kWords; ++q) {
      unsigned hi, lo;
      split_bf16x2(cr[2 * q], cr[2 * q + 1], hi, lo, sc);
      W.wr_h[h][q] = hi;
      W.wr_l[h][q] = lo;
      split_bf16x2(ci[2 * q], ci[2 * q + 1], hi, lo, sc);
      W.wi_h[h][q] = hi;
      W.wi_l[h][q] = lo;
      W.ni_h[h][q] = hi ^ 0x80008000u;   // -Wi: flip both signs
      W.ni_l[h][q] = lo ^ 0x80008000u;
    }
  }
}

// One transform column of the unit (lane (r, g) holds its elements
// j = kRun g + e): the data as hi/lo words, then for half h the real and
// imaginary parts of outputs 16h + 4g + i, i < 4 (the matrix-core output
// layout), each real product formed as hi*hi + hi*lo + lo*hi.
template <int S>
struct DftData {
  typename DftShape<S>::Run xr_h, xr_l, xi_h, xi_l;
};
template <int S>
__device__ __forceinline__ void dft_data(DftData<S> &X, const float *xr, const float *xi,
                                         SplitConsts sc) {
#pragma unroll
  for (int q = 0; q < DftShape<S>::kWords; ++q) {
    unsigned hi, lo;
    split_bf16x2(xr[2 * q], xr[2 * q + 1], hi, lo, sc);
    X.xr_h[q] = hi;
    X.xr_l[q] = lo;
    split_bf16x2(xi[2 * q], xi[2 * q + 1], hi, lo, sc);
    X.xi_h[q] = hi;
    X.xi_l[q] = lo;
  }
}
// Elements of a narrow level's column that are not finite as bfloat16 words
// (Inf, NaN, or a magnitude that rounds to Inf): whether a lane holds one, the
// largest magnitude of its elements (NaN if one is) given ...
constexpr unsigned kDftLimit = 0x7f7f8000u;   // halfway from the largest bfloat16 to Inf
template <int S>
__device__ __forceinline__ float dft_largest(float m, const f32x2 (&v)[DftShape<S>::kRun]) {
#pragma unroll
  for (int e = 0; e < DftShape<S>::kRun; ++e)
    m = __builtin_elementwise_maximum(
        __builtin_elementwise_maximum(m, __builtin_fabsf(v[e][0])), __builtin_fabsf(v[e][1]));
  return m;
}
__device__ __forceinline__ bool dft_not_finite(float largest) {
  return !(largest < bitcast<float>(kDftLimit));
}
// ... and their replacement by zero; returns the column's set of transforms that
// hold one, bit u for slots u R .. u R + R - 1.
template <int S>
__device__ __forceinline__ unsigned dft_set_apart(f32x2 (&v)[DftShape<S>::kRun], int g, int lg_r) {
  unsigned set = 0;
#pragma unroll
  for (int e = 0; e < DftShape<S>::kRun; ++e) {
    if (dft_not_finite(__builtin_elementwise_maximum(__builtin_fabsf(v[e][0]),
                                                     __builtin_fabsf(v[e][1])))) {
      v[e] = f32x2{0.f, 0.f};
      set |= 1u << ((DftShape<S>::kRun * g + e) >> lg_r);
    }
  }
  set |= (unsigned)__shfl_xor((int)set, 16);
  return set | (unsigned)__shfl_xor((int)set, 32);
}
// NaN to this lane's outputs of the transforms in the set, after the others:
// `put(k, nan)` stores output k (a rolled loop: this is the rare case).
template <int S, typename Put>
__device__ __forceinline__ void dft_put_spoilt(unsigned set, int g, int lg_r, Put put) {
  const float nan = __builtin_nanf("");
#pragma unroll 1
  for (int j = 0; j < 4 * DftShape<S>::kH; ++j) {
    const int k = 16 * (j >> 2) + 4 * g + (j & 3);
    if (set >> (k >> lg_r) & 1u) put(k, f32x2{nan, nan});
  }
}
template <int S>
__device__ __forceinline__ void dft_half(const DftWeights<S> &W, const DftData<S> &X, int h,
                                         f32x4 &re, f32x4 &im) {
  typedef typename DftShape<S>::Run Run;
  auto mma = [&](const Run &w, const Run &x, f32x4 d) __attribute__((always_inline)) {
    if constexpr (S == 32)
      return mfma_k32(TCU_BF16_F32, w, x, d);
    else
      return mfma_k16(TCU_BF16_F32, w, x, d);
  };
  re = f32x4{0.f, 0.f, 0.f, 0.f};
  im = f32x4{0.f, 0.f, 0.f, 0.f};
  re = mma(W.wr_h[h], X.xr_h, re);
  re = mma(W.wr_h[h], X.xr_l, re);
  re = mma(W.wr_l[h], X.xr_h, re);
  re = mma(W.ni_h[h], X.xi_h, re);
  re = mma(W.ni_h[h], X.xi_l, re);
  re = mma(W.ni_l[h], X.xi_h, re);
  im = mma(W.wi_h[h], X.xr_h, im);
  im = mma(W.wi_h[h], X.xr_l, im);
  im = mma(W.wi_l[h], X.xr_h, im);
  im = mma(W.wr_h[h], X.xi_h, im);
  im = mma(W.wr_h[h], X.xi_l, im);
  im = mma(W.wr_l[h], X.xi_h, im);
}
// Outputs k0 .. k0+3 of one transform times w_N^(m0 + i m), i < 4: the first
// factor, then repeated products with step = w_N^m.
__device__ __forceinline__ void dft_twiddle4(f32x2 (&y)[4], int64_t m0, const TwTab &tab,
                                             f32x2 step) {
  f32x2 w = tw(tab, m0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    y[i] = cmul(y[i], w);
    if (i < 3) w = cmul(w, step);
  }
}
// The same with the first twiddles of a pair: v points at those of output k0
// (16-byte aligned).
__device__ __forceinline__ void dft_pair_twiddle4(f32x2 (&y)[4], const f32x2 *v) {
  const f32x4 a = *(const f32x4 *)v, b = *(const f32x4 *)(v + 2);
  y[0] = cmul(y[0], f32x2{a[0], a[1]});
  y[1] = cmul(y[1], f32x2{a[2], a[3]});
  y[2] = cmul(y[2], f32x2{b[0], b[1]});
  y[3] = cmul(y[3], f32x2{b[2], b[3]});
}

// How a level's outputs are scaled: not at all (the last level), by its own
// twiddles, or by the first or second factors of a pair.
enum Scale { kNone = 0, kOwn = 1, kPairFirst = 2, kPairSecond = 3 };

// One transform column's outputs scaled: outputs k0 .. k0+3 of transform (J,
// K) of a level with lg_p = log2 P, N_t = 2^lg_nt.
template <int S>
struct DftScale {
  static constexpr int lg_s = S == 32 ? 5 : 4;
  int scale = kNone;
  int lg_jp = 0;                 // first of a pair: log2 (N'/S)
  int lg_p0 = 0;                 // second: log2 P of the first
  const f32x2 *pair = nullptr;   // w_(S^2)^(j' k)
  TwTab tab;                     // of N_t (own) or the first level's N_t (second)
  // log2 of the table's N (0: none) of a level with these sizes
  __device__ __forceinline__ static int tab_lg(int scale, int lg_nt) {
    return scale == kOwn ? lg_nt : scale == kPairSecond ? lg_nt + lg_s : 0;
  }
  struct Col {                   // per transform
    int64_t base, per_k;         // exponent of output k0: base + per_k k0
    f32x2 step;
    const f32x2 *v;
  };
  __device__ __forceinline__ Col col(int64_t J, int64_t K) const {
    Col c{0, 0, f32x2{1.f, 0.f}, nullptr};
    if (scale == kOwn) {
      c.per_k = J;
      c.step = tw(tab, J);
    } else if (scale == kPairFirst) {
      c.v = pair + ((J >> lg_jp) << lg_s);
    } else if (scale == kPairSecond) {
      c.base = J * (K >> lg_p0);
      c.per_k = J << lg_s;
      c.step = tw(tab, c.per_k);
    }
    return c;
  }
  __device__ __forceinline__ void apply(f32x2 (&y)[4], const Col &c, int k0) const {
    if (scale == kPairFirst)
      dft_pair_twiddle4(y, c.v + k0);
    else if (scale != kNone)
      dft_twiddle4(y, c.base + c.per_k * k0, tab, c.step);
  }
};

// Element indices of one wave step of a level, in an array of whole vectors:
// lane (r, g) of column r holds slots kRun g + e, and outputs 16 h + 4 g + i.
// kNarrow (a last level of radix R < S): slot u R + j is element j of
// transform tr + 16 u, and the outputs likewise; otherwise one transform.
template <int S, bool kNarrow, typename Idx>
struct LevelIndex {
  static constexpr int kRun = DftShape<S>::kRun;
  int lg_n, lg_r, lg_p;
  Idx tr, vec, c;              // first transform of this lane's column; its vector and c
  int g;
  __device__ __forceinline__ LevelIndex(int lg_n_, int lg_r_, int lg_p_, Idx tr_, int g_)
      : lg_n(lg_n_), lg_r(lg_r_), lg_p(lg_p_), tr(tr_), g(g_) {
    const int lg_pv = lg_n - lg_r;
    vec = (tr >> lg_pv) << lg_n;
    c = tr & (((Idx)1 << lg_pv) - 1);
  }
  __device__ __forceinline__ Idx trans(int slot) const {   // the slot's transform
    return kNarrow ? tr + 16 * (slot >> lg_r) : tr;
  }
  __device__ __forceinline__ Idx in(int e) const {
    const int slot = kRun * g + e, lg_pv = lg_n - lg_r;
    if constexpr (!kNarrow) return vec + c + ((Idx)slot << lg_pv);
    const Idx t = trans(slot);
    return ((t >> lg_pv) << lg_n) + (t & (((Idx)1 << lg_pv) - 1)) +
           ((Idx)(slot & ((1 << lg_r) - 1)) << lg_pv);
  }
  __device__ __forceinline__ Idx out(int k) const {
    if constexpr (!kNarrow) {
      const Idx J = c >> lg_p, K = c & (((Idx)1 << lg_p) - 1);
      return vec + (((J << lg_r) + k) << lg_p) + K;
    }
    // the last level: J = 0, P = n / R
    const Idx t = trans(k);
    return ((t >> lg_p) << lg_n) + (t & (((Idx)1 << lg_p) - 1)) +
           ((Idx)(k & ((1 << lg_r) - 1)) << lg_p);
  }
};

// One level.  n, R, P, N_t are powers of two and enter as their base-2
// logarithms; ntrans = batch * n / R transforms, 16 S/R per wave step.
// R < S (kNarrow) only on the last level, which scales nothing: its kernel holds no
// table and no code for one (n = 2^14, s = 32, 32 MiB: 194 -> 161 registers, two ->
// three waves per SIMD; with the grid of launch_level 17.8 -> 12.1 us).
template <int S, bool kNarrow>
__global__ __launch_bounds__(kDftThreads) void dft_level_kernel(
    const f32x2 *__restrict__ src, f32x2 *__restrict__ dst, int lg_n, int lg_r, int lg_p,
    int64_t ntrans, int scale_, int lg_p0) {
  constexpr int kRun = DftShape<S>::kRun, kH = DftShape<S>::kH;
  constexpr int lg_s = DftScale<S>::lg_s;
  __shared__ f32x2 wtab[S];               // w_R^m, m < R
  // the one table that `scale` asks for: of a pair's first twiddles, or of N_t
  constexpr int kPool = kNarrow ? 1 : tab_entries(kTabLg);
  static_assert(kNarrow || kPool >= S * S, "the pair table fits");
  __shared__ __attribute__((aligned(16))) f32x2 pool[kPool];
  const int scale = kNarrow ? kNone : scale_;

  const int R = 1 << lg_r;
  const int lg_nt = lg_n - lg_p;          // log2 N_t
  const int lg_sub = lg_s - lg_r;         // log2 of the transforms per column
  const bool contiguous = lg_p == 0 && R >= 4;   // a lane's 4 outputs are adjacent

  if (threadIdx.x < (unsigned)R) wtab[threadIdx.x] = twiddle(threadIdx.x, R);
  DftScale<S> sf;
  sf.scale = scale;
  sf.lg_jp = lg_nt - 2 * lg_s;
  sf.lg_p0 = lg_p0;
  sf.pair = pool;
  if (scale == kPairFirst) build_pair_tab<S>(pool, threadIdx.x, kDftThreads);
  if (scale == kOwn || scale == kPairSecond)
    sf.tab = build_tab(pool, DftScale<S>::tab_lg(scale, lg_nt), threadIdx.x, kDftThreads);
  __syncthreads();

  const int lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const SplitConsts sc = split_consts();
  DftWeights<S> W;
  dft_weights<S>(W, wtab, lg_r, r, g, sc);

  const int64_t wave = (int64_t)blockIdx.x * (kDftThreads / 64) + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * (kDftThreads / 64);
  const int64_t nchunks = (ntrans + (16 << lg_sub) - 1) >> (4 + lg_sub);
  for (int64_t chunk = wave; chunk < nchunks; chunk += nwaves) {
    const LevelIndex<S, kNarrow, int64_t> at(lg_n, lg_r, lg_p, (chunk << (4 + lg_sub)) + r, g);
    f32x2 v[kRun];
#pragma unroll
    for (int e = 0; e < kRun; ++e) {
      v[e] = f32x2{0.f, 0.f};
      if (at.trans(kRun * g + e) < ntrans) v[e] = src[at.in(e)];
    }
    const bool apart = kNarrow && __any(dft_not_finite(dft_largest<S>(0.f, v)));
    unsigned spoilt = 0;
    if (apart) spoilt = dft_set_apart<S>(v, g, lg_r);
    float xr[kRun], xi[kRun];
#pragma unroll
    for (int e = 0; e < kRun; ++e) {
      xr[e] = v[e][0];
      xi[e] = v[e][1];
    }
    DftData<S> X;
    dft_data<S>(X, xr, xi, sc);
    const typename DftScale<S>::Col col = sf.col(at.c >> lg_p, at.c & (((int64_t)1 << lg_p) - 1));
#pragma unroll
    for (int h = 0; h < kH; ++h) {
      f32x4 re, im;
      dft_half<S>(W, X, h, re, im);
      const int k0 = 16 * h + 4 * g;
      f32x2 y[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] = f32x2{re[i], im[i]};
      sf.apply(y, col, k0);
      if (contiguous) {   // outputs k0 .. k0+3 of one transform: 32 adjacent bytes
        if (at.trans(k0) < ntrans) {
          f32x4 *o = (f32x4 *)(dst + at.out(k0));
          o[0] = f32x4{y[0][0], y[0][1], y[1][0], y[1][1]};
          o[1] = f32x4{y[2][0], y[2][1], y[3][0], y[3][1]};
        }
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (at.trans(k0 + i) < ntrans) dst[at.out(k0 + i)] = y[i];
      }
    }
    if (apart)
      dft_put_spoilt<S>(spoilt, g, lg_r, [&](int k, f32x2 nan) {
        if (at.trans(k) < ntrans) dst[at.out(k)] = nan;
      });
  }
}

// Two consecutive levels t, t+1 of radix S in one launch (both R = S, and
// P_t >= 16 or P_t = 1).  With P = P_t, N' = N_t / S and P' = P S, level
// t+1's transform (J', K' = k P + K) reads output k of level t's
// transforms J = J' + j' (N'/S), j' < S, with the same K.  So the S x S
// values of group (J', K) -- level t's transforms J (rows j') by their
// outputs k -- are formed and consumed inside one workgroup, through LDS:
//   * a workgroup takes 16 groups at once: 16 consecutive K (P >= 16,
//     kLaneK) or 16 consecutive J' (P = 1), so that the level-t loads and
//     the level-(t+1) stores of the 16 matrix-core columns are contiguous;
//   * level t: S steps j' (a wave takes every 8th), each the 16 groups'
//     transforms J = J' + j' (N'/S) as in dft_level_kernel (all of a wave's
//     loads issued first), outputs times w_(S^2)^(j' k) into the LDS tile
//     T[group][j'][k];
//   * level t+1: S steps, each 16 transforms over j' read from the tiles
//     (kLaneK: output k of the 16 groups; otherwise 16 consecutive k of one
//     group), outputs times w_(N_t)^(J' (k + S k')) unless it is the last
//     level, stored in level t+1's Stockham order.
// A tile's time is its memory traffic plus both levels' vector work (one
// workgroup per CU, its phases in turn), so the twiddles matter: with each
// level's own ones -- a table product and three more complex products per four
// outputs on both levels -- n = 2^20, batch 16 took 67 + 53 us (memory alone
// 54 each).
constexpr int kPairGroups = 16;
template <int S>
constexpr int pair_row() { return S + 1; }                          // j' rows, padded
template <int S>
constexpr int pair_group() { return S * pair_row<S>() + 1; }       // one group's tile

constexpr int kPairThreads = 512;   // 8 waves: two per SIMD

template <int S, bool kLaneK, bool kStream>
__global__ __launch_bounds__(kPairThreads) void dft_pair_kernel(
    const f32x2 *__restrict__ src, f32x2 *__restrict__ dst, int lg_n, int lg_p, int64_t ntiles,
    int last2) {
  constexpr int kRun = DftShape<S>::kRun, kH = DftShape<S>::kH;
  constexpr int lg_s = DftScale<S>::lg_s;
  constexpr int kWaves = kPairThreads / 64;
  constexpr int kSteps = S / kWaves;                // level steps per wave
  constexpr int kRow = pair_row<S>(), kGrp = pair_group<S>();
  __shared__ f32x2 wtab[S];
  __shared__ f32x2 tile[kPairGroups * kGrp];
  __shared__ __attribute__((aligned(16))) f32x2 vtab[S * S];
  __shared__ f32x2 pool[tab_entries(kTabLg)];

  const int lg_nt = lg_n - lg_p;             // level t: N_t
  const int lg_jp = lg_nt - 2 * lg_s;        // log2 (N'/S): the J' range
  const int lg_pv = lg_n - lg_s;             // n / S: level t's element stride

  if (threadIdx.x < (unsigned)S) wtab[threadIdx.x] = twiddle(threadIdx.x, S);
  build_pair_tab<S>(vtab, threadIdx.x, kPairThreads);
  TwTab tab;
  if (!last2) tab = build_tab(pool, lg_nt, threadIdx.x, kPairThreads);
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int wv = threadIdx.x >> 6;
  const SplitConsts sc = split_consts();
  DftWeights<S> W;
  dft_weights<S>(W, wtab, lg_s, r, g, sc);

  // tiles per vector: (N'/S) (P/16) with kLaneK, (N'/S)/16 otherwise
  const int lg_tpv = kLaneK ? lg_jp + lg_p - 4 : lg_jp - 4;
  for (int64_t q = blockIdx.x; q < ntiles; q += gridDim.x) {
    const int64_t b = q >> lg_tpv;
    const int64_t ql = q & (((int64_t)1 << lg_tpv) - 1);
    const f32x2 *vsrc = src + (b << lg_n);
    f32x2 *vdst = dst + (b << lg_n);
    // this lane's group: J'_r and K_r
    const int64_t Jp = kLaneK ? ql >> (lg_p - 4) : (ql << 4) + r;
    const int64_t Kr = kLaneK ? ((ql & (((int64_t)1 << (lg_p - 4)) - 1)) << 4) + r : 0;

    // ---- level t: the wave's steps j' = wv + kWaves i, loads issued first
    f32x2 v[kSteps][kRun];
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      const int64_t J = Jp + ((int64_t)(wv + kWaves * i) << lg_jp);
      const f32x2 *vin = vsrc + (J << lg_p) + Kr;
#pragma unroll
      for (int e = 0; e < kRun; ++e)
        v[i][e] = kStream ? __builtin_nontemporal_load(vin + ((int64_t)(kRun * g + e) << lg_pv))
                          : vin[(int64_t)(kRun * g + e) << lg_pv];
    }
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      const int jp = wv + kWaves * i;
      float xr[kRun], xi[kRun];
#pragma unroll
      for (int e = 0; e < kRun; ++e) {
        xr[e] = v[i][e][0];
        xi[e] = v[i][e][1];
      }
      DftData<S> X;
      dft_data<S>(X, xr, xi, sc);
#pragma unroll
      for (int h = 0; h < kH; ++h) {
        f32x4 re, im;
        dft_half<S>(W, X, h, re, im);
        const int k0 = 16 * h + 4 * g;
        f32x2 y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = f32x2{re[e], im[e]};
        dft_pair_twiddle4(y, vtab + jp * S + k0);
        f32x2 *t = tile + r * kGrp + jp * kRow + k0;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = y[e];
      }
    }
    __syncthreads();

    // ---- level t+1: the wave's steps
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      const int ch = wv + kWaves * i;
      int grp, k;
      if constexpr (kLaneK) {
        grp = r;
        k = ch;
      } else {
        grp = ch / (S / 16);
        k = 16 * (ch % (S / 16)) + r;
      }
      const int64_t J2 = kLaneK ? Jp : (ql << 4) + grp;          // level t+1's J'
      const int64_t K2 = ((int64_t)k << lg_p) + (kLaneK ? Kr : 0);
      float xr[kRun], xi[kRun];
      const f32x2 *t = tile + grp * kGrp + k;
#pragma unroll
      for (int e = 0; e < kRun; ++e) {
        const f32x2 a = t[(kRun * g + e) * kRow];
        xr[e] = a[0];
        xi[e] = a[1];
      }
      DftData<S> X;
      dft_data<S>(X, xr, xi, sc);
      f32x2 *vout = vdst + ((J2 << lg_s) << (lg_p + lg_s)) + K2;
      const f32x2 step = last2 ? f32x2{1.f, 0.f} : tw(tab, J2 << lg_s);
#pragma unroll
      for (int h = 0; h < kH; ++h) {
        f32x4 re, im;
        dft_half<S>(W, X, h, re, im);
        const int k0 = 16 * h + 4 * g;
        f32x2 y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = f32x2{re[e], im[e]};
        if (!last2) dft_twiddle4(y, J2 * k + (J2 << lg_s) * k0, tab, step);
#pragma unroll
        for (int e = 0; e < 4; ++e) vout[(int64_t)(k0 + e) << (lg_p + lg_s)] = y[e];
      }
    }
    __syncthreads();   // the tiles are rewritten by the next iteration
  }
}

// Whole transforms in LDS: vectors of n <= 2^kLgT elements, kLgT >= 12 being
// the tile a workgroup holds -- one vector, or 2^kLgT / n short ones.  The tile is
// read and written in order (whole lines, past the caches: each byte is touched
// once), every level works in place on it: a wave reads its columns' elements of a
// level into registers, all waves synchronise, and the outputs go where the
// Stockham order puts them.  16 waves per CU: two workgroups of 8 with a tile
// of 2^12 (122 registers), one of 16 with 2^13.  With the weights in registers
// instead of LDS the first spilled (batch 4096 of n = 4096: 180 us, 70 here).
// Three launches of n = 4096, batch 512 moved the array three times and took
// 38.3 us, one takes 12.4; n = 64, batch 2^18 237 -> 54 us (5 TB/s).
// Elements are padded by one per 32 against bank conflicts.
template <int kLgT>
constexpr int local_pad() { return (1 << kLgT) + (1 << (kLgT - 5)); }
__device__ __forceinline__ int local_at(int i) { return i + (i >> 5); }

constexpr int local_threads(int lg_t) { return lg_t == 12 ? 512 : 1024; }

template <int S, int kLgT>
__global__ __attribute__((amdgpu_flat_work_group_size(local_threads(kLgT), local_threads(kLgT)),
                          amdgpu_waves_per_eu(4))) void
dft_local_kernel(const f32x2 *__restrict__ src, f32x2 *__restrict__ dst, int lg_n, int64_t total,
                 int64_t ntiles) {
  constexpr int kThreads = local_threads(kLgT);
  constexpr int kRun = DftShape<S>::kRun, kH = DftShape<S>::kH;
  constexpr int lg_s = DftScale<S>::lg_s;
  constexpr int kWaves = kThreads / 64;
  constexpr int T = 1 << kLgT;
  constexpr int kSteps = T / (16 * S) / kWaves;      // columns' steps per wave
  constexpr int kLin = T / kThreads;             // elements per thread, in order
  typedef typename DftShape<S>::Run Run;
  __shared__ f32x2 wtab[2][S];                       // w_S^m; w_R^m of the last level
  __shared__ f32x2 tile[local_pad<kLgT>()];
  __shared__ __attribute__((aligned(16))) f32x2 vtab[S * S];
  __shared__ f32x2 pool[tab_entries(kLgT) + tab_entries(6)];
  // the weights of W_S and of the last level, kept in LDS: the registers go
  // to the columns, and a level reads them once per half and step
  __shared__ Run weights[2][4 * kH][64];

  int levels = 1;
  for (int l = lg_s; l < lg_n; l += lg_s) ++levels;
  const int lg_last = lg_n - lg_s * (levels - 1);    // the last level's radix
  const bool narrow = lg_last < lg_s;

  if (threadIdx.x < (unsigned)S) {
    wtab[0][threadIdx.x] = twiddle(threadIdx.x, S);
    if ((int)threadIdx.x < (1 << lg_last))
      wtab[1][threadIdx.x] = twiddle(threadIdx.x, 1 << lg_last);
  }
  // Levels in pairs from the first; one left alone has its own twiddles
  // (unless it is the last).  n <= 2^13 has at most four levels, so only the
  // first pair's second level and one level alone need tables.
  const int full = narrow ? levels - 1 : levels;     // full-radix levels
  const int first_alone = full & ~1;                 // index of the unpaired one, if any
  const bool alone = full % 2 == 1 && first_alone < levels - 1;
  const bool second = full >= 2 && levels > 2;       // the first pair's second level scales
  TwTab tab_n, tab_a;
  if (full >= 2) build_pair_tab<S>(vtab, threadIdx.x, kThreads);
  if (second) tab_n = build_tab(pool, lg_n, threadIdx.x, kThreads);
  if (alone)
    tab_a = build_tab(pool + (second ? tab_entries(lg_n) : 0), lg_n - lg_s * first_alone,
                      threadIdx.x, kThreads);
  __syncthreads();

  const int lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SplitConsts sc = split_consts();
  if (wv < 2) {
    DftWeights<S> W;
    dft_weights<S>(W, wtab[wv], wv ? lg_last : lg_s, r, g, sc);
#pragma unroll
    for (int h = 0; h < kH; ++h) {
      weights[wv][4 * h][lane] = W.wr_h[h];
      weights[wv][4 * h + 1][lane] = W.wr_l[h];
      weights[wv][4 * h + 2][lane] = W.wi_h[h];
      weights[wv][4 * h + 3][lane] = W.wi_l[h];
    }
  }

  // One level in place: radix 2^lg_r, P = 2^lg_p.
  auto level = [&](auto narrow_c, int lg_r, int lg_p, const DftScale<S> &sf)
      __attribute__((always_inline)) {
    constexpr bool kNarrow = decltype(narrow_c)::value;
    typedef LevelIndex<S, kNarrow, int> Index;
    const int lg_sub = lg_s - lg_r;
    const Run(*const ws)[64] = weights[kNarrow ? 1 : 0];
    f32x2 v[kSteps][kRun];
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      const Index at(lg_n, lg_r, lg_p, ((wv + kWaves * i) << (4 + lg_sub)) + r, g);
#pragma unroll
      for (int e = 0; e < kRun; ++e) v[i][e] = tile[local_at(at.in(e))];
    }
    bool apart = false;
    unsigned spoilt[kSteps];
    if constexpr (kNarrow) {
      float largest = 0.f;
#pragma unroll
      for (int i = 0; i < kSteps; ++i) largest = dft_largest<S>(largest, v[i]);
      apart = __any(dft_not_finite(largest));
      if (apart) {
#pragma unroll
        for (int i = 0; i < kSteps; ++i) spoilt[i] = dft_set_apart<S>(v[i], g, lg_r);
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      const Index at(lg_n, lg_r, lg_p, ((wv + kWaves * i) << (4 + lg_sub)) + r, g);
      float xr[kRun], xi[kRun];
#pragma unroll
      for (int e = 0; e < kRun; ++e) {
        xr[e] = v[i][e][0];
        xi[e] = v[i][e][1];
      }
      DftData<S> X;
      dft_data<S>(X, xr, xi, sc);
      const typename DftScale<S>::Col col = sf.col(at.c >> lg_p, at.c & ((1 << lg_p) - 1));
#pragma unroll
      for (int h = 0; h < kH; ++h) {
        DftWeights<S> W;
        W.wr_h[h] = ws[4 * h][lane];
        W.wr_l[h] = ws[4 * h + 1][lane];
        W.wi_h[h] = ws[4 * h + 2][lane];
        W.wi_l[h] = ws[4 * h + 3][lane];
        W.ni_h[h] = W.wi_h[h] ^ 0x80008000u;
        W.ni_l[h] = W.wi_l[h] ^ 0x80008000u;
        f32x4 re, im;
        dft_half<S>(W, X, h, re, im);
        const int k0 = 16 * h + 4 * g;
        f32x2 y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = f32x2{re[e], im[e]};
        sf.apply(y, col, k0);
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[local_at(at.out(k0 + e))] = y[e];
      }
    }
    if (apart) {
#pragma unroll
      for (int i = 0; i < kSteps; ++i) {
        const Index at(lg_n, lg_r, lg_p, ((wv + kWaves * i) << (4 + lg_sub)) + r, g);
        dft_put_spoilt<S>(spoilt[i], g, lg_r,
                          [&](int k, f32x2 nan) { tile[local_at(at.out(k))] = nan; });
      }
    }
    __syncthreads();
  };

  for (int64_t q = blockIdx.x; q < ntiles; q += gridDim.x) {
    const int64_t base = q << kLgT;
    const int count = (int)(total - base < T ? total - base : T);   // whole vectors
    f32x2 in[kLin];
#pragma unroll
    for (int i = 0; i < kLin; ++i) {
      const int at = threadIdx.x + kThreads * i;
      in[i] = at < count ? __builtin_nontemporal_load(src + base + at) : f32x2{0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < kLin; ++i) tile[local_at(threadIdx.x + kThreads * i)] = in[i];
    __syncthreads();

    int lg_p = 0;
    for (int t = 0; t < full; ++t) {
      const bool last = t == levels - 1;
      DftScale<S> sf;
      sf.pair = vtab;
      sf.lg_jp = lg_n - lg_p - 2 * lg_s;
      sf.lg_p0 = lg_p - lg_s;
      if (t < first_alone)
        sf.scale = t % 2 == 0 ? kPairFirst : last ? kNone : kPairSecond;
      else
        sf.scale = last ? kNone : kOwn;
      sf.tab = sf.scale == kPairSecond ? tab_n : tab_a;
      level(std::false_type{}, lg_s, lg_p, sf);
      lg_p += lg_s;
    }
    if (narrow) level(std::true_type{}, lg_last, lg_p, DftScale<S>{});

#pragma unroll
    for (int i = 0; i < kLin; ++i) {
      const int at = threadIdx.x + kThreads * i;
      if (at < count) __builtin_nontemporal_store(tile[local_at(at)], dst + base + at);
    }
    __syncthreads();   // the tile is rewritten by the next iteration
  }
}

// Scratch of the allocation-free DFT (tcu_dft_noalloc): the levels' second
// buffer.  In host code this name is only a stand-in for the symbol; the
// array's device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[TCU_DFT_NOALLOC_MAX_BYTES];

int ilog2(int64_t v) {
  int l = 0;
  while (((int64_t)1 << l) < v) ++l;
  return l;
}

// Whether levels t, t+1 (radix S each, P = P_t) form a pair (both full
// radix), and whether a pair runs as one launch: a coalesced lane order exists
// (16 consecutive K, or P = 1 with at least 16 groups J' per vector).
bool is_pair(int64_t n, int s, int64_t P) { return n / P / s >= s; }
bool pair_launch(int64_t n, int s, int64_t P) {
  if (knob(TCU_KNOB_DFT_PAIRS) == 1) return false;   // test override: single levels
  return P >= 16 || (P == 1 && n / s / s >= 16);
}

template <int S>
hipError_t launch_pair(const f32x2 *src, f32x2 *dst, int64_t n, int64_t P, int64_t batch,
                       bool last2, hipStream_t stream, int num_cus) {
  const int64_t ntiles = batch * (n / ((int64_t)S * S)) / kPairGroups;
  const int64_t cap = num_cus;      // one workgroup per CU (the tiles take most of the LDS)
  const int blocks = (int)(ntiles < cap ? ntiles : cap);
  // The caller's input (P = 1) of an array that the memory-side cache cannot
  // hold beside the other two is read past the caches, so that it does not
  // push out what the next launch reads: n = 2^20, batch 16 (128 MiB) 127 ->
  // 118 us, n = 2^16, batch 256, s = 16 128 -> 114 us.  Below that it depends on
  // the input (us, plain / past the caches; in the cache from the call before, from a
  // kernel that wrote it just before, or in neither):
  //   s = 16, n = 2^20, 32 MiB 48.3 / 51.3, 60.4 / 63.4, 50.0 / 51.4;
  //                     64 MiB 84.9 / 91.3, 108 / 112, 90.9 / 92.1;
  //           n = 2^14, 64 MiB 73.0 / 77.9, 94.9 / 99.4, 83.0 / 80.0;
  //           n = 2^16, 96 MiB 85.5 / 81.6, 111 / 111, 87.4 / 85.3;
  //   s = 32, n = 2^20, 32 MiB 29.6 / 35.1, 42.5 / 44.7, 35.9 / 35.1;
  //                     64 MiB 54.9 / 59.3, 78.4 / 81.7, 60.7 / 57.9;
  //           n = 2^14, 32 MiB 30.1 / 30.6, 42.1 / 43.2, 36.3 / 30.7.
  // So s = 16 reads it plainly up to 64 MiB; s = 32, whose shorter launches lose
  // more on an input that is in no cache, below 32 (n = 2^20, 16 MiB 23.2 / 24.9).
  const bool stream_in = S == 32 ? batch * n * 8 >= (int64_t)32 << 20
                             : batch * n * 8 > (int64_t)64 << 20;
  // Later pairs read the other buffer for the last time, past the caches from
  // 64 MiB on: its lines then make room for the output's.  n = 2^20, batch 16
  // 113.1 -> 110.2 us, batch 8 58.7 -> 57.2; batch 4 (32 MiB) 30.8 both.
  const bool stream_work = batch * n * 8 >= (int64_t)64 << 20;
  if (P >= 16 && stream_work)
    hipLaunchKernelGGL((dft_pair_kernel<S, true, true>), dim3(blocks), dim3(kPairThreads), 0,
                       stream, src, dst, ilog2(n), ilog2(P), ntiles, last2 ? 1 : 0);
  else if (P >= 16)
    hipLaunchKernelGGL((dft_pair_kernel<S, true, false>), dim3(blocks), dim3(kPairThreads), 0,
                       stream, src, dst, ilog2(n), ilog2(P), ntiles, last2 ? 1 : 0);
  else if (stream_in)
    hipLaunchKernelGGL((dft_pair_kernel<S, false, true>), dim3(blocks), dim3(kPairThreads), 0,
                       stream, src, dst, ilog2(n), ilog2(P), ntiles, last2 ? 1 : 0);
  else
    hipLaunchKernelGGL((dft_pair_kernel<S, false, false>), dim3(blocks), dim3(kPairThreads), 0,
                       stream, src, dst, ilog2(n), ilog2(P), ntiles, last2 ? 1 : 0);
  return hipGetLastError();
}

template <int S>
hipError_t launch_level(const f32x2 *src, f32x2 *dst, int64_t n, int R, int64_t P,
                        int64_t batch, Scale scale, hipStream_t stream, int num_cus) {
  const int64_t ntrans = batch * (n / R);
  const int64_t per_chunk = 16 * S / R;
  const int64_t nchunks = (ntrans + per_chunk - 1) / per_chunk;
  const int64_t want = (nchunks + 3) / 4;
  // A narrow level's workgroups are bound by its two passes over memory and hold
  // three per CU (s = 32): with that many the weights are formed once, 12 per CU
  // are faster when the array no longer stays in the memory-side cache (us, 3 / 8 / 12
  // per CU, whole transforms of n = 2^14, s = 32: 24 MiB 23.8 / 25.2 / 25.4, 32 MiB
  // 29.0 / 30.6 / 30.8, 64 MiB 53.1 / 53.2 / 54.2, 256 MiB 219 / 222 / 217; n = 2^18,
  // 256 MiB 320 / 314 / 307).
  const int64_t per_cu = R == S ? 8 : batch * n * 8 <= (int64_t)64 << 20 ? 3 : 12;
  const int64_t cap = num_cus * per_cu;
  const int blocks = (int)(want < cap ? want : cap);
  const int lg_p0 = scale == kPairSecond ? ilog2(P / S) : 0;
  if (R < S)
    hipLaunchKernelGGL((dft_level_kernel<S, true>), dim3(blocks), dim3(kDftThreads), 0, stream,
                       src, dst, ilog2(n), ilog2(R), ilog2(P), ntrans, (int)scale, lg_p0);
  else
    hipLaunchKernelGGL((dft_level_kernel<S, false>), dim3(blocks), dim3(kDftThreads), 0, stream,
                       src, dst, ilog2(n), ilog2(R), ilog2(P), ntrans, (int)scale, lg_p0);
  return hipGetLastError();
}

// Whole transforms per workgroup (n <= 2^kLocalLg).
constexpr int kLocalLg = 13;
template <int S, int kLgT>
hipError_t launch_local_t(const f32x2 *src, f32x2 *dst, int64_t n, int64_t batch,
                          hipStream_t stream, int num_cus) {
  const int64_t total = batch * n, ntiles = (total + (1 << kLgT) - 1) >> kLgT;
  const int64_t cap = (int64_t)num_cus * (kLgT == 12 ? 2 : 1);
  hipLaunchKernelGGL((dft_local_kernel<S, kLgT>), dim3((unsigned)(ntiles < cap ? ntiles : cap)),
                     dim3(local_threads(kLgT)), 0, stream, src, dst, ilog2(n), total, ntiles);
  return hipGetLastError();
}
template <int S>
hipError_t launch_local(const f32x2 *src, f32x2 *dst, int64_t n, int64_t batch,
                        hipStream_t stream, int num_cus) {
  if (n <= 1 << 12) return launch_local_t<S, 12>(src, dst, n, batch, stream, num_cus);
  return launch_local_t<S, 13>(src, dst, n, batch, stream, num_cus);
}

// Whether whole vectors per workgroup are the faster division: up to 2^13
// elements, except few long vectors with s = 16, whose three or four levels in one
// workgroup each take longer than the launches that spread them over the chip
// (us, whole / divided: n = 2^13, batch 1 13.1 / 10.3, 32 14.2 / 12.4, 64 14.4 / 14.9;
// n = 2^12, 1 7.6 / 6.7, 32 8.3 / 7.4, 64 8.2 / 8.1, 128 8.3 / 9.4; s = 32, n = 2^13,
// 1 10.7 / 11.8).
bool local_fits(int64_t n, int64_t batch, int s, int num_cus) {
  if (n > (int64_t)1 << kLocalLg || knob(TCU_KNOB_DFT_PAIRS) == 1) return false;
  return !(s == 16 && n >= 1 << 12 && 4 * batch < num_cus);
}

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxScratchDevices] = {};

// The scratch array's address on the current device (each device holds its
// own copy), resolved with that device current on its first use there.
hipError_t scratch_on_current_device(void **ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace

int dft_levels(int64_t n, int s) {
  int L = 1;
  for (int64_t m = s; m < n; m *= s) ++L;
  return L;
}

hipError_t launch_dft(const void *x, void *y, void *work, int64_t n, int64_t batch, int s,
                      hipStream_t stream, int num_cus) {
  if (n <= 0 || batch <= 0) return hipSuccess;
  if (local_fits(n, batch, s, num_cus))
    return s == 32 ? launch_local<32>((const f32x2 *)x, (f32x2 *)y, n, batch, stream, num_cus)
                   : launch_local<16>((const f32x2 *)x, (f32x2 *)y, n, batch, stream, num_cus);
  const int L = dft_levels(n, s);
  // The launches (decided before anything is launched): a pair of levels as
  // one where possible, else one per level.
  struct Step {
    bool pair;      // both levels of a pair
    Scale scale;    // single level: how its outputs are scaled
  } steps[64];
  int launches = 0;
  {
    int64_t P = 1;
    for (int t = 1; t <= L;) {
      if (t < L && is_pair(n, s, P)) {
        if (pair_launch(n, s, P)) {
          steps[launches++] = Step{true, kNone};
        } else {
          steps[launches++] = Step{false, kPairFirst};
          steps[launches++] = Step{false, t + 1 == L ? kNone : kPairSecond};
        }
        P *= (int64_t)s * s;
        t += 2;
      } else {
        steps[launches++] = Step{false, t == L ? kNone : kOwn};
        P *= s;
        t += 1;
      }
    }
  }
  int64_t P = 1;
  const f32x2 *src = (const f32x2 *)x;
  for (int i = 0, t = 1; i < launches; ++i) {
    // the launches alternate between work and y so that the last lands in y
    f32x2 *dst = (f32x2 *)((launches - 1 - i) % 2 == 0 ? y : work);
    hipError_t e;
    if (steps[i].pair) {
      const bool last2 = t + 1 == L;
      e = s == 32 ? launch_pair<32>(src, dst, n, P, batch, last2, stream, num_cus)
                  : launch_pair<16>(src, dst, n, P, batch, last2, stream, num_cus);
      P *= (int64_t)s * s;
      t += 2;
    } else {
      const int R = (int)(t < L ? s : n / P);
      e = s == 32 ? launch_level<32>(src, dst, n, R, P, batch, steps[i].scale, stream, num_cus)
                  : launch_level<16>(src, dst, n, R, P, batch, steps[i].scale, stream, num_cus);
      P *= R;
      t += 1;
    }
    if (e != hipSuccess) return e;
    src = dst;
  }
  return hipSuccess;
}

hipError_t launch_dft_noalloc(const void *x, void *y, int64_t n, int64_t batch, int s,
                              hipStream_t stream, int num_cus) {
  if (n <= 0 || batch <= 0) return hipSuccess;
  void *work = nullptr;
  if (dft_levels(n, s) > 1) {
    const hipError_t e = scratch_on_current_device(&work);
    if (e != hipSuccess) return e;
  }
  return launch_dft(x, y, work, n, batch, s, stream, num_cus);
}

}  // namespace tcu

// Batch polynomial evaluation of Theorem 11 (Section 4.8):
// out[i] = A(x_i) = sum_{h<n} a_h x_i^h for p points x_i.
//
// The theorem's method, fused into one launch, with KP powers per column:
//   * X (p x KP): row i holds x_i^0 .. x_i^(KP-1);
//   * the coefficients, read column-major, form the KP x (n/KP) matrix with
//     entry (k, j) = a_(k + j KP);
//   * C = X times that matrix;
//   * A(x_i) = sum_j C[i][j] x_i^(j KP).
// KP is 16 or 32: the unit size s, or 16 for a short polynomial.
// Each wave owns chunks of 32 points, one point per matrix-core column:
//   * it computes the powers of its points in binary32 (the theorem's
//     initial exponentiation, as a ladder of squarings shared by all lanes
//     plus a short chain per lane) and hands X to the unit as an unevaluated
//     sum of two bfloat16 words, X = X_hi + X_lo, so the unit multiplies X
//     to about 2^-17 relative accuracy instead of one 16-bit rounding -- the
//     model multiplies exactly, and one rounding of x^k would dominate the
//     error;
//   * a block is 32 columns; its weights come from LDS, where the workgroup
//     stages the coefficients, padded with zeros past n, once (or, for
//     polynomials longer than the stage, per stage and pass).  Read from
//     memory by every wave, the rows 2 KP bytes apart kept L1 busy as long as
//     the products, and a last block that n cut was read element by element (n = 1000,
//     2^24 points: 454 us, 127 now);
//   * two 32x32x16 matrix-core products per 16 powers (X_hi, then X_lo into the
//     same binary32 accumulators);
//   * binary16 inputs are driven through the unit in bfloat16 too: the
//     5-bit exponent of a binary16 word cannot hold x^k for small |x|
//     (x^(KP-1) below 2^-14 loses bits, below 2^-25 vanishes), while bfloat16
//     has binary32's range.  Each binary16 coefficient is split exactly into
//     two bfloat16 words c_hi + c_lo (its 11 significant bits fit in 8 + 8)
//     when it is staged, and every step takes four products,
//     (X_hi + X_lo)(c_hi + c_lo);
//   * lane (r, g) then holds C[point r][columns 8a + 4g + i] of the block
//     and forms t = sum over them of C y^(8a + i), y = x^KP, by Horner's
//     rule in y; the blocks are walked last to first and combined by
//     Horner's rule in y^32 (acc = acc * y^32 + t), and the lane's factor
//     y^(4g) is applied once -- the final combine, never writing C;
//   * the two lanes holding one point add their sums (cross-lane
//     exchange) and one stores A(x_i).
// Coefficients past n and points past p are zero padding.  Results are
// meaningful while |x|^(n-1) and the partial sums stay within binary32
// range (the theorem assumes evaluation without overflow or underflow).
// The vector work (powers, split, combine) and the matrix cores add up rather
// than overlap here: a pass of 64 points at n = 4096 spends about as long on
// each, and at n = 65536 the products run at the rate the power limit allows
// the large matrix products; reading the weights a block ahead, interleaving the
// combine with the products by scheduling barriers, or raising the priority of the
// products changed nothing or lost.  16 x 16 blocks (four lanes per point: twice
// the ladders, half the columns per product) took 290 us for n = 4096 and 2^24
// points where 32 x 32 take 272.
#include "tcu_device.h"
#include "tcu_split.h"
#include "tcu_launch.h"

namespace tcu {
namespace {

constexpr int kPolyCols = 32;      // output columns per block of coefficients

template <int DT>
__device__ __forceinline__ float in_to_f32(unsigned bits16) {
  if constexpr (DT == TCU_F16_F32)
    return (float)__builtin_bit_cast(_Float16, (unsigned short)bits16);
  else
    return bf16_to_f32(bits16);
}

// A word of two binary16 coefficients as the exact sum of two words of
// bfloat16 pairs (11 significant bits in 8 + 8).
__device__ __forceinline__ void f16_pair_to_bf16(unsigned w, unsigned &hi, unsigned &lo,
                                                 SplitConsts sc) {
  const float f0 = (float)bitcast<_Float16>((unsigned short)(w & 0xffffu));
  const float f1 = (float)bitcast<_Float16>((unsigned short)(w >> 16));
  split_bf16x2(f0, f1, hi, lo, sc);
}

// KP powers per column of the coefficient matrix (X is p x KP), U chunks of 32
// points per wave and pass, kThreads per workgroup around a stage of kStage
// bytes of coefficients in LDS.
template <int DT, int KP, int U, int kThreads, int kStage>
__global__ __launch_bounds__(kThreads) void poly_kernel(const unsigned char *__restrict__ coef,
                                                        int64_t n,
                                                        const unsigned char *__restrict__ pts,
                                                        int64_t np, unsigned char *__restrict__ out,
                                                        int64_t nchunks, int64_t nblocks) {
  // Powers a shorter polynomial never uses (k >= n in X, output columns
  // j >= ceil(n/KP) in the combine) are replaced by zeros rather than
  // computed, so they cannot overflow where the polynomial itself does not.
  const int64_t ncols = (n + KP - 1) / KP;
  constexpr int kQ = KP / 16;             // matrix-core steps of 16 powers
  // The unit runs in bfloat16 for every input type (binary16 coefficients
  // split into two bfloat16 words each, see above).
  constexpr bool kF16 = DT == TCU_F16_F32;
  constexpr int UDT = TCU_BF16_F32;
  constexpr int kBlock = kPolyCols * KP;  // coefficients per block

  const int lane = threadIdx.x & 63;
  const int r = lane & 31, g = lane >> 5;
  const SplitConsts sc = split_consts();
  // Wave-uniform chunk indices (readfirstlane: the compiler cannot prove
  // threadIdx.x >> 6 uniform), so point addresses are a scalar base plus a
  // per-lane 32-bit offset.
  const int64_t wave = (int64_t)blockIdx.x * (kThreads / 64) +
                       __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * (kThreads / 64);
  const unsigned short *pt16 = (const unsigned short *)pts;

  // Coefficients of a stage of up to kStageBlocks blocks, in LDS: block b, output
  // column row r at KP 2-byte words each, its 16-byte chunks XOR-swizzled so
  // that the rows one pass of a 16-byte read touches fall in distinct banks;
  // zeros past n.  Binary16 coefficients are stored split (hi, then lo).
  __shared__ __attribute__((aligned(16))) unsigned char stage[kStage];
  constexpr int kBlockBytes = 2 * kBlock;
  constexpr int kStageBlocks = kStage / kBlockBytes / (kF16 ? 2 : 1);
  constexpr int kLo = kStageBlocks * kBlockBytes;
  auto chunk_at = [&](int row, int c) {   // row of a block, chunk c of its KP / 8
    return row * (2 * KP) + 16 * (c ^ ((row >> 2) & (KP / 8 - 1)));
  };
  auto fill_stage = [&](int64_t J0, int count) {   // blocks J0 .. J0 + count - 1
    for (int i = threadIdx.x; i < count * (kBlock / 8); i += kThreads) {
      const int64_t at = J0 * kBlock + 8 * (int64_t)i;
      const int64_t left = n - at;
      const unsigned char *src = coef + 2 * at;
      u32x4 v = left >= 8 ? *(const u32x4 *)src
                          : load_chunk<2>(src, left > 0 ? (int)left : 0);
      const int blk = i / (kBlock / 8), in = i % (kBlock / 8);
      unsigned char *dst = stage + blk * kBlockBytes + chunk_at(in / (KP / 8), in % (KP / 8));
      if constexpr (kF16) {
        u32x4 lo;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          unsigned h, l;
          f16_pair_to_bf16(v[c], h, l, sc);
          v[c] = h;
          lo[c] = l;
        }
        *(u32x4 *)(dst + kLo) = lo;
      }
      *(u32x4 *)dst = v;
    }
  };
  // Step q of this lane's row of block `blk` of the stage (offset kLo: the
  // low words).
  auto weights = [&](int blk, int q, int lo) {
    return *(const u32x4 *)(stage + blk * kBlockBytes + lo + chunk_at(r, 2 * q + g));
  };
  // Polynomials of one stage fill it once; longer ones once per stage and pass.
  const bool one_stage = nblocks <= kStageBlocks;
  if (one_stage) {
    fill_stage(0, (int)nblocks);
    __syncthreads();
  }

  // (every wave of a workgroup takes as many passes, for the barriers)
  const int64_t wg0 = (int64_t)blockIdx.x * (kThreads / 64) * U;
  for (int64_t w0 = wg0; w0 < nchunks; w0 += nwaves * U) {
    const int64_t t0 = w0 + (wave - (int64_t)blockIdx.x * (kThreads / 64)) * U;
    u32x4 xh[U][kQ], xl[U][kQ];
    float yv[U], y8v[U], yg[U], acc[U], ystep[U];
    // All U points first, so their loads are in flight together; points
    // past np read as zero bits (+0 in both formats), and a pass whose
    // points all exist takes no range test.
    const int64_t p0 = t0 * 32;
    const bool whole = p0 + 32 * U <= np;   // every point of the pass exists
    const unsigned short *pp = pt16 + p0;
    unsigned short praw[U];
    if (whole) {
#pragma unroll
      for (int u = 0; u < U; ++u) praw[u] = pp[32 * u + r];
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t idx = p0 + 32 * u + r;
        praw[u] = idx < np ? pt16[idx] : (unsigned short)0;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float x = in_to_f32<DT>(praw[u]);
      // Power ladder (same products in both lanes of a point): x^2 .. x^16,
      // y = x^KP.
      const float x2 = x * x, x4 = x2 * x2, x8 = x4 * x4, x16 = x8 * x8;
      // X fragment: x^(16 q + 8 g + e), e < 8, as hi + lo words.
      float pw[8];
      pw[0] = g ? x8 : 1.f;
#pragma unroll
      for (int e = 1; e < 8; ++e) pw[e] = pw[e - 1] * x;
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        float pq[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (q > 0) pw[e] *= x16;
          pq[e] = n < KP && 16 * q + 8 * g + e >= n ? 0.f : pw[e];   // past the degree: unused
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          unsigned hi, lo;
          split_bf16x2(pq[2 * c], pq[2 * c + 1], hi, lo, sc);
          xh[u][q][c] = hi;
          xl[u][q][c] = lo;
        }
      }
      // The combine: column c = 8a + 4g + i of a block has weight
      // y^c = y^(4g) y^(8a) y^i, y = x^KP; a lane forms its columns' sum by
      // Horner's rule in y (and y^8 across the groups of four), the blocks
      // by Horner's rule in y^32, and applies y^(4g) once at the end.  A
      // power that only multiplies unused (zero) columns is replaced by 0,
      // so that it cannot overflow where the polynomial does not: every
      // power kept divides x^(n-1).
      const float x32 = x16 * x16;
      const float y = KP == 32 ? x32 : x16;
      const float y2 = y * y, y4 = y2 * y2, y8 = y4 * y4, y16 = y8 * y8;
      yv[u] = ncols >= 2 ? y : 0.f;
      y8v[u] = ncols > 8 ? y8 : 0.f;
      yg[u] = g == 0 ? 1.f : ncols > 4 ? y4 : 0.f;
      ystep[u] = nblocks >= 2 ? y16 * y16 : 0.f;
      acc[u] = 0.f;
    }

    // Chunk u's products of a block are issued around the combine of the
    // chunk before it (of the previous block for u = 0): vector work between a
    // wave's own matrix-core instructions runs under them.
    auto products = [&](int u, const u32x4 (&wf)[kQ], const u32x4 (&wl)[kQ])
        __attribute__((always_inline)) {
      f32x16 d;
#pragma unroll
      for (int i = 0; i < 16; ++i) d[i] = 0.f;
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        d = mfma32_k16(UDT, wf[q], xh[u][q], d);
        d = mfma32_k16(UDT, wf[q], xl[u][q], d);
        if constexpr (kF16) {
          d = mfma32_k16(UDT, wl[q], xh[u][q], d);
          d = mfma32_k16(UDT, wl[q], xl[u][q], d);
        }
      }
      return d;
    };
    auto combine = [&](int u, const f32x16 &d) __attribute__((always_inline)) {
      float t = 0.f;
#pragma unroll
      for (int a = 3; a >= 0; --a) {
        const float ta = __builtin_fmaf(
            __builtin_fmaf(__builtin_fmaf(d[4 * a + 3], yv[u], d[4 * a + 2]), yv[u], d[4 * a + 1]),
            yv[u], d[4 * a]);
        t = a == 3 ? ta : __builtin_fmaf(t, y8v[u], ta);
      }
      acc[u] = __builtin_fmaf(acc[u], ystep[u], t);
    };
    // The pass's first products are issued alone; the others around the
    // combine of the chunk before them.
    f32x16 prev;
    bool first = true;
    for (int64_t J1 = nblocks; J1 > 0;) {   // stages of blocks [J0, J1), last first
      const int64_t J0 = (J1 - 1) / kStageBlocks * kStageBlocks;
      if (!one_stage) {
        __syncthreads();   // the last stage has been read
        fill_stage(J0, (int)(J1 - J0));
        __syncthreads();
      }
      int blk = (int)(J1 - J0) - 1;
      u32x4 wf[kQ], wl[kQ];
      auto read_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          wf[q] = weights(blk, q, 0);
          if constexpr (kF16) wl[q] = weights(blk, q, kLo);
        }
      };
      if (first) {
        read_weights();
        prev = products(0, wf, wl);
#pragma unroll
        for (int u = 1; u < U; ++u) {
          const f32x16 d = products(u, wf, wl);
          combine(u - 1, prev);
          prev = d;
        }
        first = false;
        --blk;
      }
      for (; blk >= 0; --blk) {
        read_weights();
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const f32x16 d = products(u, wf, wl);
          combine(u == 0 ? U - 1 : u - 1, prev);
          prev = d;
        }
      }
      J1 = J0;
    }
    if (nblocks > 0) combine(U - 1, prev);

#pragma unroll
    for (int u = 0; u < U; ++u) {
      float v = acc[u] * yg[u];
      v += __shfl_xor(v, 32);
      if (g == 0 && (whole || p0 + 32 * u + r < np)) {
        if constexpr (DT == TCU_BF16_BF16)
          ((unsigned short *)out + p0)[32 * u + r] =
              (unsigned short)(pack_bf16x2(v, 0.f) & 0xffffu);
        else
          ((float *)out + p0)[32 * u + r] = v;
      }
    }
  }
}

template <int DT, int KP, int U, int kThreads, int kStage>
hipError_t launch_poly_cfg(const void *coef, int64_t n, const void *pts, int64_t np, void *out,
                           hipStream_t stream, int num_cus) {
  const int64_t nchunks = (np + 31) / 32;
  const int64_t nblocks = (n + kPolyCols * KP - 1) / (kPolyCols * KP);
  const int64_t per_wg = (int64_t)(kThreads / 64) * U;
  const int64_t want = (nchunks + per_wg - 1) / per_wg;
  const int64_t cap = (int64_t)num_cus * (1024 / kThreads);   // 16 waves per CU
  const int blocks = (int)(want < cap ? want : cap);
  hipLaunchKernelGGL((poly_kernel<DT, KP, U, kThreads, kStage>), dim3(blocks), dim3(kThreads), 0,
                     stream, (const unsigned char *)coef, n, (const unsigned char *)pts, np,
                     (unsigned char *)out, nchunks, nblocks);
  return hipGetLastError();
}

// The shape by size (us for 2^24 points, n = 100 and 1000; 2^22, n = 65536; bf16):
//   * powers per column: with s = 32 and more than 1024 coefficients 32, which
//     halves the combine (n = 4096, 2^24 points: 336 / 275; 64 powers: 315); up to
//     1024 the powers and their split are most of the work and 16 are faster (KP = 16:
//     89, 127; KP = 32: 128, 136).  With s = 16 always 16, the s of the method: its
//     columns hold fewer powers that the split rounds (x^0 to x^2 are exact in
//     bfloat16 hi + lo), and 32 raised the error's norm by 6 to 22 % (n = 1025 to 20000).
//     The price of 16 at s = 16 (us, 16 / 32): n = 20000, 30000 points 8.9 / 6.9; n = 65536,
//     131072 points 35.4 / 30.7; n = 2^20, 1000 points, a long chain per wave, 331 / 207;
//   * coefficients beyond a 32 KiB stage: one workgroup of 16 waves around
//     128 KiB, so that up to 2^16 bfloat16 coefficients are loaded once (n = 65536:
//     858 with the small stage refilled on every pass);
//   * too few points to give every SIMD a wave of two chunks: one chunk per
//     wave (n = 65536, 1000 points: 20.9 -> 15.7).
template <int DT, int KP>
hipError_t launch_poly_kp(const void *coef, int64_t n, const void *pts, int64_t np, void *out,
                          hipStream_t stream, int num_cus) {
  constexpr int kSmall = 32768, kBig = 131072;
  const int64_t waves = (np + 63) / 64;   // with two chunks each
  if (waves < 4 * (int64_t)num_cus)
    return launch_poly_cfg<DT, KP, 1, 256, kSmall>(coef, n, pts, np, out, stream, num_cus);
  const int64_t bytes = n * (DT == TCU_F16_F32 ? 4 : 2);   // binary16 is stored split
  if (bytes > kSmall && waves >= 16 * (int64_t)num_cus)
    return launch_poly_cfg<DT, KP, 2, 1024, kBig>(coef, n, pts, np, out, stream, num_cus);
  return launch_poly_cfg<DT, KP, 2, 256, kSmall>(coef, n, pts, np, out, stream, num_cus);
}
template <int DT>
hipError_t launch_poly_dt(int s, const void *coef, int64_t n, const void *pts, int64_t np,
                          void *out, hipStream_t stream, int num_cus) {
  if (s == 16 || n <= 1024)
    return launch_poly_kp<DT, 16>(coef, n, pts, np, out, stream, num_cus);
  return launch_poly_kp<DT, 32>(coef, n, pts, np, out, stream, num_cus);
}

}  // namespace

hipError_t launch_poly(int dtype, int s, const void *coef, int64_t n, const void *pts, int64_t np,
                       void *out, hipStream_t stream, int num_cus) {
  switch (dtype) {
    case TCU_F16_F32: return launch_poly_dt<TCU_F16_F32>(s, coef, n, pts, np, out, stream, num_cus);
    case TCU_BF16_F32:
      return launch_poly_dt<TCU_BF16_F32>(s, coef, n, pts, np, out, stream, num_cus);
    case TCU_BF16_BF16:
      return launch_poly_dt<TCU_BF16_BF16>(s, coef, n, pts, np, out, stream, num_cus);
  }
  return hipErrorInvalidValue;
}

}  // namespace tcu

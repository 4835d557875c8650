// Transitive closure of a directed graph (Section 4.3, Theorem 5), in place
// on its n x n 0/1 adjacency matrix X (int8, row pitch ld).
//
// The section's blocked algorithm walks the pivot blocks k in order and, for
// each, closes the diagonal block (function A), updates the pivot block row
// (B) and block column (C) through it, and updates every other block with
// X_ij <- min(X_ij + X_ik X_kj, 1) (function D) -- an OR of ANDs.
//
// Here the pivot band is 256 vertices and X is held as bits while the bands
// are walked: the bytes of row i are packed into its first n/8 bytes, and
// unpacked at the end, so no other memory is needed and a pass over X moves
// an eighth of the bytes.  With D* the closed diagonal block, B, C and D of
// a band are one formula for every row i of the matrix,
//   R_i = X[i, band] (I + D*),   X[i, :] |= R_i X[band, :],
// R_i being the band's vertices that i reaches through the band.  Both
// products are taken four pivots at a time from LDS tables of all 16 unions
// of four consecutive rows: 64 16-byte lookups per 128 columns and row
// instead of 256 masked terms.  One launch per band:
//   * a workgroup takes a slab of 1024 columns (its tables: 64 groups x 16
//     unions x 128 bytes) and a range of rows, eight lanes per row;
//   * workgroup 0 instead updates the next band's diagonal block and closes
//     it (tcu_tc_diag.h), beside the others' work.
// The rows are updated in place while other workgroups read them as
// operands.  Every value only grows (0 -> 1) and stays between its value
// before the band and the closure, and with D* final any mix of old and new
// values of the operands gives the same product; a word is written by one
// workgroup only (the diagonal block's by workgroup 0).
//
// At n = 8192 a band's launch takes 11 us while few rows reach its pivots
// (rows whose band words are zero are skipped): the chain of the next
// diagonal block's update and closure.  Once the closure has filled in it
// takes 16 us: launch and tables about 6, and 272 rows of 64 lookups of
// 16 bytes per lane against the LDS's 128 bytes per clock and CU.  On int8
// matrix cores over the bytes of X the same band took 31 us (panel loads and
// fragment reads of eight times the bytes) after 7 us for its column panel:
// 1.28 ms for the whole closure, 0.515 ms here (deg 2).
#include "tcu_device.h"
#include "tcu_launch.h"
#include "tcu_tc_diag.h"

namespace tcu {
namespace {

constexpr int kBand = kDiagBand;     // pivot band width (vertices)
constexpr int kThreads = kDiagThreads;
constexpr int kSlabQuads = 8;        // 16-byte quads of 128 columns per slab row
constexpr int kGroups = kBand / 4;   // groups of four pivots
constexpr int kStepRows = kThreads / kSlabQuads;   // rows a workgroup takes at once

// Every nonzero byte -> 1.
__device__ __forceinline__ unsigned nonzero_bytes(unsigned x) {
  unsigned t = x | (x >> 4);   // low nibble of each byte: OR of its halves
  t |= t >> 2;                 // bits 0, 1: OR of the byte's bit pairs
  t |= t >> 1;                 // bit 0: OR of all 8 bits of the byte
  return t & 0x01010101u;
}
// Nonzero bytes of a 16-byte chunk -> 16 bits (the products put bit 0 of
// byte i at bit 28 + i without carries), and 4 bits -> 4 bytes of 0/1.
__device__ __forceinline__ unsigned chunk_bits(u32x4 v) {
  unsigned b = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) b |= ((nonzero_bytes(v[c]) * 0x10204080u) >> 28) << (4 * c);
  return b;
}
__device__ __forceinline__ unsigned bits4_to_bytes(unsigned b) {
  return ((b & 15u) * 0x00204081u) & 0x01010101u;
}

// Bytes [c, c + 16) of a row of n bytes (any address), zeros past n; nothing
// past it is read.
__device__ __forceinline__ u32x4 row_chunk(const unsigned char *row, int64_t c, int64_t n) {
  if (c + 16 <= n) return load16_any(row + c);
  if (c >= n) return u32x4{0u, 0u, 0u, 0u};
  if (n < 16) return load_chunk<1>(row + c, (int)(n - c));
  return shift_down(load16_any(row + n - 16), (int)(c - (n - 16)));
}
// Word w of a row: the edges to vertices 32 w .. 32 w + 31.
__device__ __forceinline__ unsigned row_word(const unsigned char *row, int64_t w, int64_t n) {
  return chunk_bits(row_chunk(row, 32 * w, n)) | (chunk_bits(row_chunk(row, 32 * w + 16, n)) << 16);
}
// Its bytes back, clipped to n.
__device__ __forceinline__ void store_row_word(unsigned char *row, int64_t w, int64_t n,
                                               unsigned word) {
  unsigned char *p = row + 32 * w;
  if (32 * w + 32 <= n) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 v;
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = bits4_to_bytes(word >> (16 * h + 4 * c));
      store16_any(p + 16 * h, v);
    }
  } else {
    for (int b = 0; b < 32 && 32 * w + b < n; ++b) p[b] = (unsigned char)((word >> b) & 1u);
  }
}

// Rows of at most 256 vertices: the whole closure in one workgroup.
__global__ __launch_bounds__(kThreads) void tc_small_kernel(unsigned char *__restrict__ X, int n,
                                                            int64_t ld) {
  __shared__ __attribute__((aligned(16))) DiagShared s;
  const int i = threadIdx.x / 2, w0 = 4 * (threadIdx.x % 2);
  unsigned char *p = X + (int64_t)i * ld;
  unsigned row[4] = {0u, 0u, 0u, 0u};
  if (i < n) {
#pragma unroll
    for (int q = 0; q < 4; ++q) row[q] = row_word(p, w0 + q, n);
  }
  close_diag_rows(row, n, s);
  if (i < n) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (32 * (w0 + q) < n) store_row_word(p, w0 + q, n, row[q]);
  }
}

// Bytes -> bits, in place: word w of row i (w < words, a multiple of 4 with
// 4 words <= n bytes) into bytes [4 w, 4 w + 4) of the row.  A workgroup
// takes whole rows; its words of a pass are stored once every thread has
// read its bytes, and a later pass stores only over bytes of earlier ones.
__global__ __launch_bounds__(256) void tc_pack_kernel(unsigned char *__restrict__ X, int64_t n,
                                                      int64_t ld, int64_t words) {
  for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
    unsigned char *row = X + i * ld;
    for (int64_t w0 = 0; w0 < words; w0 += blockDim.x) {
      const int64_t w = w0 + threadIdx.x;
      const unsigned word = w < words ? row_word(row, w, n) : 0u;
      __syncthreads();
      if (w < words) store4_any(row + 4 * w, word);
    }
  }
}

// Bits -> bytes, in place: passes from the row's end, each read whole before
// its bytes are stored; a pass stores only over words of later ones.
__global__ __launch_bounds__(256) void tc_unpack_kernel(unsigned char *__restrict__ X, int64_t n,
                                                        int64_t ld, int64_t words) {
  for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
    unsigned char *row = X + i * ld;
    for (int64_t w0 = (words - 1) / blockDim.x * blockDim.x; w0 >= 0; w0 -= blockDim.x) {
      const int64_t w = w0 + threadIdx.x;
      const unsigned word = w < words ? load4_any(row + 4 * w) : 0u;
      __syncthreads();
      if (32 * w < n) store_row_word(row, w, n, word);
    }
  }
}

// Close the diagonal block of the first of several bands (packed rows).
__global__ __launch_bounds__(kThreads) void tc_diag_kernel(unsigned char *__restrict__ X,
                                                           int64_t ld) {
  __shared__ __attribute__((aligned(16))) DiagShared s;
  unsigned char *p = X + (int64_t)(threadIdx.x / 2) * ld + 16 * (threadIdx.x % 2);
  const u32x4 v = load16_any(p);
  unsigned row[4] = {v[0], v[1], v[2], v[3]};
  close_diag_rows(row, kBand, s);
  store16_any(p, u32x4{row[0], row[1], row[2], row[3]});
}

constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor3 = 0x1B, kHalfMirror = 0x141;   // DPP controls
// OR over the four lanes of a row's eight that hold the same quad parity
// (lanes l, l ^ 2, l ^ 4, l ^ 6).
__device__ __forceinline__ u32x4 or_parts(u32x4 v) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    unsigned x = v[c];
    x |= dpp<kXor2>(x);
    x |= dpp<kXor3>(dpp<kHalfMirror>(x));   // l -> 7 - l -> l ^ 4
    v[c] = x;
  }
  return v;
}

// The 16-byte quad at LDS byte address addr + offset.
__device__ __forceinline__ u32x4 lds_quad(unsigned addr, int offset) {
  return *(const __attribute__((address_space(3))) u32x4 *)(uintptr_t)(addr + offset);
}

// Tables of all unions of four consecutive rows of a 256-row operand 8 words
// wide: entry m of group g at 128 (16 (g / 4) + m) + 32 (g % 4) bytes, two
// quads.  A row's eight lanes (quad l % 2, groups = l / 2 mod 4) then read
// four distinct 32-byte bank windows whatever their subsets are.
constexpr int kNarrowBytes = kGroups * 16 * 32;
__device__ __forceinline__ int narrow_at(int g, int m) {
  return 128 * (16 * (g >> 2) + m) + 32 * (g & 3);
}
// Thread t builds subsets 4 (t % 4) .. + 3 of group t / 8, quad (t / 4) % 2;
// rows come from `get(row, quad)`.
template <typename Get>
__device__ __forceinline__ void build_narrow(unsigned char *tab, Get get) {
  const int t = threadIdx.x, g = t >> 3, q = (t >> 2) & 1, hi = t & 3;
  u32x4 v[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) v[b] = get(4 * g + b, q);
  u32x4 base = {0u, 0u, 0u, 0u};
  if (hi & 1) base |= v[2];
  if (hi & 2) base |= v[3];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    u32x4 e = base;
    if (m & 1) e |= v[0];
    if (m & 2) e |= v[1];
    *(u32x4 *)(tab + narrow_at(g, 4 * hi + m) + 16 * q) = e;
  }
}
// Union over the pivots in the 256-bit set (lo, hi quads, the same in the
// row's eight lanes) of the operand's rows: this lane's quad l % 2.
__device__ __forceinline__ u32x4 union_narrow(const unsigned char *tab, u32x4 lo, u32x4 hi, int l) {
  const int q = l & 1, part = l >> 1;
  const unsigned char *base = tab + 32 * part + 16 * q;
  u32x4 r = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const unsigned word = (w < 4 ? lo[w & 3] : hi[w & 3]) >> (4 * part);
#pragma unroll
    for (int h = 0; h < 2; ++h)     // groups 8 w + 4 h + part
      r |= *(const u32x4 *)(base + 128 * (16 * (2 * w + h) + ((word >> (16 * h)) & 15u)));
  }
  return or_parts(r);
}

// One band: rows [0, n) of the packed matrix, pivots [k0, k0 + Bk).  Blocks
// after the first (or all, with next = 0) take column slab s and rows
// [share j, share (j + 1)), s + slabs j the block's index; block 0
// with next > 0 updates and closes the diagonal block of the next band,
// which is `next` vertices wide.  quads: 16-byte quads per packed row.
__global__ __launch_bounds__(kThreads) void tc_band_kernel(unsigned char *__restrict__ X,
                                                           int64_t ld, int64_t n, int64_t k0,
                                                           int Bk, int64_t quads, int slabs,
                                                           int64_t share, int next) {
  // tables of the slab, then of D* (narrow); block 0 keeps the next block's
  // narrow tables, its rows and the closure's data in the slab's place
  constexpr int kWideBytes = kGroups * 16 * 128;
  // (a group's 16 unions start at a multiple of 2048 bytes: their index is
  // or-ed into the address)
  __shared__ __attribute__((aligned(2048))) unsigned char smem[kWideBytes + kNarrowBytes];
  unsigned char *const tabX = smem, *const tabD = smem + kWideBytes;
  static_assert(kNarrowBytes + 256 * 32 + sizeof(DiagShared) <= kWideBytes, "block 0's LDS");

  const int lane8 = threadIdx.x & 7, row8 = threadIdx.x >> 3;
  const int64_t kq = k0 / 128;                 // the band's first quad
  const u32x4 zero = {0u, 0u, 0u, 0u};
  const unsigned char *const band = X + k0 * ld;
  auto band_quad = [&](int r, int64_t q) {
    return r < Bk && q < quads ? load16_any(band + r * ld + 16 * q) : zero;
  };
  const bool diag = next > 0 && blockIdx.x == 0;
  const int64_t k1 = k0 + kBand;               // the next band
  const int64_t nq = k1 / 128;                 // its first quad

  // this block's rows and quad, and the first rows' operands
  const int64_t unit = (int64_t)blockIdx.x - (next > 0 ? 1 : 0);
  const int64_t quad = diag ? nq + (lane8 & 1) : (unit % slabs) * kSlabQuads + lane8;
  const int64_t first = diag ? k1 : unit / slabs * share;
  const int64_t last = diag ? k1 + next : (first + share < n ? first + share : n);
  auto load_row = [&](int64_t i, u32x4 &lo, u32x4 &hi, u32x4 &old) {
    lo = hi = old = zero;
    if (i < last) {
      const unsigned char *p = X + i * ld;
      lo = load16_any(p + 16 * kq);
      if (kq + 1 < quads) hi = load16_any(p + 16 * (kq + 1));
      if (quad < quads) old = load16_any(p + 16 * quad);
    }
  };
  u32x4 lo, hi, old;
  load_row(first + row8, lo, hi, old);

  build_narrow(tabD, [&](int r, int q) { return band_quad(r, kq + q); });
  if (diag) {
    build_narrow(tabX, [&](int r, int q) { return band_quad(r, nq + q); });
  } else {
    // group t / 8, quad t % 8: all 16 unions of the group's four rows
    const int g = threadIdx.x >> 3;
    u32x4 v[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) v[b] = band_quad(4 * g + b, quad);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      u32x4 e = zero;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (m & (1 << b)) e |= v[b];
      *(u32x4 *)(tabX + 128 * (16 * g + m) + 16 * lane8) = e;
    }
  }
  __syncthreads();
  // LDS addresses of the wide tables' halves for this lane's quad
  unsigned wide0 = lds_addr(tabX) + 16 * lane8, wide1 = lds_addr(tabX) + kWideBytes / 2 + 16 * lane8;
  asm("" : "+v"(wide1));   // (kept apart: 65536 is past the offset's range)

  for (int64_t i0 = first; i0 < last; i0 += kStepRows) {
    const int64_t i = i0 + row8;
    u32x4 nlo, nhi, nold;
    if (i0 + kStepRows < last) load_row(i + kStepRows, nlo, nhi, nold);
    u32x4 now = old;
    // (the band's quads past its last vertex hold zeros)
    if (__any((lo[0] | lo[1] | lo[2] | lo[3] | hi[0] | hi[1] | hi[2] | hi[3]) != 0u)) {
      // R_i: this lane's quad from the tables of D*, the other from its
      // neighbour
      const u32x4 own = union_narrow(tabD, lo, hi, lane8);
      u32x4 other;
#pragma unroll
      for (int c = 0; c < 4; ++c) other[c] = dpp<kXor1>(own[c]);
      const bool odd = lane8 & 1;
      const u32x4 rlo = (odd ? other : own) | lo, rhi = (odd ? own : other) | hi;
      if (diag) {
        now |= union_narrow(tabX, rlo, rhi, lane8);
      } else {
        // Two bases, so that every table lies within the instruction's
        // 16-bit offset of one of them; a half whose pivots no row of the
        // wave reaches is skipped.
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const u32x4 set = half ? rhi : rlo;
          if (!__any((set[0] | set[1] | set[2] | set[3]) != 0u)) continue;
          const unsigned at = half ? wide1 : wide0;
#pragma unroll
          for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int g = 0; g < 8; ++g) {
              const unsigned m = g < 2 ? set[w] << (7 - 4 * g) : set[w] >> (4 * g - 7);
              now |= lds_quad((m & 0x780u) | at, 2048 * (8 * w + g));
            }
        }
      }
    }
    if (diag) {
      // the block's rows, for its closure (two quads per row)
      if (lane8 < 2)
        *(u32x4 *)(tabX + kNarrowBytes + 32 * (i - k1) + 16 * lane8) = i < last ? now : zero;
    } else if (i < last && quad < quads) {
      const bool next_block = next > 0 && i >= k1 && i < k1 + next && quad >= nq && quad < nq + 2;
      const u32x4 d = now ^ old;
      if (!next_block && (d[0] | d[1] | d[2] | d[3]) != 0u) store16_any(X + i * ld + 16 * quad, now);
    }
    lo = nlo;
    hi = nhi;
    old = nold;
  }
  if (diag) {
    const unsigned char *rows = tabX + kNarrowBytes;
    DiagShared &s = *reinterpret_cast<DiagShared *>(tabX + kNarrowBytes + 256 * 32);
    __syncthreads();
    const int i = threadIdx.x / 2, q = threadIdx.x % 2;
    const u32x4 v = i < next ? *(const u32x4 *)(rows + 32 * i + 16 * q) : zero;
    unsigned row[4] = {v[0], v[1], v[2], v[3]};
    close_diag_rows(row, next, s);
    if (i < next && nq + q < quads)
      store16_any(X + (k1 + i) * ld + 16 * (nq + q), u32x4{row[0], row[1], row[2], row[3]});
  }
}

}  // namespace

hipError_t launch_tc(unsigned char *X, int64_t ld, int64_t n, hipStream_t stream, int num_cus) {
  if (n <= 0) return hipSuccess;
  if (n <= kBand) {
    hipLaunchKernelGGL(tc_small_kernel, dim3(1), dim3(kThreads), 0, stream, X, (int)n, ld);
    return hipGetLastError();
  }
  const int64_t quads = (n + 127) / 128, words = 4 * quads;
  const unsigned pack_threads = words <= 64 ? 64 : words <= 128 ? 128 : 256;
  const int64_t pack_cap = (int64_t)num_cus * 8 * (256 / pack_threads);
  const unsigned pack_grid = (unsigned)(n < pack_cap ? n : pack_cap);
  hipLaunchKernelGGL(tc_pack_kernel, dim3(pack_grid), dim3(pack_threads), 0, stream, X, n, ld,
                     words);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // From here on X holds bits: whatever fails, it is unpacked before the call
  // returns (each step leaves a graph between the one given and its closure).
  hipLaunchKernelGGL(tc_diag_kernel, dim3(1), dim3(kThreads), 0, stream, X, ld);
  e = hipGetLastError();
  // A workgroup per CU (its tables fill the LDS), one of them for the next
  // diagonal block: the others share the slabs' rows evenly, a wave's eight
  // at a time (n = 8192: 31 ranges of 272 rows; whole steps of 64 made them
  // 26 of 320).  The test override TCU_KNOB_PP_GRID stands for the number of CUs.
  const int64_t cus = knob(TCU_KNOB_PP_GRID) > 0 ? knob(TCU_KNOB_PP_GRID) : num_cus;
  const int64_t slabs = (quads + kSlabQuads - 1) / kSlabQuads;
  int64_t ranges = cus > slabs ? (cus - 1) / slabs : 1;   // per slab
  if (ranges > (n + kStepRows - 1) / kStepRows) ranges = (n + kStepRows - 1) / kStepRows;
  const int64_t share = ((n + ranges - 1) / ranges + 7) / 8 * 8;
  ranges = (n + share - 1) / share;
  for (int64_t k0 = 0; k0 < n && e == hipSuccess; k0 += kBand) {
    const int64_t left = n - k0 - kBand;
    const int Bk = (int)(left < 0 ? left + kBand : kBand);
    const int next = (int)(left <= 0 ? 0 : left < kBand ? left : kBand);
    hipLaunchKernelGGL(tc_band_kernel, dim3((unsigned)(slabs * ranges + (next > 0 ? 1 : 0))),
                       dim3(kThreads), 0, stream, X, ld, n, k0, Bk, quads, (int)slabs, share, next);
    e = hipGetLastError();
  }
  hipLaunchKernelGGL(tc_unpack_kernel, dim3(pack_grid), dim3(pack_threads), 0, stream, X, n, ld,
                     words);
  const hipError_t unpacked = hipGetLastError();
  return e != hipSuccess ? e : unpacked;
}

}  // namespace tcu

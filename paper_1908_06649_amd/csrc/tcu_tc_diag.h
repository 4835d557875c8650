// Closure of a diagonal block of the transitive closure (Section 4.3,
// function A on a 256-vertex pivot band), as a workgroup-wide device function
// on rows of bits held in registers.
#pragma once

#include "tcu_device.h"

namespace tcu {

constexpr int kDiagBand = 256;                  // vertices per pivot band
constexpr int kDiagWords = kDiagBand / 32;      // 32-bit words per row
constexpr int kDiagThreads = 512;               // two threads per row

template <int kCtrl>
__device__ __forceinline__ unsigned dpp(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, false);
}

// LDS of one diagonal closure: two sets, for sub-bands of even and odd index.
struct DiagShared {
  u32x4 krow[2][32][2];             // the sub-band's published pivot rows
  unsigned tab1[2][8 * 16];         // [group][subset] over T*
  u32x4 tab2[2][8 * 16 * 2];        // over the published rows, see tab2_at
};
// Quad q of entry m of group g, as a u32x4 index: entry m of groups 4 j ..
// 4 j + 3 share a 128-byte window, 32 bytes each.
__device__ __forceinline__ int tab2_at(int g, int m, int q) {
  return 8 * (16 * (g >> 2) + m) + 2 * (g & 3) + q;
}

// Close the Bk x Bk block, Bk <= 256, whose rows the workgroup's 512 threads
// (every one must call it: it synchronises the workgroup) hold as bits: row i
// is 8 words (bit b of word w = column 32 w + b; zero past Bk, as are the rows
// past Bk), words 0-3 in thread 2 i and 4-7 in thread 2 i + 1.  The pivots are
// taken in sub-bands K of 32, the rows of wave K; for each:
//   * the pivots' current rows are published to LDS;
//   * wave K closes the 32 x 32 block of K's rows and columns (the iterative
//     algorithm on 32 one-word rows, the pivot row broadcast with readlane),
//     giving T*[k]: the pivots reachable from pivot k through K, k included;
//   * every row i (pivot or not) forms R_i, the union of T*[k] over the
//     pivots k it has an edge to, and ORs in the published rows of R_i.
// That is the iterative algorithm's 32 steps over K: a vertex reaches v
// through K exactly when some pivot it reaches through K has an edge to v.
// Both unions over a 32-bit set are taken 4 bits at a time from tables of
// all 16 unions of 4 consecutive pivots' words (8 lookups instead of 32
// masked terms): tab1 over T*, built by wave K, and tab2 over the published
// rows, built by the others meanwhile.  The eight lanes of one pass of a
// 16-byte lookup are four rows; row p of them takes groups p, p + 1, .. (mod
// 4), so that the four read distinct bank windows whatever their subsets.
// The sub-bands alternate between two sets of tables: two barriers each.  The
// chain of eight sub-bands sets the time: 8.5 us with tables of single words
// (32 lookups per thread), three barriers and wave 0 closing every block.
__device__ __forceinline__ void close_diag_rows(unsigned (&row)[4], int Bk, DiagShared &s) {
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int q = t & 1, p = (t >> 1) & 3;        // this thread's quad; its row mod 4
#pragma unroll
  for (int sb = 0; sb < kDiagWords; ++sb) {
    if (32 * sb >= Bk) break;
    const int buf = sb & 1;
    if (wave == sb) s.krow[buf][lane >> 1][q] = u32x4{row[0], row[1], row[2], row[3]};
    __syncthreads();
    // word sb of this thread's row, in both its lanes (quad permutations
    // [0, 0, 2, 2] and [1, 1, 3, 3])
    const unsigned edges = sb < 4 ? dpp<0xa0>(row[sb & 3]) : dpp<0xf5>(row[sb & 3]);
    if (wave == sb) {
      unsigned tk = edges;
#pragma unroll
      for (int kk = 0; kk < 32; ++kk) {
        const unsigned pivot = (unsigned)__builtin_amdgcn_readlane((int)tk, 2 * kk);
        tk |= pivot & (0u - ((tk >> kk) & 1u));
      }
      tk |= 1u << (lane >> 1);
      // tab1: lanes 8 g .. 8 g + 7 hold pivots 4 g .. 4 g + 3 twice; lane
      // 8 g + l builds subsets 2 l and 2 l + 1.
      const unsigned mine0 = dpp<0x00>(tk), mine1 = dpp<0xaa>(tk);   // its quad's two pivots
      const unsigned far0 = dpp<0x141>(mine0), far1 = dpp<0x141>(mine1);   // the other quad's
      const bool upper = lane & 4;
      const unsigned v0 = upper ? far0 : mine0, v1 = upper ? far1 : mine1;
      const unsigned v2 = upper ? mine0 : far0, v3 = upper ? mine1 : far1;
      unsigned e = 0;                                  // subset 2 (lane % 8)
      if (lane & 1) e |= v1;
      if (lane & 2) e |= v2;
      if (lane & 4) e |= v3;
      unsigned *t1 = s.tab1[buf] + 2 * lane;
      t1[0] = e;
      t1[1] = e | v0;
    } else {
      // tab2: 256 quads (subset m of group g, quad q) by the seven others
      const int idx = 64 * (wave < sb ? wave : wave - 1) + lane;
      if (idx < 256) {
        const int g = idx >> 5, m = (idx >> 1) & 15, qq = idx & 1;
        u32x4 e = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const u32x4 v = s.krow[buf][4 * g + b][qq];
          const unsigned mask = 0u - ((unsigned)(m >> b) & 1u);
#pragma unroll
          for (int c = 0; c < 4; ++c) e[c] |= v[c] & mask;
        }
        s.tab2[buf][tab2_at(g, m, qq)] = e;
      }
    }
    __syncthreads();
    if (__any(edges != 0u)) {
      unsigned reach = 0;
#pragma unroll
      for (int g = 0; g < 8; ++g) reach |= s.tab1[buf][16 * g + ((edges >> (4 * g)) & 15u)];
      u32x4 add = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int w = (j + p) & 3;                     // groups w and 4 + w
        const unsigned bits = reach >> (4 * w);
        add |= s.tab2[buf][tab2_at(w, (int)(bits & 15u), q)];
        add |= s.tab2[buf][tab2_at(4 + w, (int)((bits >> 16) & 15u), q)];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) row[c] |= add[c];
    }
  }
}

}  // namespace tcu

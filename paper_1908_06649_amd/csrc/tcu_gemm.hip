// Blocked dense multiplication of Theorem 2 (Section 4.1), fused into one
// launch: C (N x N) = A (N x N) * B (N x N) with unit size s.
//
// Theorem 2 cuts A into N x s vertical strips A_i and B into s x s blocks
// B_{i,j}, issues the (N/s)^2 tensor-unit calls C_{i,j} = A_i * B_{i,j} and
// sums output strip j over i.  Issued literally, every call would re-stream
// its N x s strip from memory, giving about s/2 flops per byte -- far below
// what the matrix cores need.  Here each workgroup owns one BM x BN output
// tile and walks the contracted index: for every strip i it performs the
// calls A_i[rows of the tile] * B_{i,j} for all column blocks j of the tile,
// accumulating sum_i in registers.  So every one of the (N/s)^2 calls is
// executed (restricted to the tile's rows, across the grid), no partial
// product C_{i,j} is ever written, and each staged slab of A_i is reused
// across all the tile's B_{i,j}.
//
// Compute: 16 x 16 accumulator blocks fed by 16x16x32 (16-bit) or 16x16x64
// (int8) matrix-core instructions from LDS.  The product is formed as
// C^T = B^T A^T, the s x s blocks B_{i,j} being the matrix core's resident row
// operand, so each lane holds 4 consecutive columns of one row of C, stored
// as one 16-byte write.
// Workgroup order is XCD-aware (see map_tile).
#include <climits>

#include "tcu_device.h"
#include "tcu_launch.h"

namespace tcu {
namespace {

// Tile rows per group of the tile order (map_tile) and LDS ring depth of
// the full-tile kernel, both measured best on the order-8192 products.
constexpr int kGroupM = 2;
constexpr int kRingStages = 5;

// Map a workgroup id to an output tile (tm, tn): groups of kGroupM tile
// rows are walked column by column.  Consecutive workgroup ids are dispatched
// round-robin over the 8 XCDs, so with groups of 2 rows each XCD's concurrent
// workgroups cover a compact block of tiles (shared A row-panels and B
// column-panels in its L2) while all XCDs together sweep a band of full rows
// (B panels shared through the memory-side cache).  Measured best for N=8192
// against larger groups and an explicit per-XCD remap of the ids.
template <int kRows = kGroupM>
__device__ __forceinline__ void map_tile(int pid, int tiles_m, int tiles_n, int &tm, int &tn) {
  const int per_group = kRows * tiles_n;
  const int group = pid / per_group;
  const int first_m = group * kRows;
  const int gsz = min(tiles_m - first_m, kRows);
  const int in_group = pid % per_group;
  tm = first_m + in_group % gsz;
  tn = in_group / gsz;
}

// ---------------------------------------------------------------------------
// Full-tile kernel (M, N multiples of 256, K a multiple of one stage):
// 256 x 256 output tiles, a persistent grid of one workgroup per CU walking
// the tiles, and a ring of LDS stages, each holding 64 bytes of the
// contracted index (32 16-bit or 64 int8 values: one matrix-core K step, and
// one or two strips A_i of the unit).
//   * Both operands go HBM/L2 -> LDS with direct 16-byte DMA loads
//     (global_load_lds_dwordx4): no register staging, no VALU work.
//   * A stage of A is 256 rows x 64 bytes, kept as 1 KiB blocks of 16 rows
//     stored chunk-major (the DMA lane -> row/chunk assignment does this for
//     free), so every fragment read is a linear ds_read_b128, the access
//     pattern LDS serves at full rate.
//   * A stage of B is kept row-major as it is in memory (k rows of 256
//     columns); the weights operand (B^T) is formed by transposing LDS
//     reads (ds_read_b64_tr_b16 / _tr_b8), chunks XOR-swizzled per row so
//     the 16 lanes of a read group hit distinct banks.
//   * The DMA is issued through an instruction the compiler cannot see
//     into, so it adds no conservative waits; the kernel orders it with
//     explicit vmcnt waits and fence-free barriers.
// ---------------------------------------------------------------------------
constexpr int kFastKB = 64;                     // bytes of K per stage
constexpr int kFastStage = 256 * kFastKB;       // 16 KiB per operand per stage

// B stage, 16-bit: 512-byte rows (32 chunks).
__device__ __forceinline__ int fb16_swz(int k) { return ((k & 3) << 1) | (((k >> 3) & 3) << 3); }
// B stage, int8: 256-byte rows (16 chunks).
__device__ __forceinline__ int fb8_swz(int k) { return (k & 7) | (((k >> 4) & 1) << 3); }

// ---------------------------------------------------------------------------
// The full-tile kernel runs 8 waves, two per SIMD, in two groups.  Group 0 (waves 0-3) owns rows 0-127 of the 256 x 256 tile, group 1
// (waves 4-7) rows 128-255; wave q of a group owns columns 64q .. 64q+63.
// Each K stage is two phases separated by barriers:
//   phase A(t): group 0 runs its matrix-core work of stage t while group 1
//               reads its fragments of stage t and issues DMA loads;
//   phase B(t): group 1 runs its matrix-core work of stage t while group 0
//               reads its fragments of stage t+1 and issues DMA loads.
// The fragment reads go first: they are the phase's critical path (LDS
// reads of four waves take about as long as the 32 products), and queued
// behind the DMA instructions they started later (measured 1.5 % slower).
// A wave stalled on memory (full load queues, late data) therefore never
// idles its SIMD's matrix core: the other wave on that SIMD is computing,
// with raised issue priority.  Group 0 loads the A part of every stage and
// group 1 the B part (4 DMA instructions per wave per stage).
// Ring bookkeeping: the slot of stage t has been read by group 0 (in
// B(t-1)) and by group 1 (in A(t)) once A(t) ends, so it is refilled with
// stage t+kRing in B(t) (A part, group 0) and A(t+1) (B part, group 1).
// Stage t+1 must be complete when A(t) ends, so every wave waits there for
// its own loads of stage t+1 before the barrier.
// ---------------------------------------------------------------------------
// Wait until at most n of this wave's DMA loads are in flight and all its
// LDS reads have returned, then a workgroup barrier.  The barrier is an
// instruction with a memory clobber: the compiler may not move LDS accesses
// across it (the barrier intrinsic alone does not order memory), while no
// memory fence -- which would drain every in-flight DMA -- is emitted.
template <int n>
__device__ __forceinline__ void vm_wait_barrier() {
  __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (0 << 8) | (((n >> 4) & 3) << 14));
  asm volatile("s_barrier" ::: "memory");
}

// kEdge: C's edge may cut through tiles and K may end inside a stage (the
// ragged shapes); without it every tile and stage is whole.
template <int DT, int kRing, bool kEdge>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2))) void
gemm_pp_kernel(const unsigned char *__restrict__ A, const unsigned char *__restrict__ B,
               unsigned char *__restrict__ C, int K, int64_t lda, int64_t ldb, int64_t ldc,
               int accum, int tiles_m, int tiles_n, int full, int nsplit, int m_lim,
               int n_lim) {
  constexpr bool kI8 = (in_bytes(DT) == 1);
  constexpr int ES = in_bytes(DT);
  constexpr int OB = out_bytes(DT);
  constexpr int KE = kFastKB / ES;     // contracted elements per stage
  constexpr int BROW = 256 * ES;       // bytes per B row in a stage
  constexpr int FM = 8, FN = 4;        // 16 x 16 blocks per wave (128 x 64)
  constexpr int kDma = 4;              // DMA instructions per wave per stage
  static_assert(kRing - 2 <= 3, "waits cover at most 3 later stages");
  typedef typename std::conditional<kI8, i32x4, f32x4>::type Acc;

  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * kRing * kFastStage];
  unsigned char *const sA = smem;
  unsigned char *const sB = smem + kRing * kFastStage;

  // Work items: the first `full` tiles (in map_tile order) whole, then the
  // other tiles as (K slice, tile) pairs, slice-major so that the workgroups
  // running at one time share the K range of their A and B panels.  With
  // nsplit > 1 such an item sums one contiguous range of whole stages
  // (about nk_all / nsplit strips A_i of the unit) and adds its partial
  // tile into C atomically.  full = 0 splits every tile; full = tiles (or
  // nsplit = 1) none.
  const int tiles = tiles_m * tiles_n;
  const int tail_tiles = tiles - full;
  const int total = full + tail_tiles * nsplit;
  // Stages of the contracted index; when K is not a whole number of stages
  // the last one holds k_tail < KE elements and is loaded element-wise with
  // zeros past K (the zero padding of a ragged dimension).
  const int nk_all = kEdge ? (K + KE - 1) / KE : K / KE;
  const int k_tail = K - (nk_all - 1) * KE;
  const int64_t lda_b = lda * ES, ldb_b = ldb * ES, ldc_b = ldc * OB;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wid >> 2, q = wid & 3;
  const int r = lane & 15, g = lane >> 4;
  int item = (int)blockIdx.x;
  int m0, n0, nk;
  int tail_t = -1;   // item-relative index of a partial last stage, if the item holds it
  // This wave's DMA share of a stage: group 0 -> A blocks 4q..4q+3 (16 rows
  // each, stored chunk-major), group 1 -> B blocks 4q..4q+3 (1 KiB each).
  // Wave-uniform 64-bit base + per-lane 32-bit offsets (saddr form).
  const unsigned char *gbase;
  unsigned voff[kDma];
  // Per-lane offsets.  In a tile that crosses the edge of C (rows >= m_lim
  // or columns >= n_lim) a lane past the edge loads the last row of A, or
  // the last 16-byte chunk of B's row, inside it instead: every load stays
  // in the operands, every DMA instruction is issued (the wait counts rely
  // on it), and the products it feeds are never stored.
  auto set_voff = [&]() {
#pragma unroll
    for (int i = 0; i < kDma; ++i) {
      const int blk = q * 4 + i;
      if (grp == 0) {
        int row = blk * 16 + (lane & 15);
        if (kEdge && m0 + row >= m_lim) row = m_lim - 1 - m0;
        voff[i] = (unsigned)(row * lda_b) + 16u * (lane >> 4);
      } else {
        int krow, c;
        if constexpr (!kI8) {
          krow = blk * 2 + (lane >> 5);
          c = (lane & 31) ^ fb16_swz(krow);
        } else {
          krow = blk * 4 + (lane >> 4);
          c = (lane & 15) ^ fb8_swz(krow);
        }
        if constexpr (kEdge) {
          const int c_last = (n_lim - n0) * ES / 16 - 1;
          if (c > c_last) c = c_last;
        }
        voff[i] = (unsigned)(krow * ldb_b) + 16u * c;
      }
    }
  };
  // Split items are few and long, and consecutive workgroup ids go
  // round-robin to the 8 XCDs: their ids are permuted so that each XCD
  // holds a contiguous run of them (one K range, a compact block of tiles),
  // and its concurrent workgroups share their A and B panels in its own L2
  // (measured: 2048 x 65536 x 2048 int8, split 4, 0.261 -> 0.235 ms).  The
  // items past the last multiple of 8 keep their ids.
  const int split_items = nsplit > 1 ? total - full : 0;
  const int xcd_body = split_items - split_items % 8;
  bool split_item = false;   // the current item is a K slice (atomic epilogue)
  auto place = [&](int w) {
    int pid = w, slice = 0;
    split_item = nsplit > 1 && w >= full;
    if (split_item) {
      int v = w - full;
      if (v < xcd_body) v = (v % 8) * (xcd_body / 8) + v / 8;
      slice = v / tail_tiles;
      pid = full + (v - slice * tail_tiles);
    }
    int tm, tn;
    map_tile(pid, tiles_m, tiles_n, tm, tn);
    m0 = tm * 256;
    n0 = tn * 256;
    const int s_begin = split_item ? (int)((int64_t)nk_all * slice / nsplit) : 0;
    nk = split_item ? (int)((int64_t)nk_all * (slice + 1) / nsplit) - s_begin : nk_all;
    if constexpr (kEdge) tail_t = (k_tail < KE && s_begin + nk == nk_all) ? nk - 1 : -1;
    gbase = grp == 0 ? A + (int64_t)m0 * lda_b + (int64_t)s_begin * kFastKB
                     : B + (int64_t)n0 * ES + (int64_t)s_begin * KE * ldb_b;
    if constexpr (kEdge) set_voff();
  };
  place(item);
  if constexpr (!kEdge) set_voff();    // the same for every tile
  const int64_t gstep = grp == 0 ? (int64_t)kFastKB : (int64_t)KE * ldb_b;
  const unsigned lds0 = (grp == 0 ? lds_addr(sA) : lds_addr(sB)) + q * 4 * 1024;
  // The partial last stage: the same 16 bytes per lane into the same LDS
  // bytes as the DMA would write (lane L of instruction i at 1024 i + 16 L),
  // read with ordinary loads that skip every element past K -- A's columns
  // beyond K (the next row, or past the array) and B's rows beyond K -- and
  // write zeros there.  A wave may take any number of these loads (none when
  // its part lies wholly past K), so the issue ends by waiting for every
  // load of the wave: afterwards no load of this or an older stage is in
  // flight, and the stage waits below (which count kDma loads per later
  // stage in flight) hold trivially until the next tile's stages.
  auto issue_tail = [&](int slot_, int t) {
    const unsigned char *base = gbase + (int64_t)t * gstep;
    unsigned char *dst = (grp == 0 ? sA : sB) + q * 4 * 1024 + slot_ * kFastStage;
#pragma unroll
    for (int i = 0; i < kDma; ++i) {
      const int blk = q * 4 + i;
      u32x4 v = {0u, 0u, 0u, 0u};
      const unsigned char *src = base + voff[i];
      if (grp == 0) {
        const int valid = k_tail - (lane >> 4) * (16 / ES);   // elements of this chunk in K
        if (valid >= 16 / ES) {
          v = *(const u32x4 *)src;
        } else if (valid > 0) {
          unsigned w[4] = {0u, 0u, 0u, 0u};
          for (int e = 0; e < valid; ++e) {
            const unsigned x = ES == 2 ? (unsigned)((const unsigned short *)src)[e]
                                       : (unsigned)src[e];
            w[(e * ES) >> 2] |= x << (8 * ((e * ES) & 3));
          }
          v = u32x4{w[0], w[1], w[2], w[3]};
        }
      } else {
        const int krow = kI8 ? blk * 4 + (lane >> 4) : blk * 2 + (lane >> 5);
        if (krow < k_tail) v = *(const u32x4 *)src;
      }
      *(u32x4 *)(dst + i * 1024 + 16 * lane) = v;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  };
  auto issue = [&](int slot_, int t) {
    if constexpr (kEdge) {
      if (t == tail_t) {
        issue_tail(slot_, t);
        return;
      }
    }
    const unsigned char *base = gbase + (int64_t)t * gstep;
#pragma unroll
    for (int i = 0; i < kDma; ++i) dma_lds16_saddr(base, voff[i], lds0 + slot_ * kFastStage + i * 1024);
  };

  // Fragment offsets (stage 0): rows 128*grp.. of A, columns 64q.. of B^T.
  const int x_off = grp * 8 * 1024 + 16 * lane;
  int w_off[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    const int nbase = q * 64 + fn * 16;
    if constexpr (!kI8) {
      const int n = nbase + 4 * (r & 3);
      const int k0 = 8 * g + (r >> 2);
      w_off[fn] = k0 * BROW + 16 * ((n >> 3) ^ fb16_swz(k0)) + ((2 * n) & 15);
    } else {
      const int n = nbase + 8 * (r & 1);
      const int k0 = 16 * g + (r >> 1);
      w_off[fn] = k0 * BROW + 16 * ((n >> 4) ^ fb8_swz(k0)) + (n & 15);
    }
  }
  constexpr int kW1 = (kI8 ? 8 : 4) * BROW;

  Acc acc[FN][FM];
  u32x4 xf[FM], wf[FN];
  auto read_frags = [&](int slot_) {
    const unsigned char *sa = sA + slot_ * kFastStage;
    const unsigned char *sb = sB + slot_ * kFastStage;
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) xf[fm] = *(const u32x4 *)(sa + x_off + fm * 1024);
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      u32x2 w0, w1;
      if constexpr (!kI8) {
        w0 = lds_read_tr16(sb + w_off[fn]);
        w1 = lds_read_tr16(sb + w_off[fn] + kW1);
      } else {
        w0 = lds_read_tr8(sb + w_off[fn]);
        w1 = lds_read_tr8(sb + w_off[fn] + kW1);
      }
      wf[fn] = u32x4{w0[0], w0[1], w1[0], w1[1]};
    }
  };
  auto mfmas = [&]() {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) {
        if constexpr (kI8)
          acc[fn][fm] = mfma_i8_k64(wf[fn], xf[fm], acc[fn][fm]);
        else
          acc[fn][fm] = mfma_k32(DT, wf[fn], xf[fm], acc[fn][fm]);
      }
    }
    __builtin_amdgcn_s_setprio(0);
  };
  auto next_slot = [](int s0) { return s0 + 1 == kRing ? 0 : s0 + 1; };
  auto prev_slot = [](int s0) { return s0 == 0 ? kRing - 1 : s0 - 1; };
  // Wait until this wave's loads of a stage are complete while `later` of
  // its loads of later stages stay in flight, then barrier.
  auto wait_stage = [&](int later) {
    if (later >= 3)
      vm_wait_barrier<3 * kDma>();
    else if (later == 2)
      vm_wait_barrier<2 * kDma>();
    else if (later == 1)
      vm_wait_barrier<kDma>();
    else
      vm_wait_barrier<0>();
  };
  auto later_after = [&](int t) {   // loads of stages after t+1 in flight at the end of A(t)
    const int l = nk - 2 - t;
    return l < kRing - 2 ? l : kRing - 2;
  };

  for (int s0 = 0; s0 < kRing; ++s0)
    if (s0 < nk) issue(s0, s0);
  // Persistent loop over output tiles: after a tile's epilogue stores, the
  // first stages of the next tile are issued at once, so their loads overlap
  // the stores' drain instead of waiting for a new workgroup.
  for (;;) {
#pragma unroll
    for (int a = 0; a < FN; ++a)
#pragma unroll
      for (int b = 0; b < FM; ++b) acc[a][b] = Acc{0, 0, 0, 0};
    wait_stage(nk - 1 < kRing - 1 ? nk - 1 : kRing - 1);
    int slot = 0;
    if (grp == 0) {
      read_frags(0);
      for (int t = 0; t < nk; ++t) {
        mfmas();                                            // A(t): compute stage t
        wait_stage(later_after(t));
        if (t + 1 < nk) read_frags(next_slot(slot));       // B(t): read t+1, refill
        if (t + kRing < nk) issue(slot, t + kRing);
        vm_wait_barrier<63>();
        slot = next_slot(slot);
      }
    } else {
      for (int t = 0; t < nk; ++t) {
        read_frags(slot);                                   // A(t): read t, refill
        if (t >= 1 && t - 1 + kRing < nk) issue(prev_slot(slot), t - 1 + kRing);
        wait_stage(later_after(t));
        mfmas();                                            // B(t): compute stage t
        vm_wait_barrier<63>();
        slot = next_slot(slot);
      }
    }

    // Epilogue: lane holds C[row][col .. col+3] of every accumulator block.
    auto out_ptr = [&](int fn, int fm) {
      const int row = m0 + grp * 128 + fm * 16 + r;
      const int col = n0 + q * 64 + fn * 16 + 4 * g;
      return C + (int64_t)row * ldc_b + (int64_t)col * OB;
    };
    // The lane's 4 columns lie wholly inside or wholly outside C (n_lim is
    // a multiple of 4).
    auto in_c = [&](int fn, int fm) {
      return !kEdge ||
             (m0 + grp * 128 + fm * 16 + r < m_lim && n0 + q * 64 + fn * 16 + 4 * g < n_lim);
    };
    constexpr bool kSplittable = DT == TCU_F16_F32 || DT == TCU_BF16_F32 || DT == TCU_I8_I32;
    if (kSplittable && split_item) {
      // Partial tiles are added into C atomically.  In the accumulator
      // layout one atomic instruction would touch one element in each of
      // 16 rows, so every 64-byte line gets four separate requests; the
      // wave's 128 x 64 sub-tile goes through LDS instead (the ring is
      // free after the loop's last barrier), 64 rows at a time, and each
      // atomic instruction then adds 64 consecutive elements of one row.
      // Row stride 272 bytes: the 16 rows one 16-byte store instruction
      // touches land in distinct banks.
      if constexpr (kSplittable) {
        constexpr int kStride = 272;
        unsigned char *stage = (grp == 0 ? sA : sB) + q * 64 * kStride;
        const int col = n0 + q * 64 + lane;
#pragma unroll
        for (int h = 0; h < FM / 4; ++h) {
#pragma unroll
          for (int fn = 0; fn < FN; ++fn)
#pragma unroll
            for (int fm = 0; fm < 4; ++fm)
              *(Acc *)(stage + (fm * 16 + r) * kStride + (fn * 16 + 4 * g) * 4) =
                  acc[fn][h * 4 + fm];
          __syncthreads();
          const int row0 = m0 + grp * 128 + h * 64;
#pragma unroll 8
          for (int i = 0; i < 64; ++i) {
            if (kEdge && (row0 + i >= m_lim || col >= n_lim)) continue;
            unsigned char *p = C + (int64_t)(row0 + i) * ldc_b + (int64_t)col * OB;
            if constexpr (DT == TCU_I8_I32)
              __hip_atomic_fetch_add((int *)p, *(const int *)(stage + i * kStride + 4 * lane),
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else
              __hip_atomic_fetch_add((float *)p, *(const float *)(stage + i * kStride + 4 * lane),
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          __syncthreads();   // reads done before the next half (or the ring) overwrites
        }
      }
    } else {
      // Blocks fn and fn + 1 hold the two 64-byte halves of 128-byte rows
      // of C, so they are stored back to back: a half-written line left
      // in L2 while other stores intervene is written to memory twice
      // (measured: 1.37x the output bytes with fn outermost, 1.006x here).
      if (accum) {
        // C <- C + tile: the old values of two block rows (8 blocks) are
        // loaded together, then summed and stored -- one memory round trip
        // per 8 blocks instead of one per block.
#pragma unroll
        for (int fm0 = 0; fm0 < FM; fm0 += 2) {
          Old4<DT> old[2][FN];
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
              old[j][fn] = in_c(fn, fm0 + j) ? load_old4<DT>(out_ptr(fn, fm0 + j)) : Old4<DT>{};
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
              if (in_c(fn, fm0 + j))
                store_sum4<DT>(out_ptr(fn, fm0 + j), acc[fn][fm0 + j], old[j][fn]);
        }
      } else {
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int fn = 0; fn < FN; ++fn)
            if (in_c(fn, fm)) store_out4<DT, true>(out_ptr(fn, fm), acc[fn][fm], 4, false);
      }
    }
    // Every wave finished reading the ring at the last barrier of the loop.
    item += (int)gridDim.x;
    if (item >= total) break;
    place(item);
    for (int s0 = 0; s0 < kRing; ++s0)
      if (s0 < nk) issue(s0, s0);
  }
}

// ---------------------------------------------------------------------------
// Ring kernel: 128 x 128 or 64 x 64 output tiles, 4 waves (2 x 2, each a
// quarter of the tile), any M, N, K and any row pitch.  One LDS layout serves
// two ways of filling it:
//   * kDma: direct 16-byte DMA loads, kStages - 1 stages ahead (16-byte row
//     pitches, N a whole number of 16-byte chunks; a lane past the edge of C
//     loads the last row or chunk inside instead, and a partial last stage
//     goes through registers with zeros past K);
//   * otherwise: 16-byte loads at any byte address into registers one stage
//     ahead, written to the other of two LDS slots (kStages = 2).  A chunk
//     that crosses the end of a row is loaded from the last 16 bytes inside
//     it and shifted, and one past it repeats the last one (columns of B past
//     N, never stored) or becomes zero (past K), without branches, so every
//     load stays inside the operands and edge tiles cost what whole ones do.
//     Only rows shorter than 16 bytes are loaded element by element.
//   * A stage is 128 bytes of the contracted index.  Of A: BM rows of 128
//     bytes, their 16-byte chunks XOR-swizzled by the row, so that an
//     instruction fetches 8 whole lines and the rows one pass of a fragment
//     read touches hit distinct banks.  (16 rows of 64 bytes per instruction, whose
//     fragment reads are linear, took f16 1280^3 15.5 instead of 11.8 us, and
//     128 x 128 tiles with five such stages of 64 bytes took f16 2560^3 62
//     instead of 47: lines fetched in halves.)
//   * A stage of B: the stage's rows of BN columns, row-major, 16-byte chunks
//     XOR-swizzled by the row (ring_b_swz) so that the lanes of one pass of a
//     transposing read hit distinct banks.
// Work items are (K range, tile) pairs: with nsplit > 1 an item sums one of
// nsplit ranges of whole stages and adds its partial tile into C atomically
// (binary32 and int32 outputs).
// ---------------------------------------------------------------------------

// Wait until at most kPer * min(later, kMax) of this wave's DMA loads are in
// flight.
template <int kMax, int kPer>
__device__ __forceinline__ void wave_wait(int later) {
  if (kMax <= 0 || later >= kMax)
    asm volatile("s_waitcnt vmcnt(%0)" ::"i"(kMax > 0 ? kPer * kMax : 0) : "memory");
  else
    wave_wait<(kMax > 0 ? kMax - 1 : 0), kPer>(later);
}

// XOR swizzle of the 16-byte chunks of row k of a B stage whose rows hold
// `row_bytes` (64, 128 or 256) bytes.  A pass of 32 lanes of the transposing
// read touches rows 0-3 and 8-11 (32 bytes each, 16-bit) or rows 0-7 and
// 16-23 (16 bytes each, int8) of a K step; the swizzle spreads the rows that
// share a 256-byte bank window.
template <int ES, int row_bytes>
__device__ __forceinline__ int ring_b_swz(int k) {
  if constexpr (ES == 2) {
    static_assert(row_bytes == 64 || row_bytes == 128 || row_bytes == 256, "B stage rows");
    if constexpr (row_bytes == 256) return ((k & 3) << 1) | (((k >> 3) & 1) << 3);
    if constexpr (row_bytes == 128) return (((k >> 1) & 1) << 1) | (((k >> 3) & 1) << 2);
    return ((k >> 3) & 1) << 1;
  } else {
    static_assert(row_bytes == 64 || row_bytes == 128, "B stage rows");
    if constexpr (row_bytes == 128) return ((k >> 1) & 3) | (((k >> 4) & 1) << 2);
    return ((k >> 2) & 1) | (((k >> 4) & 1) << 1);
  }
}

// Wait until at most kPer * min(later, kMax) of this wave's DMA loads are in
// flight (and its LDS reads returned), then barrier.
template <int kMax, int kPer>
__device__ __forceinline__ void ring_wait(int later) {
  if constexpr (kMax == 0) {
    vm_wait_barrier<0>();
  } else {
    if (later >= kMax)
      vm_wait_barrier<kPer * kMax>();
    else
      ring_wait<kMax - 1, kPer>(later);
  }
}

constexpr int ring_lds(int bm, int bn, int stages) { return stages * (bm + bn) * 128; }

// Order a wave's own LDS accesses: its earlier reads have returned before what
// follows is issued, and the compiler moves none across.
__device__ __forceinline__ void wave_lds_order() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// gemm_wave_kernel: its tile's columns, a workgroup's waves, and the stages a
// wave of a tile of bm rows has in flight (what the LDS holds).
constexpr int kWaveN = 32, kTileWaves = 8;
constexpr int wave_stages(int bm) { return bm == 16 ? 3 : 2; }

// One work item: the BM x BN tile of C at (m0, n0), K range `slice` of nsplit,
// on ring_lds bytes of LDS.  kWaves = 4: a workgroup's.  kWaves = 1: a single
// wave's, without barriers; its sums stay in its LDS, kStride bytes per row, for
// gemm_wave_kernel to add.
template <int DT, int BM, int BN, int kStages, bool kDma, int kWaves = 4>
__device__ __forceinline__ void ring_tile(unsigned char *smem, const unsigned char *__restrict__ A,
                                          const unsigned char *__restrict__ B,
                                          unsigned char *__restrict__ C, int M, int N, int K,
                                          int64_t lda, int64_t ldb, int64_t ldc, int accum,
                                          int m0, int n0, int slice, int nsplit) {
  constexpr bool kI8 = in_bytes(DT) == 1;
  constexpr int ES = in_bytes(DT), OB = out_bytes(DT);
  constexpr int EPC = 16 / ES;
  constexpr int KB = 128;                        // bytes of the contracted index per stage
  constexpr int KE = KB / ES;                    // contracted elements per stage
  constexpr int KK = KB / 64;                    // matrix-core K steps per stage
  constexpr int BROW = BN * ES;                  // bytes per B row of a stage
  constexpr int kAStage = BM * KB, kBStage = BN * KB;
  constexpr bool kAlone = kWaves == 1;
  constexpr int JA = kAStage / 1024 / kWaves, JB = kBStage / 1024 / kWaves;   // 1 KiB pieces per wave
  constexpr int WTM = kAlone ? BM : BM / 2, WTN = kAlone ? BN : BN / 2;
  constexpr int FM = WTM / 16, FN = WTN / 16;
  static_assert(kAlone ? kStages == (kDma ? wave_stages(BM) : 1) : kWaves == 4, "four waves, or one alone");
  static_assert(!kDma || (JA + JB) * (kStages - 2) <= 63, "vmcnt range");
  static_assert(kDma || kAlone || kStages == 2, "register-staged: two slots");
  typedef typename std::conditional<kI8, i32x4, f32x4>::type Acc;
  unsigned char *const sA = smem;
  unsigned char *const sB = smem + kStages * kAStage;

  const int lane = threadIdx.x & 63;
  const int w = kAlone ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = w >> 1, wn = w & 1;
  const int r = lane & 15, g = lane >> 4;
  const int64_t lda_b = lda * ES, ldb_b = ldb * ES, ldc_b = ldc * OB;
  const int nk_all = (K + KE - 1) / KE;
  // A range of whole stages, or (alone) every kStep'th: the waves then fetch
  // adjacent lines, which are spread over the cache's channels.
  constexpr int kStep = kAlone ? kTileWaves : 1;
  const int s_begin = kAlone ? slice : (int)((int64_t)nk_all * slice / nsplit);
  const int nk = kAlone ? (nk_all - slice + kStep - 1) / kStep
                        : (int)((int64_t)nk_all * (slice + 1) / nsplit) - s_begin;
  const int k_first = s_begin * KE;

  // Piece j of a stage: LDS bytes [1024 j, 1024 (j + 1)), lane by lane -- of A
  // rows 8 j + lane / 8, of B the rows that lie there.
  auto a_row = [&](int j) { return 8 * j + (lane >> 3); };
  const int a_chunk = (lane & 7) ^ (lane >> 3);
  auto b_row = [&](int j) { return (1024 * j + 16 * lane) / BROW; };
  auto b_chunk = [&](int j) {
    return (((1024 * j + 16 * lane) % BROW) / 16) ^ ring_b_swz<ES, BROW>(b_row(j));
  };
  // DMA: wave-uniform bases, per-lane 32-bit offsets.
  unsigned aoff[JA], boff[JB];
  const unsigned char *abase = A + (int64_t)m0 * lda_b + (int64_t)k_first * ES;
  const unsigned char *bbase = B + (int64_t)k_first * ldb_b + (int64_t)n0 * ES;
  const int c_last = (N - n0) * ES / 16 - 1;
  if constexpr (kDma) {
#pragma unroll
    for (int i = 0; i < JA; ++i)
      aoff[i] = (unsigned)(min(a_row(w * JA + i), M - 1 - m0) * lda_b) + 16u * a_chunk;
#pragma unroll
    for (int i = 0; i < JB; ++i)
      boff[i] = (unsigned)(b_row(w * JB + i) * ldb_b) + 16u * min(b_chunk(w * JB + i), c_last);
  }
  const unsigned a_lds = lds_addr(sA) + w * JA * 1024, b_lds = lds_addr(sB) + w * JB * 1024;
  const bool has_last = s_begin + (nk - 1) * kStep == nk_all - 1;
  const int tail_t = K - (nk_all - 1) * KE < KE && has_last ? nk - 1 : -1;
  // Addresses of the register loads at stage 0, and for every piece of B the
  // bytes its chunk is shifted by because it crosses N.
  const bool short_rows = K < EPC || N < EPC;
  const bool cross_n = !short_rows && n0 + BN > N && N % EPC != 0;
  const unsigned char *pa[JA], *pb[JB];
  int sh_b[JB];
#pragma unroll
  for (int i = 0; i < JA; ++i)
    pa[i] = A + (int64_t)min(m0 + a_row(w * JA + i), M - 1) * lda_b + (int64_t)k_first * ES +
            16 * a_chunk;
#pragma unroll
  for (int i = 0; i < JB; ++i) {
    const int c = n0 + b_chunk(w * JB + i) * EPC, cc = short_rows ? c : min(c, N - EPC);
    pb[i] = B + (int64_t)(k_first + b_row(w * JB + i)) * ldb_b + (int64_t)cc * ES;
    sh_b[i] = c < N ? (c - cc) * ES : 0;
  }
  auto put = [&](int slot, const u32x4 (&ra)[JA], const u32x4 (&rb)[JB]) {
#pragma unroll
    for (int i = 0; i < JA; ++i)
      *(u32x4 *)(sA + slot * kAStage + (w * JA + i) * 1024 + 16 * lane) = ra[i];
#pragma unroll
    for (int i = 0; i < JB; ++i)
      *(u32x4 *)(sB + slot * kBStage + (w * JB + i) * 1024 + 16 * lane) =
          cross_n ? shift_down(rb[i], sh_b[i]) : rb[i];
  };
  // Stage t into registers: whole, or (tail) zeros past K.
  auto get = [&](int t, u32x4 (&ra)[JA], u32x4 (&rb)[JB]) __attribute__((always_inline)) {
    const int64_t at = (int64_t)t * (kStep * KB), bt = (int64_t)t * (kStep * KE) * ldb_b;
    if (t != tail_t && !short_rows) {
#pragma unroll
      for (int i = 0; i < JA; ++i) ra[i] = load16_any(pa[i] + at);
#pragma unroll
      for (int i = 0; i < JB; ++i) rb[i] = load16_any(pb[i] + bt);
      return;
    }
    const int kleft = K - k_first - t * (kStep * KE);   // contracted indices left
    if (!short_rows) {
#pragma unroll
      for (int i = 0; i < JA; ++i) {
        // the last chunk inside the row may start before this stage
        const int c = a_chunk * EPC, back = c - min(c, kleft - EPC);
        const u32x4 v = shift_down(load16_any(pa[i] + at - back * ES), (back * ES) & 15);
        ra[i] = c < kleft ? v : u32x4{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int i = 0; i < JB; ++i) {
        const int k = b_row(w * JB + i), back = k - min(k, kleft - 1);
        rb[i] = load16_any(pb[i] + bt - back * ldb_b);
        if (back > 0) rb[i] = u32x4{0u, 0u, 0u, 0u};
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < JA; ++i)
      ra[i] = load_chunk<ES>(pa[i] + at,
                                    max(min(kleft - a_chunk * EPC, EPC), 0));
#pragma unroll
    for (int i = 0; i < JB; ++i) {
      const int nleft = N - n0 - b_chunk(w * JB + i) * EPC;
      rb[i] = load_chunk<ES>(pb[i] + bt,
                                    b_row(w * JB + i) < kleft ? max(min(nleft, EPC), 0) : 0);
    }
  };
  auto issue = [&](int slot, int t) {
    if (t == tail_t) {
      u32x4 ra[JA], rb[JB];
      get(t, ra, rb);
      put(slot, ra, rb);
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the stage waits count DMA loads
      return;
    }
    const unsigned char *ga = abase + (int64_t)t * (kStep * KB);
    const unsigned char *gb = bbase + (int64_t)t * (kStep * KE) * ldb_b;
#pragma unroll
    for (int i = 0; i < JA; ++i) dma_lds16_saddr(ga, aoff[i], a_lds + slot * kAStage + i * 1024);
#pragma unroll
    for (int i = 0; i < JB; ++i) dma_lds16_saddr(gb, boff[i], b_lds + slot * kBStage + i * 1024);
  };

  // Fragment offsets within a stage: A rows WTM wm .., B^T columns WTN wn ..
  int x_off[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
    x_off[kk] = (wm * WTM + r) * KB + 16 * ((4 * kk + g) ^ (r & 7));
  int w_off[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    const int nbase = wn * WTN + fn * 16;
    if constexpr (!kI8) {
      const int n = nbase + 4 * (r & 3);
      const int k0 = 8 * g + (r >> 2);
      w_off[fn] = k0 * BROW + 16 * ((n >> 3) ^ ring_b_swz<ES, BROW>(k0)) + ((2 * n) & 15);
    } else {
      const int n = nbase + 8 * (r & 1);
      const int k0 = 16 * g + (r >> 1);
      w_off[fn] = k0 * BROW + 16 * ((n >> 4) ^ ring_b_swz<ES, BROW>(k0)) + (n & 15);
    }
  }
  constexpr int kW1 = (kI8 ? 8 : 4) * BROW;      // the second half of a lane's run
  constexpr int kWK = (kI8 ? 64 : 32) * BROW;    // the next K step

  Acc acc[FN][FM];
#pragma unroll
  for (int a = 0; a < FN; ++a)
#pragma unroll
    for (int b = 0; b < FM; ++b) acc[a][b] = Acc{0, 0, 0, 0};
  auto read_step = [&](int slot, int kk, u32x4 (&xf)[FM], u32x4 (&wf)[FN])
      __attribute__((always_inline)) {
    const unsigned char *sa = sA + slot * kAStage;
    const unsigned char *sb = sB + slot * kBStage;
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) xf[fm] = *(const u32x4 *)(sa + x_off[kk] + fm * 16 * KB);
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      u32x2 w0, w1;
      if constexpr (!kI8) {
        w0 = lds_read_tr16(sb + w_off[fn] + kk * kWK);
        w1 = lds_read_tr16(sb + w_off[fn] + kk * kWK + kW1);
      } else {
        w0 = lds_read_tr8(sb + w_off[fn] + kk * kWK);
        w1 = lds_read_tr8(sb + w_off[fn] + kk * kWK + kW1);
      }
      wf[fn] = u32x4{w0[0], w0[1], w1[0], w1[1]};
    }
  };
  auto multiply = [&](const u32x4 (&xf)[FM], const u32x4 (&wf)[FN]) __attribute__((always_inline)) {
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) {
        if constexpr (kI8)
          acc[fn][fm] = mfma_i8_k64(wf[fn], xf[fm], acc[fn][fm]);
        else
          acc[fn][fm] = mfma_k32(DT, wf[fn], xf[fm], acc[fn][fm]);
      }
  };
  auto compute = [&](int slot) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      u32x4 xf[FM], wf[FN];
      read_step(slot, kk, xf, wf);
      multiply(xf, wf);
    }
  };

  constexpr int kStride = WTN * 4 + 16;
  if constexpr (kAlone) {
    // A stage's fragments are read into registers, then the stage two later is
    // fetched in its place under their products: by DMA into the slot, or into
    // the registers it was written from.
    u32x4 xf[KK][FM], wf[KK][FN];
    auto step = [&](int slot, auto fetch) __attribute__((always_inline)) {
      wave_lds_order();
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) read_step(slot, kk, xf[kk], wf[kk]);
      wave_lds_order();
      fetch();
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) multiply(xf[kk], wf[kk]);
    };
    if constexpr (kDma) {
      for (int t = 0; t < kStages; ++t)
        if (t < nk) issue(t, t);
      int slot = 0;
      for (int t = 0; t < nk; ++t) {
        const int later = nk - 1 - t < kStages - 1 ? nk - 1 - t : kStages - 1;
        wave_wait<kStages - 1, JA + JB>(later);
        step(slot, [&]() {
          if (t + kStages < nk) issue(slot, t + kStages);
        });
        slot = slot + 1 == kStages ? 0 : slot + 1;
      }
    } else {
      constexpr int kAhead = wave_stages(BM);
      u32x4 ra[kAhead][JA], rb[kAhead][JB];
#pragma unroll
      for (int h = 0; h < kAhead; ++h)
        if (h < nk) get(h, ra[h], rb[h]);
      for (int t = 0; t < nk; t += kAhead) {
#pragma unroll
        for (int h = 0; h < kAhead; ++h) {
          if (t + h >= nk) break;
          put(0, ra[h], rb[h]);
          step(0, [&]() {
            if (t + h + kAhead < nk) get(t + h + kAhead, ra[h], rb[h]);
          });
        }
      }
    }
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
        *(Acc *)(smem + (fm * 16 + r) * kStride + (fn * 16 + 4 * g) * 4) = acc[fn][fm];
    return;
  }

  if constexpr (kDma) {
    for (int s0 = 0; s0 < kStages - 1; ++s0)
      if (s0 < nk) issue(s0, s0);
    int slot = 0;
    for (int t = 0; t < nk; ++t) {
      // This wave's loads of stage t done (those of the stages after it may
      // stay in flight); the barrier makes every wave's share visible and
      // ensures all waves finished reading stage t-1, whose slot is refilled.
      const int later = nk - 1 - t < kStages - 2 ? nk - 1 - t : kStages - 2;
      ring_wait<kAlone ? 0 : kStages - 2, JA + JB>(later);
      const int refill = t + kStages - 1;
      if (refill < nk) issue(slot == 0 ? kStages - 1 : slot - 1, refill);
      compute(slot);
      slot = slot + 1 == kStages ? 0 : slot + 1;
    }
  } else {
    u32x4 ra[JA], rb[JB];
    if (nk > 0) {
      get(0, ra, rb);
      put(0, ra, rb);
    }
    if (nk > 1) get(1, ra, rb);
    for (int t = 0; t < nk; ++t) {
      // Stage t is in its slot and every wave has finished reading the other
      // one; stage t+1's loads, issued a stage ago, go there, and stage
      // t+2's are issued before the products.
      __syncthreads();
      if (t + 1 < nk) put((t + 1) & 1, ra, rb);
      if (t + 2 < nk) get(t + 2, ra, rb);
      compute(t & 1);
    }
  }

  // Epilogue: lane holds C[row][col .. col+3] of every accumulator block.
  constexpr bool kSplittable = DT == TCU_F16_F32 || DT == TCU_BF16_F32 || DT == TCU_I8_I32;
  unsigned char *stage = smem + w * 32 * kStride;
  static_assert(kAlone || 4 * 32 * kStride <= kStages * (kAStage + kBStage), "staging fits the ring");
  if constexpr (kSplittable) {
    if (nsplit > 1) {
      // Partial tiles are added into C atomically, through this wave's part
      // of LDS so that one atomic instruction covers whole runs of a row.
      constexpr int kRowsPer = 64 / WTN;         // rows per atomic instruction
      __syncthreads();   // every wave finished reading the ring
      const int col = n0 + wn * WTN + lane % WTN;
#pragma unroll
      for (int h = 0; h < FM / 2; ++h) {
#pragma unroll
        for (int fn = 0; fn < FN; ++fn)
#pragma unroll
          for (int fm = 0; fm < 2; ++fm)
            *(Acc *)(stage + (fm * 16 + r) * kStride + (fn * 16 + 4 * g) * 4) =
                acc[fn][2 * h + fm];
        __syncthreads();
        const int row0 = m0 + wm * WTM + 32 * h;
#pragma unroll 8
        for (int i = lane / WTN; i < 32; i += kRowsPer) {
          if (row0 + i >= M || col >= N) continue;
          unsigned char *p = C + (int64_t)(row0 + i) * ldc_b + (int64_t)col * OB;
          const unsigned char *v = stage + i * kStride + (lane % WTN) * 4;
          if constexpr (DT == TCU_I8_I32)
            __hip_atomic_fetch_add((int *)p, *(const int *)v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
          else
            __hip_atomic_fetch_add((float *)p, *(const float *)v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();   // reads done before the next rows overwrite
      }
      return;
    }
  }
  if constexpr (!kDma && OB == 2 && BM == 128) {
    if ((((uintptr_t)C | (uintptr_t)ldc_b) & (4 * OB - 1)) != 0) {
      // 16-bit rows that start anywhere go through LDS too: in the accumulator
      // layout a store is 16 runs of 32 bytes, most of them across sectors;
      // here its runs are the sub-tile's whole rows.  us, direct -> staged:
      // 4101 x 1000 x 4173 71.6 -> 68.5, 3072 x 200 x 3071 20.7 -> 16.8.
      // 4-byte outputs do not gain (3072 x 1000 x 3071 39.6 -> 40.2), and 64 x
      // 64 tiles lose to the barriers (1001 x 1003 x 1005 10.4 -> 11.0).
      constexpr int kRowLanes = WTN / 4, kRowsPer = 64 / kRowLanes;
      const int col = n0 + wn * WTN + 4 * (lane % kRowLanes);
      const int valid = min(max(N - col, 0), 4);
      __syncthreads();   // every wave finished reading the ring
#pragma unroll
      for (int h = 0; h < FM / 2; ++h) {
#pragma unroll
        for (int fn = 0; fn < FN; ++fn)
#pragma unroll
          for (int fm = 0; fm < 2; ++fm)
            *(Acc *)(stage + (fm * 16 + r) * kStride + (fn * 16 + 4 * g) * 4) =
                acc[fn][2 * h + fm];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 32; i += kRowsPer) {
          const int in = i + lane / kRowLanes, row = m0 + wm * WTM + 32 * h + in;
          const Acc v = *(const Acc *)(stage + in * kStride + (lane % kRowLanes) * 16);
          unsigned char *p = C + (int64_t)row * ldc_b + (int64_t)col * OB;
          if (row < M && valid == 4)
            store_out4<DT, true>(p, v, 4, accum != 0);
          else if (row < M && valid > 0)
            store_out4<DT, false>(p, v, valid, accum != 0);
        }
        __syncthreads();   // reads done before the next rows overwrite
      }
      return;
    }
  }
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      const int row = m0 + wm * WTM + fm * 16 + r;
      const int col = n0 + wn * WTN + fn * 16 + 4 * g;
      unsigned char *p = C + (int64_t)row * ldc_b + (int64_t)col * OB;
      const int valid = row < M ? min(max(N - col, 0), 4) : 0;
      if (valid == 4)
        store_out4<DT, true>(p, acc[fn][fm], 4, accum != 0);
      else if (valid > 0)
        store_out4<DT, false>(p, acc[fn][fm], valid, accum != 0);
    }
  }
}

// Work items are (K range, tile) pairs.  kCut (128 x 128, unsplit): the tiles from
// `whole` on are cut into four quarters of 64 x 64, items of their own (empty past
// the edge of C), so that a last round of few tiles is spread over the chip.  An
// instance apart: with both bodies in one, whole tiles took bf16 3328 x 1024 x
// 3328 35.0 instead of 33.8 us.
template <int DT, int kTile, int kStages, bool kDma, bool kCut>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256),
                          amdgpu_waves_per_eu(1, kTile == 64 ? (kDma ? 3 : 4) : 2))) void
gemm_ring_kernel(const unsigned char *__restrict__ A, const unsigned char *__restrict__ B,
                 unsigned char *__restrict__ C, int M, int N, int K, int64_t lda, int64_t ldb,
                 int64_t ldc, int accum, int tiles_m, int tiles_n, int nsplit, int whole,
                 int first) {
  constexpr int kQuarterStages = kDma ? 4 : 2;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[ring_lds(kTile, kTile, kStages)];
  const int tiles = tiles_m * tiles_n;
  // Split items go K range by K range, permuted so that each XCD holds a
  // contiguous run of them (its L2 then serves one range's panels); the
  // items past the last multiple of 8 keep their ids.
  int pid = first + blockIdx.x, slice = 0, quarter = 0;
  const bool cut = kCut && pid >= whole;
  if (!kCut && nsplit > 1) {
    const int body = tiles * nsplit / 8 * 8;
    if (pid < body) pid = (pid % 8) * (body / 8) + pid / 8;
    slice = pid / tiles;
    pid -= slice * tiles;
  } else if (cut) {
    quarter = (pid - whole) & 3;
    pid = whole + ((pid - whole) >> 2);
  }
  int tm, tn;
  map_tile(pid, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * kTile, n0 = tn * kTile;
  if constexpr (kCut) {
    static_assert(ring_lds(64, 64, kQuarterStages) <= ring_lds(kTile, kTile, kStages), "a quarter's ring");
    if (cut) {
      const int mq = m0 + 64 * (quarter >> 1), nq = n0 + 64 * (quarter & 1);
      if (mq < M && nq < N)
        ring_tile<DT, 64, 64, kQuarterStages, kDma>(smem, A, B, C, M, N, K, lda, ldb, ldc, accum,
                                                    mq, nq, 0, 1);
      return;
    }
  }
  ring_tile<DT, kTile, kTile, kStages, kDma>(smem, A, B, C, M, N, K, lda, ldb, ldc, accum, m0, n0,
                                             slice, kCut ? 1 : nsplit);
}

// Few tiles, binary32 sums in a fixed order: a workgroup's 8 waves take one tile
// of kM x 32, each every eighth stage of K, with the stages that fill a CU's LDS in
// flight; the waves' sums are added in their order, then C's old value.  kM by the
// tiles: 16 rows while they are one round (192 x 1024 x 320, 120 tiles: 4.6 us, 60 of
// 32 rows 5.4), else 32 (512 x 1024 x 512, 256 tiles: 6.0, 512 of 16 rows 8.2).
template <int DT, int kM, bool kDma>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * kTileWaves, 64 * kTileWaves))) void
gemm_wave_kernel(const unsigned char *__restrict__ A, const unsigned char *__restrict__ B,
                 unsigned char *__restrict__ C, int M, int N, int K, int64_t lda, int64_t ldb,
                 int64_t ldc, int accum, int tiles_m, int tiles_n) {
  static_assert(DT == TCU_F16_F32 || DT == TCU_BF16_F32, "binary32 outputs");
  constexpr int kStages = kDma ? wave_stages(kM) : 1;
  constexpr int kPart = ring_lds(kM, kWaveN, kStages), kStride = kWaveN * 4 + 16;
  static_assert(kM * kStride <= kPart, "a wave's sums");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kTileWaves * kPart];
  // each XCD holds a contiguous run of tiles
  int pid = blockIdx.x;
  const int body = tiles_m * tiles_n / 8 * 8;
  if (pid < body) pid = (pid % 8) * (body / 8) + pid / 8;
  int tm, tn;
  map_tile<64 / kM>(pid, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * kM, n0 = tn * kWaveN;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  ring_tile<DT, kM, kWaveN, kStages, kDma, 1>(smem + w * kPart, A, B, C, M, N, K, lda, ldb, ldc, 0,
                                              m0, n0, w, kTileWaves);
  __syncthreads();
  const int col = threadIdx.x % kWaveN;
#pragma unroll
  for (int i = 0; i < kM; i += 64 * kTileWaves / kWaveN) {
    const int row = i + threadIdx.x / kWaveN;
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < kTileWaves; ++j)
      v += *(const float *)(smem + j * kPart + row * kStride + 4 * col);
    if (m0 + row < M && n0 + col < N) {
      float *p = (float *)C + (int64_t)(m0 + row) * ldc + n0 + col;
      *p = accum ? *p + v : v;
    }
  }
}

// Zero the rows x row_words view of 4-byte words at C (row pitch ldc_w
// words): the starting value of a split-K product that overwrites C.  With
// kVec, row_words and ldc_w are multiples of 4.
template <bool kVec>
__global__ __launch_bounds__(256) void zero_fill_kernel(unsigned *__restrict__ C, int64_t rows,
                                                        int64_t row_words, int64_t ldc_w) {
  constexpr int V = kVec ? 4 : 1;
  const int64_t per_row = row_words / V;
  const int64_t total = rows * per_row;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t rr = i / per_row;
    unsigned *p = C + rr * ldc_w + (i - rr * per_row) * V;
    if constexpr (kVec)
      *(u32x4 *)p = u32x4{0u, 0u, 0u, 0u};
    else
      *p = 0u;
  }
}

hipError_t zero_view(const RectArgs &a, hipStream_t stream, int num_cus) {
  unsigned *C = (unsigned *)a.C;
  if (a.N % 4 == 0 && a.ldc % 4 == 0)
    hipLaunchKernelGGL(zero_fill_kernel<true>, dim3(num_cus * 4), dim3(256), 0, stream, C, a.M,
                       a.N, a.ldc);
  else
    hipLaunchKernelGGL(zero_fill_kernel<false>, dim3(num_cus * 4), dim3(256), 0, stream, C, a.M,
                       a.N, a.ldc);
  return hipGetLastError();
}

// Zero the output tiles pid in [first, first + count) of a tiles_m x
// tiles_n grid of 256 x 256 tiles of 4-byte values (placed by map_tile),
// clipped to rows < m_lim and to the first row_bytes bytes of each row (a
// multiple of 16): the starting value of the split tail tiles of a product
// that overwrites C.
__global__ __launch_bounds__(256) void zero_tiles_kernel(unsigned char *__restrict__ C,
                                                         int64_t ldc_b, int tiles_m, int tiles_n,
                                                         int first, int count, int m_lim,
                                                         int64_t row_bytes) {
  constexpr int kChunks = 256 * 4 / 16;   // 16-byte chunks per tile row
  const int64_t total = (int64_t)count * 256 * kChunks;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int t = (int)(i / (256 * kChunks));
    const int rem = (int)(i - (int64_t)t * 256 * kChunks);
    int tm, tn;
    map_tile(first + t, tiles_m, tiles_n, tm, tn);
    const int row = tm * 256 + rem / kChunks;
    const int64_t cb = (int64_t)tn * 1024 + 16 * (rem % kChunks);
    if (row < m_lim && cb < row_bytes)
      *(u32x4 *)(C + (int64_t)row * ldc_b + cb) = u32x4{0u, 0u, 0u, 0u};
  }
}

// The tail split: when a persistent grid of `grid` workgroups walks `tiles`
// whole tiles and the last round holds only tiles % grid of them, most CUs
// would idle through it.  Those tail tiles are cut into K ranges instead (at
// least kMinSplitStages stages each, at most grid / tail of them), added into
// C atomically, so the last round is about 1 / ranges as long.
constexpr int kMinSplitStages = 32;
int tail_ranges(int64_t tiles, int64_t grid, int64_t stages) {
  if (tiles <= grid || tiles % grid == 0) return 1;
  const int64_t ns = grid / (tiles % grid), cap = stages / kMinSplitStages;
  return (int)(ns < cap ? ns : cap);
}

// The ranges of a product's tail split (1: none), with *full set to the
// number of whole tiles.  binary32 and int32 outputs only (a bfloat16 output
// is rounded once from the whole sum).  The test override
// TCU_KNOB_TAIL_SPLIT = n > 0 forces n ranges (1: none).
template <int DT>
int tail_split(int tiles, int grid, int64_t stages, int *full) {
  *full = tiles;
  if (DT == TCU_BF16_BF16 || tiles <= grid || tiles % grid == 0) return 1;
  int64_t ns = tail_ranges(tiles, grid, stages);
  const int forced = knob(TCU_KNOB_TAIL_SPLIT);
  if (forced > 0) ns = forced < stages ? forced : stages;
  if (ns < 2) return 1;
  *full = tiles - tiles % grid;
  return (int)ns;
}

// Zero the tail tiles [full, tiles) of an overwriting product split by
// tail_split (C of 4-byte values, row pitch ldc_b bytes).
hipError_t zero_tail(unsigned char *C, int64_t ldc_b, int tm, int tn, int full, int m_lim,
                     int64_t row_bytes, hipStream_t stream, int num_cus) {
  hipLaunchKernelGGL(zero_tiles_kernel, dim3(num_cus * 4), dim3(256), 0, stream, C, ldc_b, tm,
                     tn, full, tm * tn - full, m_lim, row_bytes);
  return hipGetLastError();
}

// The ring kernel with kTile x kTile tiles and nsplit K ranges, tiles from
// `whole` on in quarters (128 x 128, unsplit).  A CU holds
// two workgroups of 128 x 128 tiles (two stages each) or three of 64 x 64 (DMA:
// three stages; with eight and one workgroup per CU, order 1024 took 9.7
// instead of 8.6 us and order 1120, whose 324 tiles then run in two rounds,
// 18.6 instead of 12.2).
template <int DT, int kTile, bool kDma>
hipError_t launch_ring(const RectArgs &a, int nsplit, int whole, hipStream_t stream,
                       int num_cus) {
  const int tiles_m = (int)((a.M + kTile - 1) / kTile), tiles_n = (int)((a.N + kTile - 1) / kTile);
  if (nsplit > 1 && !a.accum) {
    const hipError_t e = zero_view(a, stream, num_cus);
    if (e != hipSuccess) return e;
  }
  constexpr int kStages = kDma && kTile == 64 ? 3 : 2;
  const int tiles = tiles_m * tiles_n;
  if (whole > tiles || nsplit > 1) whole = tiles;
  auto go = [&](auto cut, int items) {
    // A launch's work items count in 32 bits (2^30 rows of one column are 2^24
    // tiles of 64 x 64): more workgroups than that take several launches.
    constexpr int kMost = 1 << 23;
    for (int first = 0; first < items && (first == 0 || hipPeekAtLastError() == hipSuccess);
         first += kMost)
      hipLaunchKernelGGL((gemm_ring_kernel<DT, kTile, kStages, kDma, decltype(cut)::value>),
                         dim3(items - first < kMost ? items - first : kMost), dim3(256), 0, stream,
                         (const unsigned char *)a.A, (const unsigned char *)a.B,
                         (unsigned char *)a.C, (int)a.M, (int)a.N, (int)a.K, a.lda, a.ldb, a.ldc,
                         a.accum ? 1 : 0, tiles_m, tiles_n, nsplit, whole, first);
  };
  if (kTile == 128 && whole < tiles)
    go(std::integral_constant<bool, kTile == 128>{}, whole + 4 * (tiles - whole));
  else
    go(std::false_type{}, tiles * nsplit);
  return hipGetLastError();
}

template <int DT>
constexpr bool kWaveSums = DT == TCU_F16_F32 || DT == TCU_BF16_F32;
template <int DT, int kM, bool kDma>
hipError_t launch_wave(const RectArgs &a, hipStream_t stream) {
  const int tiles_m = (int)((a.M + kM - 1) / kM), tiles_n = (int)((a.N + kWaveN - 1) / kWaveN);
  hipLaunchKernelGGL((gemm_wave_kernel<DT, kM, kDma>), dim3(tiles_m * tiles_n),
                     dim3(64 * kTileWaves), 0, stream, (const unsigned char *)a.A,
                     (const unsigned char *)a.B, (unsigned char *)a.C, (int)a.M, (int)a.N,
                     (int)a.K, a.lda, a.ldb, a.ldc, a.accum ? 1 : 0, tiles_m, tiles_n);
  return hipGetLastError();
}

// Kernel selection by size; the test override TCU_KNOB_GEMM_KERNEL forces the
// full-tile (ping-pong) kernel wherever its shape conditions hold (ragged
// shapes too), the ring kernel filled through registers, or its 64 x 64 tiles.
enum class GemmPath { kAuto, kFast, kGeneral, kRing };
GemmPath gemm_path() {
  switch (knob(TCU_KNOB_GEMM_KERNEL)) {
    case TCU_PATH_FULL_TILE: return GemmPath::kFast;
    case TCU_PATH_GENERAL: return GemmPath::kGeneral;
    case TCU_PATH_RING: return GemmPath::kRing;
  }
  return GemmPath::kAuto;
}

// ---------------------------------------------------------------------------
// Choice of kernel, tile and K split: the cheapest by a model of the time
// (microseconds) of t tiles whose contracted index is n64 pieces of 64 bytes
// on `cus` compute units.  The constants are measured per 64-byte piece; both
// sides at the sizes where the choice turns (us; full tile / 128 / 64):
//   bf16 N = 1024: 31 / 14.4 / 9.0     N = 1536: 43 / 20.3 / 18.1
//        N = 2048: 50 / 27.4 / 33.0    N = 2560: 64 / 42 / 62
//        N = 3072: 73 / 79 / 95        N = 4096: 110 / 132 / 220
//   int8 N = 1536: 28 / 13.7 / 13.6    N = 2560: 39 / 26 / 41
//        N = 3072: 44 / 47 / 74        N = 4096: 64 / 73 / 190
// (N = 3072's last round of 64 tiles whole; in quarters int8 takes 41.)
//   M x K x N full / 128, operands not in the caches:
//   f16  4350 x 4096 x 4352 (last round of 33 tiles split) 166 / 189
//        6000 x 1000 x 6000 116 / 125   6000 x 6000 x 6000 395 / 571
//        7000 x 1024 x 7008 128 / 148   4350 x 1024 x 4352 77 / 65
//   bf16 out 6000 x 512 x 6000 57 / 61  4350 x 4096 x 4352 208 / 186
// Fitted to 170 such sizes of 100 to 2500 full tiles: the full-tile kernel within 6
// %, 128 x 128 within 7 %; the choice is 0.4 % from the better one on average, and
// up to 16 % (7000 x 1024 x 7008, whose last round is 16 full tiles).  Rows of A or B that start inside a 128-byte line cost
// the smaller tiles, which fetch whole lines, more than the full ones.
// Filled through registers the ring kernel takes 1.1 to 1.25 times as long.
// Split ranges are added atomically, after zeroing C when overwriting:
// f16 192 x 8192 x 320 (15 tiles of 64) 37 us whole, 10.1 with 18 ranges,
// 12.9 with 32; bf16 N = 3072 full-tile 74 whole, 135 with 2 ranges.
// ---------------------------------------------------------------------------
enum class Tile { kFull, k128, k64, kWave32, kWave16 };
struct Choice {
  Tile tile = Tile::k64;
  int nsplit = 1;
  double us = 1e30;
};

// What a product's time depends on besides its tiles: whether the ring kernel
// fills by DMA, the bytes of an output, and the rows that start inside a line.
struct Traits {
  bool dma;
  int ob;
  bool a_inside, b_inside;
};
template <int DT>
Traits traits(const RectArgs &a, bool dma) {
  constexpr int ES = in_bytes(DT);
  return Traits{dma, out_bytes(DT), a.lda * ES % 128 != 0, a.ldb * ES % 128 != 0};
}

// *cut: whether the tiles of a last, partial round are cut into quarters (128).
double model_us(Tile tile, const Traits &f, int64_t t, double n64, int64_t cus, bool splittable,
                bool *cut = nullptr) {
  const bool dma = f.dma;
  switch (tile) {
    case Tile::kFull: {
      // one workgroup per CU, whole rounds; the last may be split
      const double stages = 0.7 * n64 * (1 + 0.07 * (f.a_inside + f.b_inside));
      const double round = stages + 8 + 1.7 * f.ob * (t < cus ? (double)t / (double)cus : 1.0);
      const int ns = splittable ? tail_ranges(t, cus, (int64_t)n64) : 1;
      if (ns > 1) return (double)(t / cus) * round + stages / ns + 33;
      return (double)((t + cus - 1) / cus) * round;
    }
    case Tile::k128: {
      // two workgroups per CU, which share its LDS bandwidth
      if (cut) *cut = false;
      if (t < 2 * cus) return (t > cus ? 0.44 * n64 + 5 : 0.33 * n64 + 4) * (dma ? 1.0 : 1.22);
      const double fill = dma ? 1 + 0.22 * f.a_inside + 0.1 * f.b_inside : 1.22;
      const double pair = 0.46 * n64 * fill + 4 + f.ob, single = 0.35 * n64 * fill + 4.5;
      const int64_t rem = t % (2 * cus);
      const double rounds = (double)(t / (2 * cus)) * pair;
      const double last = rem > cus ? pair : rem > 0 ? single : 0.0;
      if (rem == 0) return rounds;
      // The tiles of a last round of at most cus / 2 are cut into quarters, two
      // per CU at most, which take about 0.55 of a tile's time (us, whole / cut;
      // odd pitches, bf16: 3072 x 1000 x 3071, 64 tiles, 45.9 / 40.2; 3200 x
      // 1000 x 3199, 113 tiles, 45.7 / 42.9; 3328 x 1000 x 3327, 164 tiles,
      // 46.1 / 50.7; by DMA 3072 x 2048 x 3072, 64 tiles, 56.7 / 46.7; 3200 x
      // 512 x 3200, 113 tiles, 23.9 / 21.5; 3328 x 1024 x 3328 35.3 / 36.2).
      if (2 * rem > cus) return rounds + last;
      if (cut) *cut = true;
      return rounds + 0.55 * last;
    }
    case Tile::kWave32:   // one workgroup per CU, whole rounds
      return (double)((t + cus - 1) / cus) * (1.9 + (dma ? 0.06 : 0.093) * n64);
    case Tile::kWave16:
      return (double)((t + cus - 1) / cus) * (1.7 + (dma ? 0.048 : 0.07) * n64);
    default: {
      // several workgroups per CU; below one per CU the latency of a stage
      const double per_cu = t > cus ? (double)t / (double)cus : 1.0;
      const double stage = 0.04 + 0.105 * per_cu;
      return n64 * (dma || stage > 0.24 ? stage : 0.24) + 1.5 * per_cu;
    }
  }
}

void consider(Choice &best, Tile tile, const Traits &f, int64_t t, int64_t n64, int64_t cus,
              bool ranges, bool tail, double split_us, double add_us) {
  for (int64_t ns = 1;; ns += 1 + ns / 4) {
    // each range keeps at least 512 bytes of the contracted index
    if (ns > 1 && (!ranges || n64 / ns < 8 || t * ns > 3 * cus)) break;
    double us = model_us(tile, f, t * ns, (double)((n64 + ns - 1) / ns), cus,
                         tail && ns == 1);
    if (ns > 1) us += split_us + add_us * (double)ns;
    if (us < best.us) best = Choice{tile, (int)ns, us};
  }
}

// Whether K may be cut into ranges added atomically.  int32 sums are the same
// in any order; a binary32 sum is not, and is cut only from kRangesK on (as by
// tail_split, whose ranges keep as many stages): below it every product repeats
// bit for bit.  us, K in order (gemm_wave_kernel) / in ranges, f16 accumulating,
// operands not in the caches: 128 x 1024 x 128 4.4 / 4.6, 300 x 1024 x 300 at an odd
// pitch 5.7 / 6.3, 16 x 1536 x 1024 5.8 / 4.2, 192 x 2048 x 320 6.2 / 5.3, 192 x 8192
// x 320 15.8 / 9.1; whole on 64 x 64 tiles 192 x 1024 x 320 8.0, 2048 12.0.
constexpr int64_t kRangesK = 2 * kMinSplitStages * (kFastKB / 2);   // 2048
template <int DT>
constexpr bool ranges_ok(int64_t K) {
  return DT == TCU_I8_I32 || (DT != TCU_BF16_BF16 && K >= kRangesK);
}

// The ring kernel: tile and split by the model.
template <int DT>
Choice choose_ring(const RectArgs &a, bool dma, GemmPath path, int64_t cus) {
  constexpr int ES = in_bytes(DT);
  const int64_t n64 = (a.K * ES + 63) / 64;
  const double mn = (double)a.M * (double)a.N;
  const double split_us = 1.5 + (a.accum ? 0.0 : 2.5 + mn * 4e-6), add_us = mn / 1.2e6;
  Choice c;
  const bool ranges = ranges_ok<DT>(a.K);
  const Traits f = traits<DT>(a, dma);
  consider(c, Tile::k64, f, ((a.M + 63) / 64) * ((a.N + 63) / 64), n64, cus, ranges, false,
           split_us, add_us);
  if (path == GemmPath::kRing) return c;
  consider(c, Tile::k128, f, ((a.M + 127) / 128) * ((a.N + 127) / 128), n64, cus, ranges, false,
           split_us, add_us);
  if (kWaveSums<DT> && !ranges && path != GemmPath::kGeneral) {
    const int64_t tn = (a.N + kWaveN - 1) / kWaveN;
    consider(c, Tile::kWave32, f, (a.M + 31) / 32 * tn, n64, cus, false, false, 0, 0);
    consider(c, Tile::kWave16, f, (a.M + 15) / 16 * tn, n64, cus, false, false, 0, 0);
  }
  return c;
}

// Whether the ring kernel may fill its stages by DMA: 16-byte row pitches, N
// a whole number of 16-byte chunks, the per-lane 32-bit offsets in range.
template <int DT>
bool ring_dma_ok(const RectArgs &a) {
  constexpr int ES = in_bytes(DT);
  return (a.lda * ES) % 16 == 0 && (a.ldb * ES) % 16 == 0 && (a.N * ES) % 16 == 0 &&
         128 * a.lda * ES < ((int64_t)1 << 32) && 128 * a.ldb * ES < ((int64_t)1 << 32);
}

template <int DT>
hipError_t launch_ring_choice(const RectArgs &a, bool dma, const Choice &c, hipStream_t stream,
                              int num_cus, int64_t cus) {
  // Test override of the ranges (at most one per 128-byte stage).
  int ns = c.nsplit;
  const int forced = knob(TCU_KNOB_SPLIT_K);
  if (forced > 0 && DT != TCU_BF16_BF16) {
    const int64_t stages = (a.K * in_bytes(DT) + 127) / 128;
    ns = (int)(forced < stages ? forced : stages > 1 ? stages : 1);
  }
  if (c.tile == Tile::k128) {
    const int64_t t = ((a.M + 127) / 128) * ((a.N + 127) / 128);
    const int64_t n64 = (a.K * in_bytes(DT) + 63) / 64;
    bool cut = false;
    model_us(Tile::k128, traits<DT>(a, dma), t, (double)n64, cus, false, &cut);
    const int whole = (int)(cut ? t - t % (2 * cus) : t);
    return dma ? launch_ring<DT, 128, true>(a, ns, whole, stream, num_cus)
               : launch_ring<DT, 128, false>(a, ns, whole, stream, num_cus);
  }
  if constexpr (kWaveSums<DT>) {
    if (c.tile == Tile::kWave32 && forced <= 0)
      return dma ? launch_wave<DT, 32, true>(a, stream) : launch_wave<DT, 32, false>(a, stream);
    if (c.tile == Tile::kWave16 && forced <= 0)
      return dma ? launch_wave<DT, 16, true>(a, stream) : launch_wave<DT, 16, false>(a, stream);
  }
  return dma ? launch_ring<DT, 64, true>(a, ns, INT_MAX, stream, num_cus)
             : launch_ring<DT, 64, false>(a, ns, INT_MAX, stream, num_cus);
}

template <int DT>
hipError_t launch_general(const RectArgs &a, GemmPath path, hipStream_t stream, int num_cus,
                          int64_t cus) {
  const bool dma = path != GemmPath::kGeneral && ring_dma_ok<DT>(a);
  return launch_ring_choice<DT>(a, dma, choose_ring<DT>(a, dma, path, cus),
                                stream, num_cus, cus);
}

// The full-tile kernel on tm x tn tiles of C (all of it, or its 256-aligned
// interior), split nsplit ways, or its last partial round split (nsplit 1).
template <int DT, bool kEdge>
hipError_t launch_full(const RectArgs &a, int tm, int tn, int nsplit, hipStream_t stream,
                       int num_cus) {
  constexpr int ES = in_bytes(DT), OB = out_bytes(DT);
  constexpr int KE = kFastKB / ES;
  const int tiles = tm * tn;
  // Persistent grid: one workgroup per CU (the LDS ring admits one), each
  // walking tiles blockIdx, blockIdx + grid, ...  The test override
  // TCU_KNOB_PP_GRID sets the grid size instead (a tiny grid gives every
  // workgroup many tiles).
  const int want = knob(TCU_KNOB_PP_GRID) > 0 ? knob(TCU_KNOB_PP_GRID) : num_cus;
  int full = 0;
  if (nsplit > 1) {
    if (!a.accum) {
      const hipError_t e = zero_view(a, stream, num_cus);
      if (e != hipSuccess) return e;
    }
  } else {
    nsplit = tail_split<DT>(tiles, want < tiles ? want : tiles, a.K / KE, &full);
    if (nsplit > 1 && !a.accum) {
      // clipped to this launch's part of C
      const int64_t rows = a.M < 256 * (int64_t)tm ? a.M : 256 * (int64_t)tm;
      const int64_t cols = a.N < 256 * (int64_t)tn ? a.N : 256 * (int64_t)tn;
      const hipError_t e = zero_tail((unsigned char *)a.C, a.ldc * OB, tm, tn, full, (int)rows,
                                     cols * OB, stream, num_cus);
      if (e != hipSuccess) return e;
    }
  }
  const int items = full + (tiles - full) * nsplit;
  const int grid = want < items ? want : items;
  hipLaunchKernelGGL((gemm_pp_kernel<DT, kRingStages, kEdge>), dim3(grid), dim3(512), 0, stream,
                     (const unsigned char *)a.A, (const unsigned char *)a.B,
                     (unsigned char *)a.C, (int)a.K, a.lda, a.ldb, a.ldc, a.accum ? 1 : 0, tm, tn,
                     full, nsplit, (int)a.M, (int)a.N);
  return hipGetLastError();
}

template <int DT>
hipError_t launch_dt(const RectArgs &a, hipStream_t stream, int num_cus) {
  constexpr int ES = in_bytes(DT), OB = out_bytes(DT);
  constexpr int KE = kFastKB / ES;
  constexpr bool kSplit = DT != TCU_BF16_BF16;
  const GemmPath path = gemm_path();
  const int64_t cus = knob(TCU_KNOB_PP_GRID) > 0 ? knob(TCU_KNOB_PP_GRID) : num_cus;
  if (path == GemmPath::kGeneral || path == GemmPath::kRing)
    return launch_general<DT>(a, path, stream, num_cus, cus);
  // The full-tile kernel takes 16-byte pitches (per-lane 32-bit DMA offsets
  // in range):
  //   * whole 256 x 256 tiles and whole K stages;
  //   * ragged shapes with N a whole number of 16-byte chunks: its edge tiles
  //     load clamped rows and chunks and store only inside C, the contracted
  //     index's partial last stage is zero-padded;
  //   * other ragged shapes: the 256-aligned interior -- rows [0, M0) and
  //     columns [0, N0) over the whole K -- while the ring kernel takes the
  //     bottom rows [M0, M) (all columns) and the right columns [N0, N) of
  //     rows [0, M0).
  // Every output element is formed by one launch over the whole K, so a
  // bfloat16 output is rounded once.
  const bool vec = (a.lda * ES) % 16 == 0 && (a.ldb * ES) % 16 == 0 && (a.ldc * OB) % 16 == 0 &&
                   256 * a.lda * ES < ((int64_t)1 << 32) && KE * a.ldb * ES < ((int64_t)1 << 32);
  const bool whole = vec && a.M % 256 == 0 && a.N % 256 == 0 && a.K % KE == 0 && a.K > 0;
  const int64_t n64 = (a.K + KE - 1) / KE;
  if (path == GemmPath::kFast && whole) {
    const int tm = (int)(a.M / 256), tn = (int)(a.N / 256);
    // forced: the split by the override, or one range per spare CU
    int64_t ns = kSplit && tm * tn < num_cus ? (num_cus + tm * tn - 1) / (tm * tn) : 1;
    if (ns > n64 / kMinSplitStages) ns = n64 / kMinSplitStages > 1 ? n64 / kMinSplitStages : 1;
    const int forced = knob(TCU_KNOB_SPLIT_K);
    if (forced > 0 && kSplit) ns = forced < n64 ? forced : n64;
    return launch_full<DT, false>(a, tm, tn, (int)ns, stream, num_cus);
  }
  const bool dma = ring_dma_ok<DT>(a);
  Choice best = choose_ring<DT>(a, dma, path, cus);
  const int64_t M0 = a.M / 256 * 256, N0 = a.N / 256 * 256;
  const bool edges_in_kernel = (a.N * ES) % 16 == 0;
  const int64_t tm = edges_in_kernel ? (a.M + 255) / 256 : M0 / 256;
  const int64_t tn = edges_in_kernel ? (a.N + 255) / 256 : N0 / 256;
  if (vec && a.K >= KE && tm >= 1 && tn >= 1) {
    Choice full;
    const double mn = (double)a.M * (double)a.N;
    // Ranges of every tile are taken on whole tiles only, of a last round's
    // tiles on any shape (as launch_full does).
    consider(full, Tile::kFull, traits<DT>(a, true), tm * tn, n64, cus,
             whole && ranges_ok<DT>(a.K), kSplit && a.K / KE >= 2 * kMinSplitStages,
             1.5 + (a.accum ? 0.0 : 2.5 + mn * 4e-6), mn / 1.2e6);
    if (!edges_in_kernel) {
      // the strips, one launch each
      RectArgs b = a, r = a;
      b.M = a.M - M0;
      r.M = M0;
      r.N = a.N - N0;
      if (b.M > 0) full.us += 3 + choose_ring<DT>(b, false, path, cus).us;
      if (r.N > 0) full.us += 3 + choose_ring<DT>(r, false, path, cus).us;
    }
    if (full.us < best.us || path == GemmPath::kFast) best = full;
  }
  if (best.tile != Tile::kFull) return launch_ring_choice<DT>(a, dma, best, stream, num_cus, cus);
  if (whole)
    return launch_full<DT, false>(a, (int)tm, (int)tn, best.nsplit, stream, num_cus);
  hipError_t e = launch_full<DT, true>(a, (int)tm, (int)tn, 1, stream, num_cus);
  if (e != hipSuccess || edges_in_kernel) return e;
  if (a.M > M0) {
    RectArgs b = a;
    b.A = (const unsigned char *)a.A + M0 * a.lda * ES;
    b.C = (unsigned char *)a.C + M0 * a.ldc * OB;
    b.M = a.M - M0;
    e = launch_general<DT>(b, path, stream, num_cus, cus);
    if (e != hipSuccess) return e;
  }
  if (a.N > N0) {
    RectArgs r = a;
    r.B = (const unsigned char *)a.B + N0 * ES;
    r.C = (unsigned char *)a.C + N0 * OB;
    r.M = M0;
    r.N = a.N - N0;
    e = launch_general<DT>(r, path, stream, num_cus, cus);
  }
  return e;
}

}  // namespace

hipError_t launch_rect(int dtype, int s, const RectArgs &a, hipStream_t stream, int num_cus) {
  // A single contiguous strip times a single block is one native call.
  if (a.K == s && a.N == s && a.lda == s && a.ldb == s && a.ldc == s)
    return launch_tall(dtype, s, a.A, a.M, a.B, a.C, a.accum, stream, num_cus);
  switch (dtype) {
    case TCU_F16_F32: return launch_dt<TCU_F16_F32>(a, stream, num_cus);
    case TCU_BF16_F32: return launch_dt<TCU_BF16_F32>(a, stream, num_cus);
    case TCU_BF16_BF16: return launch_dt<TCU_BF16_BF16>(a, stream, num_cus);
    case TCU_I8_I32: return launch_dt<TCU_I8_I32>(a, stream, num_cus);
  }
  return hipErrorInvalidValue;
}

}  // namespace tcu

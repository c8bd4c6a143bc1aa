// FP64 product C = alpha op(A) B + beta Cin for the per-block solve
// X~ = L^-1 X and the refinement residual X - L X~ (also the setup's panel and
// trailing products and the adjoint's L-bar update): A column-major and lower
// or upper triangular (or full), B column-major (full or lower
// triangular), C column-major, optionally only the tiles that reach C's
// lower part.  The same
// v_mfma_f64_4x4x4_4b_f64 accumulation as gemm_f64_kernel with the k order
// permuted within each 16-deep stage; operands reach LDS by direct
// global-to-LDS loads into a ring of stages.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_f64.hpp"
#include "lds_dma.hpp"

namespace gls {

// Results of a tile of 128 rows (two strips wm of 64) x BN columns: lane holds
// C[4 ((lane >> 2) & 3) + (lane >> 4)][lane & 3] of each of its wave's 4 x FC
// slices of 16 x 4.  red: LDS for 2 red_q BN doubles.
// The tile's columns are j0.. of the count listed in cols.
template <int BN, int FC, int NT>
__device__ __forceinline__ void trmm_f64_epilogue(const GemmArgs& g, const double (&acc)[4][FC], double* red, int ti,
                                                  int i0, int j0, int wm, int wn, ColList cols, int count) {
  constexpr int WTN = 4 * FC;
  const int lane = threadIdx.x & 63;
  if (g.red_q > 0) {
    // Per-column sums over this tile's rows instead of C: each lane sums its four rows (a ascending), a
    // butterfly over the sixteen lanes of a column adds those (every lane ends with the same sum), and the
    // two row-strip waves are added in the order wm = 0, 1.  The order depends only on the tile, so every
    // column's sums are independent of the block's width and of the column's place in it.
    __syncthreads();   // every wave is done with the ring, which now holds the two strips' sums as red[wm][q][BN columns]
    for (int q = 0; q < g.red_q; ++q) {
      const bool norm = q == g.red_q - 1;
      double w[4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
        w[a] = norm ? 0.0 : g.red_W[(int64_t)(i0 + wm * 64 + a * 16 + 4 * ((lane >> 2) & 3) + (lane >> 4)) +
                                   (int64_t)q * g.ld_red_W];
#pragma unroll
      for (int c = 0; c < FC; ++c) {
        double t = 0.0;
#pragma unroll
        for (int a = 0; a < 4; ++a) t += acc[a][c] * (norm ? acc[a][c] : w[a]);
#pragma unroll
        for (int off = 4; off < 64; off <<= 1) t += __shfl_xor(t, off, 64);
        if (lane < 4) red[(wm * g.red_q + q) * BN + wn * WTN + c * 4 + lane] = t;
      }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < g.red_q * BN; e += NT) {
      const int q = e / BN, jl = e % BN;
      if (j0 + jl < count)
        g.red_part[(int64_t)(ti * g.red_q + q) * g.ncols + cols[j0 + jl]] =
            red[q * BN + jl] + red[(g.red_q + q) * BN + jl];
    }
    return;
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int i = i0 + wm * 64 + a * 16 + 4 * ((lane >> 2) & 3) + (lane >> 4);
    if (i >= g.mvalid) continue;
#pragma unroll
    for (int c = 0; c < FC; ++c) {
      int j = j0 + wn * WTN + c * 4 + (lane & 3);
      if (j >= count || (g.only.at && !g.only.flagged(j))) continue;
      j = cols[j];
      double val = g.alpha * acc[a][c];
      if (g.beta != 0.0 && !g.acc_cin) val += g.beta * g.Cin[(int64_t)i + (int64_t)j * g.ldcin];
      g.C[(int64_t)i + (int64_t)j * g.ldc] = val;
    }
  }
}

// 128 x 64 tiles, 16 k per stage, eight waves of 64 x 16 (two row strips x four
// column strips; each wave 4 x 4 v_mfma_f64_4x4x4_4b_f64 accumulators as in
// gemm_f64_kernel).  Permuting k saves half of the B fragment reads.  A stage
// is 16 KB of A (16 k-columns of 128 rows, one 1 KB load instruction each) and
// 8 KB of B (64 columns of 16 k, eight columns per instruction), in a ring of
// two stages.  16-byte chunks are placed so that both fragment reads are
// conflict-free: in A's k-column kc, chunk c (rows 2c, 2c + 1) sits in slot
// c ^ 8 (kc & 1); in B's column j, chunk c (k = 2c, 2c + 1) sits in slot
// c ^ (j & 7).
//
// Occupancy is what bounds this kernel: a workgroup takes 48 KB of LDS, so
// three fit on a compute unit (six waves per SIMD) only if a wave stays within
// 80 VGPRs.  The loads therefore address global memory as a scalar base plus a
// 32-bit lane offset, the B pairs are read one half-stage at a time, and the
// compiler is held to six waves per SIMD (76 VGPRs, no spills).  With 99 VGPRs
// (two workgroups per compute unit) the same instruction stream ran 6-8%
// slower at n = 10,000 and n = 20,000.
//
// With 128 x 32 tiles (eight waves of 64 x 8, 20 KB a stage) a product of few
// tiles has twice as many and its longest one ends sooner: a single workgroup
// on a compute unit takes 1.45 us a stage of 64 columns, whose MFMAs take 0.92.
constexpr int DB_BM = 128, DB_BN = 64, DB_BK = 16, DB_THREADS = 512, DB_STAGES = 2;
// Products of up to this many 128 x 64 tiles take tiles of 128 x 32: what the chip holds at once.  n = 3,325, 998
// columns (416 tiles) 331 -> 237 us a block, n = 5,000, 600 (400) 535 -> 436, n = 10,000, 300 (395) 1,432 -> 887, n = 2,000,
// 3,000 (752) 287 -> 262; beyond, A's columns are read twice as often for it: n = 5,000, 1,500 (960) 711 -> 776, 4,096
// (2,560) 1,715 -> 1,900.  Sums of up to 896 have few stages to win back and go up and down with the rounds (n = 640,
// 200, 320, 480 and 640 tiles: 0.93, 1.11, 1.08 and 1.15 of the wide tiles' time): up to 256 tiles.
inline int narrow_tiles(int K) { return K <= 896 ? 256 : 768; }

template <int BN>
__global__ __launch_bounds__(DB_THREADS) __attribute__((amdgpu_waves_per_eu(6, 8)))
void trmm_f64_dma_kernel(GemmArgs g) {
  constexpr int BM = DB_BM, BK = DB_BK, NS = DB_STAGES, NW = DB_THREADS / 64;
  constexpr int WGM = BM / 64, WTN = BN / (NW / WGM), FC = WTN / 4;
  constexpr int ASZ = BM * BK * 8, BSZ = BN * BK * 8, STAGE = ASZ + BSZ;
  constexpr int AINS = ASZ / 1024;   // load instructions of A per stage, one k-column each
  constexpr int BINS = BSZ / 1024;   // load instructions of B per stage, eight columns each
  static_assert(BM == 128 && BK == 16 && 16 * FC == BN && AINS == 2 * NW && BINS <= NW, "tile split");
  static_assert(2 * 21 * BN * 8 <= NS * STAGE, "the ring holds the fused sums (p + 1 <= 21)");
  __shared__ __align__(1024) char smem[NS * STAGE];

  int ti, tj;
  const int Mt = g.M / BM, Nt = ((g.tile_cols ? g.tile_cols : g.ncols) + BN - 1) / BN;
  if (!XcdMap::tile(g, blockIdx.x, Mt, Nt, &ti, &tj)) return;
  const int i0 = ti * BM, j0 = tj * BN;
  if (g.c_lower && (i0 + BM - 1) < (j0 + g.c_diag)) return;   // a tile wholly above the lower part
  const int count = g.cols.count(g.ncols);
  if (j0 >= count || (g.cols.at && !g.range.holds(count))) return;
  const ColList cols = g.cols.or_all(count, g.ncols);
  // k range of the tile: a lower-triangular A ends at the tile's last row, an upper-triangular one starts at its
  // first, a lower-triangular B starts at the tile's first column (each holds explicit zeros across its diagonal
  // block)
  int khi = g.K;
  if (g.a_tri == TRI_LOWER) khi = imin(khi, i0 + BM);
  const int nk = (khi + BK - 1) / BK;
  int k0 = (g.a_tri == TRI_UPPER) ? i0 / BK : 0;
  if (g.b_tri == TRI_LOWER) k0 = imax(k0, j0 / BK);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WGM, wn = wave / WGM;

  // loader: this wave issues instructions wave and wave + 8 (A's k-columns) and
  // wave + 16 (B's columns 8 wave .. 8 wave + 7, if the tile has them) of every stage
  uint32_t voff[3];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int kc = q * NW + wave;
    const int c = lane ^ ((kc & 1) << 3);
    voff[q] = (uint32_t)((2 * c + (int64_t)kc * g.lda) * 8);
  }
  {
    const int jl = 8 * wave + (lane >> 3);
    const int c = (lane & 7) ^ (jl & 7);
    const int j = imin(j0 + jl, count - 1);   // columns past the end: any valid one, dropped
    voff[2] = (uint32_t)((2 * c + (int64_t)(g.b_listed ? cols[j] - cols[j0] : j - j0) * g.ldb) * 8);
  }
  const double* Abase = g.A + i0;
  const double* Bbase = g.B + (int64_t)(g.b_listed ? cols[j0] : j0) * g.ldb;
  const uint32_t lds0 = lds_address(smem);
  auto issue = [&](int kstep) {
    const uint32_t base = lds0 + (uint32_t)((kstep % NS) * STAGE);
    const int kt = kstep * BK;
    const double* a = Abase + (int64_t)kt * g.lda;   // A advances kt columns, B kt rows
    const double* b = Bbase + kt;
    lds_load16_sv(a, voff[0], base + (uint32_t)(wave * 1024));
    lds_load16_sv(a, voff[1], base + (uint32_t)((NW + wave) * 1024));
    if (BINS == NW || wave < BINS) lds_load16_sv(b, voff[2], base + (uint32_t)(ASZ + wave * 1024));
  };

  double acc[4][FC];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < FC; ++c) acc[a][c] = 0.0;
  if (g.acc_cin) {   // start from alpha Cin (alpha = +-1: exact)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int i = i0 + wm * 64 + a * 16 + 4 * ((lane >> 2) & 3) + (lane >> 4);
#pragma unroll
      for (int c = 0; c < FC; ++c) {
        const int j = j0 + wn * WTN + c * 4 + (lane & 3);
        if (i < g.mvalid && j < g.ncols) acc[a][c] = g.alpha * g.Cin[(int64_t)i + (int64_t)j * g.ldcin];
      }
    }
  }

  // k order within a stage: MFMA s sums k = 4 (lane / 16) + s over the four lane groups (a permutation of the
  // stage's 16 k that both operands share), so a lane's four B values of a column are adjacent: two 16-byte reads
  // per column and stage instead of four 8-byte ones.  A's fragment of MFMA s, row block a sits at
  // abase + 1024 s + 128 (a ^ (s & 1)) (the chunk swizzle flips bit 0 of a on odd k).
  const int g4 = 4 * (lane >> 4);
  const int abase = g4 * (8 * BM) + wm * 512 + ((lane & 15) >> 1) * 16 + (lane & 1) * 8;

  if (k0 < nk) issue(k0);
  for (int it = k0; it < nk; ++it) {
    wait_vmcnt<0>();   // this wave's loads of stage it have landed ...
    __syncthreads();   // ... and every wave's; the other stage is free
    if (it + 1 < nk) issue(it + 1);
    const char* st = smem + (it % NS) * STAGE;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      double2 bq[FC];
#pragma unroll
      for (int c = 0; c < FC; ++c) {
        const int j = wn * WTN + c * 4 + (lane & 3);
        bq[c] = *reinterpret_cast<const double2*>(st + ASZ + j * 128 + ((((g4 >> 1) + h) ^ (j & 7)) << 4));
      }
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        const int s = 2 * h + s2;
        double af[4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
          af[a] = *reinterpret_cast<const double*>(st + abase + s * (8 * BM) + ((a ^ (s & 1)) * 128));
#pragma unroll
        for (int c = 0; c < FC; ++c) {
          const double bf = s2 ? bq[c].y : bq[c].x;
#pragma unroll
          for (int a = 0; a < 4; ++a) acc[a][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(af[a], bf, acc[a][c], 0, 0, 0);
        }
      }
    }
  }

  trmm_f64_epilogue<BN, FC, DB_THREADS>(g, acc, reinterpret_cast<double*>(smem), ti, i0, j0, wm, wn, cols, count);
}

// The same product, bitwise, for short sums and grids of few tiles: 128 x BN tiles (BN = 16 or
// 8), each wave 64 x 4, so that the tile's own MFMA time per stage (0.85 us for 64
// columns, which a lone workgroup cannot hide) falls to a quarter or less and
// there are more workgroups.  The columns of B that the tile needs are read once,
// KMAX rows at a time, into LDS through registers: any alignment, and rows past
// kvalid become zero, so no padded copy of the block is made first.  A's stages
// follow in a ring of four.  Every output sums the same k in the same order as in
// trmm_f64_dma_kernel (columns of A that it skips hold zeros).
// A block of 108 columns at n = 712 took 71 us with the other kernel and takes 32
// with this one, 48 columns at n = 1,000 91 and 40, 16,000 at n = 256 156 and 80,
// 40 columns at n = 10,000 1,432 and 373.
template <int BN, int KMAX>
__global__ __launch_bounds__(32 * BN) void trmm_f64_small_kernel(GemmArgs g) {
  constexpr int BM = DB_BM, BK = DB_BK, NS = 4, NW = BN / 2, NT = 64 * NW;
  constexpr int STAGE = BM * BK * 8, LDB = KMAX + 2, QA = BK / NW;   // load instructions per wave and stage
  static_assert(NS * STAGE + BN * LDB * 8 <= 160 * 1024 && 2 * 21 * BN * 8 <= NS * STAGE && QA * NW == BK, "LDS");
  __shared__ __align__(1024) char smem[NS * STAGE];
  __shared__ __align__(16) double Bs[BN * LDB];   // Bs[column][k - 16 b0]

  const int ti = g.map_desc ? (int)(gridDim.y - 1 - blockIdx.y) : (int)blockIdx.y, tj = blockIdx.x;
  const int i0 = ti * BM, j0 = tj * BN;
  if (g.c_lower && (i0 + BM - 1) < (j0 + g.c_diag)) return;
  const int count = g.cols.count(g.ncols);
  if (j0 >= count || (g.cols.at && !g.range.holds(count))) return;
  const ColList cols = g.cols.or_all(count, g.ncols);
  if (g.only.at) {
    int* any = reinterpret_cast<int*>(smem);
    if (threadIdx.x == 0) *any = 0;
    __syncthreads();
    if (threadIdx.x < BN && j0 + (int)threadIdx.x < g.ncols && g.only.flagged(j0 + threadIdx.x)) *any = 1;
    __syncthreads();
    const bool none = *any == 0;
    if (none) return;
    __syncthreads();   // smem is the ring from here on
  }
  int khi = g.K;
  if (g.a_tri == TRI_LOWER) khi = imin(khi, i0 + BM);
  const int nk = (khi + BK - 1) / BK;
  int k0 = (g.a_tri == TRI_UPPER) ? i0 / BK : 0;
  if (g.b_tri == TRI_LOWER) k0 = imax(k0, j0 / BK);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;

  const uint32_t lds0 = lds_address(smem);
  const uint32_t voff = 16 * lane;
  auto issue = [&](int kstep) {
    const uint32_t base = lds0 + (uint32_t)((kstep % NS) * STAGE);
    const double* a = g.A + i0 + (int64_t)kstep * BK * g.lda;
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int kc = q * NW + wave;
      lds_load16_sv(a + (int64_t)kc * g.lda, voff, base + (uint32_t)(kc * 1024));
    }
  };
  for (int q = 0; q < NS - 1; ++q)
    if (k0 + q < nk) issue(k0 + q);
  // B's rows [16 it, 16 it + KMAX) of the tile's columns, two columns a wave
  const int kend = imin(nk * BK, g.kvalid ? g.kvalid : g.K);
  auto load_b = [&](int it) {
#pragma unroll
    for (int c = wave; c < BN; c += NW) {
      const int j = j0 + c;
      const double* col = g.B + (int64_t)(g.b_listed && j < count ? cols[j] : j) * g.ldb;
      double v[KMAX / 64];
#pragma unroll
      for (int u = 0; u < KMAX / 64; ++u) {
        const int k = it * BK + lane + 64 * u;
        v[u] = (j < count && k < kend) ? col[k] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < KMAX / 64; ++u) Bs[c * LDB + lane + 64 * u] = v[u];
    }
  };

  double acc[4][1];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    acc[a][0] = 0.0;
    if (g.acc_cin) {   // start from alpha Cin (alpha = +-1: exact)
      const int i = i0 + wm * 64 + a * 16 + 4 * ((lane >> 2) & 3) + (lane >> 4), j = j0 + wn * 4 + (lane & 3);
      if (i < g.mvalid && j < g.ncols) acc[a][0] = g.alpha * g.Cin[(int64_t)i + (int64_t)j * g.ldcin];
    }
  }
  const int g4 = 4 * (lane >> 4);
  const int abase = g4 * 1024 + wm * 512 + (lane & 15) * 8;
  const double* bcol = Bs + (wn * 4 + (lane & 3)) * LDB + g4;
  int b0 = k0;   // first stage of the rows of B in LDS
  for (int it = k0; it < nk; ++it) {
    if (it == k0 || it - b0 == KMAX / BK) {
      __syncthreads();   // every wave is done with the last rows
      load_b(it);
      b0 = it;
    }
    wait_stages<QA>(imin(nk - 1 - it, NS - 2));   // this wave's loads of stage it have landed ...
    __syncthreads();                              // ... and every wave's (and B); stage (it - 1) % NS is free
    if (it + NS - 1 < nk) issue(it + NS - 1);
    const char* st = smem + (it % NS) * STAGE + abase;
    const double2 b01 = *reinterpret_cast<const double2*>(bcol + (it - b0) * BK);
    const double2 b23 = *reinterpret_cast<const double2*>(bcol + (it - b0) * BK + 2);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double bf = s == 0 ? b01.x : s == 1 ? b01.y : s == 2 ? b23.x : b23.y;
#pragma unroll
      for (int a = 0; a < 4; ++a)
        acc[a][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(*reinterpret_cast<const double*>(st + s * 1024 + a * 128), bf,
                                                       acc[a][0], 0, 0, 0);
    }
  }
  trmm_f64_epilogue<BN, 1, NT>(g, acc, reinterpret_cast<double*>(smem), ti, i0, j0, wm, wn, cols, count);
}

// Whether a product of M rows, ncols columns and K goes to it.  Short sums over
// few rows do whatever the number of columns: the other kernel's start and end
// are most of its time there (n = 512, 16,000 columns: 306 us against 257; n =
// 128, 30,000: 176 against 64).  Longer ones do while there are few tiles of
// 128 x 64, so that the other kernel's time is that of its longest one, which sets
// the line by the length of the sum.  Blocks of fractional SNPs, the time with this
// kernel over that with tiles of 128 x 32 (n: tiles ratio ...):
//   640: 95 0.80, 125 0.98, 140 1.13;  800: 63 1.00, 91 1.35;  1,024: 64 0.85, 96 1.21
//   (sums of 513 to 1,024 take 8 columns a tile);  1,152: 126 1.02, 144 1.18, 180 0.86,
//   234 1.07;  1,280: 120 0.96, 160 1.28, 200 0.90, 240 1.06;  2,048: 128 0.92, 160 1.22;
//   3,072: 144 0.93, 168 1.10;  4,096: 160 0.98, 192 1.12;  6,144: 192 0.89, 240 1.03;
//   8,192: 256 0.90, 320 1.15;  10,240: 240 0.78, 320 1.04.
// (Between 160 and 208 tiles at 1,152 to 1,280 it would be ahead again, for the other
// kernel's second round; 1% of a study of 10,000 samples, whose setup has such products.)
inline int small_tiles(int K) {
  return K <= 640 ? 128 : K <= 1024 ? 64 : K <= 4096 ? 128 : K <= 6144 ? 192 : K <= 8192 ? 256 : 320;
}
inline bool small_product(int M, int ncols, int K) {
  if (K <= 512 && M <= 512) return true;
  return (int64_t)((M + DB_BM - 1) / DB_BM) * ((ncols + DB_BN - 1) / DB_BN) <= small_tiles(K);
}

// Columns that a tile's lane offsets into B span: 64 adjacent ones, or with a list any of the block.
inline int64_t dma_b_span(int ncols, bool listed) { return listed ? ncols - 1 : 63; }

// Whether the two kernels above apply to a product without transposes: A
// full, lower or upper triangular, B full or lower triangular (diagonal offsets 0),
// 16-byte aligned operands with even leading dimensions,
// K a multiple of 16, the rows of A up to M rounded up to 128 inside A's
// leading dimension (they are read; rows past M are not stored), and lane
// offsets within a stage (15 columns of A, a tile's columns of B) below 2^32 bytes.
inline bool trmm_dma_ok(const GemmArgs& g) {
  auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  const bool small = small_product(g.M, g.ncols, g.K);   // takes any B
  if (!al16(g.A) || (g.lda & 1) || (!small && (!al16(g.B) || (g.ldb & 1) || g.kvalid))) return false;
  if (g.b_tri == TRI_UPPER || (g.b_tri == TRI_LOWER && g.b_diag != 0) || g.a_diag != 0) return false;
  if (g.M <= 0 || g.K % DB_BK || g.K <= 0 || g.ncols <= 0 || g.mvalid > g.M) return false;
  if (g.lda < (int64_t)(g.M + DB_BM - 1) / DB_BM * DB_BM || g.ldb < (g.kvalid ? g.kvalid : g.K)) return false;
  if (small) return true;
  if ((15 * g.lda + DB_BM) * 8 >= ((int64_t)1 << 32) || (dma_b_span(g.ncols, g.b_listed) * g.ldb + DB_BK) * 8 >= ((int64_t)1 << 32))
    return false;
  return true;
}

// Whether a column-major B operand with K rows can feed trmm_f64_dma_kernel
// as it is (otherwise it is first copied into a buffer of that shape).
inline bool dma_b_operand_ok(const double* B, int64_t ldb, int64_t K, int ncols, bool listed) {
  return ((uintptr_t)B & 15) == 0 && (ldb & 1) == 0 && K % DB_BK == 0 && ldb >= K &&
         (dma_b_span(ncols, listed) * ldb + DB_BK) * 8 < ((int64_t)1 << 32);
}

}  // namespace gls

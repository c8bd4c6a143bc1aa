// Setup-phase kernels: forming M, the in-LDS factorization and inversion of
// the diagonal blocks, packing, and the small Gram matrix of [X~_L | y~].
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gls {

// Leaf (diagonal block) size of the blocked Cholesky / inversion.
constexpr int NB_LEAF = 128;

// L <- M = h2 * Phi + (1 - h2) * I in the lower triangle of the leading n x n
// block (read from Phi's lower triangle), identity on the padding rows
// n..N-1, and zeros above the diagonal within its diagonal blocks of NB_LEAF;
// Li <- zeros in its diagonal blocks, and the identity in rows r0..N-1 (past the
// factored blocks); info <- 0.  N x N column-major, ld = N.  Nothing reads L or
// L^-1 above the diagonal blocks, and the factorization writes every block of
// L^-1 below them, so the rest is left as it is (N = 10,240: two kernels that
// wrote both matrices in full took 350 us, this one 150 us).
// One column per workgroup in turn, so that a thread's index needs no division.
// With sc, M[i, j] is scaled by sc[i] sc[j] (powers of two).
__global__ __launch_bounds__(256) void setup_init_kernel(double* __restrict__ L, double* __restrict__ Li, int N, int n,
                                                         int r0, const double* __restrict__ Phi, int64_t ld_phi,
                                                         double h2, const double* __restrict__ sc,
                                                         int* __restrict__ info) {
  if (blockIdx.x == 0 && threadIdx.x < 2) info[threadIdx.x] = 0;
  for (int j = blockIdx.x; j < N; j += gridDim.x) {
    double2* Lc = reinterpret_cast<double2*>(L + (int64_t)j * N);
    double* Ic = Li + (int64_t)j * N;
    const double* Pc = Phi + (int64_t)j * ld_phi;
    const int d0 = j / NB_LEAF * NB_LEAF;   // first row of the column's diagonal block
    const double sj = sc ? sc[j] : 1.0;
#pragma unroll 4
    for (int r = d0 / 2 + threadIdx.x; r < N / 2; r += 256) {
      double v[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k = 2 * r + u;
        v[u] = 0.0;
        if (k >= j) {
          if (k < n) v[u] = h2 * Pc[k] + (k == j ? (1.0 - h2) : 0.0);
          else if (k == j) v[u] = 1.0;
          if (sc) v[u] *= sc[k] * sj;
        }
      }
      Lc[r] = double2{v[0], v[1]};
    }
    if (threadIdx.x < NB_LEAF) Ic[d0 + threadIdx.x] = 0.0;
    __syncthreads();   // the padding's ones come after its zeros
    for (int i = r0 + threadIdx.x; i < N; i += 256) Ic[i] = (i == j) ? 1.0 : 0.0;
  }
}

// Powers of two that bring M's diagonal into [1/2, 2]: sc[i] = 2^-e with
// M[i, i] 4^-e there, and *any = 1 if one of them is not 1 (set to 0 before the
// launch).  A product formed by residues rounds its operands at a
// fraction of their row's norm, which is harmless against an error bound like
// that of the Cholesky factorization, sqrt(M_ii M_jj) 2^-53 per entry, only where
// the rows of M are of one scale.
__global__ void diagonal_scale_kernel(const double* __restrict__ Phi, int64_t ld_phi, int n, int N, double h2,
                                      double* __restrict__ sc, double* __restrict__ any) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const double d = i < n ? h2 * Phi[(int64_t)i * (ld_phi + 1)] + (1.0 - h2) : 1.0;
  int e = 0;
  if (d > 0.0 && d < __builtin_inf() && !(d >= 0.5 && d <= 2.0)) {
    frexp(d, &e);   // d 2^-e in [1/2, 1)
    e = e >= 0 ? e / 2 : -((1 - e) / 2);
  }
  sc[i] = ldexp(1.0, -e);
  if (e != 0) *any = 1.0;
}

// The factor and its inverse of M from those of the scaled matrix: L[i, j] /= sc[i], Li[i, j] *= sc[j] (lower parts).
__global__ __launch_bounds__(256) void unscale_factor_kernel(double* __restrict__ L, double* __restrict__ Li, int N,
                                                             const double* __restrict__ sc,
                                                             const double* __restrict__ any) {
  if (*any == 0.0) return;
  for (int j = blockIdx.x; j < N; j += gridDim.x) {
    const double sj = sc[j];
    for (int i = j + threadIdx.x; i < N; i += 256) {
      L[(int64_t)i + (int64_t)j * N] /= sc[i];
      Li[(int64_t)i + (int64_t)j * N] *= sj;
    }
  }
}

__global__ void fill_kernel(double* __restrict__ p, int64_t count, double v) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; idx < count; idx += (int64_t)gridDim.x * blockDim.x) p[idx] = v;
}

// dst (rows x cols, ld_dst) <- src (rows x cols, ld_src)
__global__ void copy2d_kernel(double* __restrict__ dst, int64_t ld_dst,
                              const double* __restrict__ src, int64_t ld_src, int rows, int cols) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t total = (int64_t)rows * cols;
  for (; idx < total; idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx % rows);
    int j = (int)(idx / rows);
    dst[(int64_t)i + (int64_t)j * ld_dst] = src[(int64_t)i + (int64_t)j * ld_src];
  }
}

// dst (cols x rows, ld_dst) <- src^T for src (rows x cols, ld_src), through
// 32 x 32 LDS tiles so that both the reads and the writes are column runs.
__global__ __launch_bounds__(256) void transpose_kernel(double* __restrict__ dst, int64_t ld_dst,
                                                        const double* __restrict__ src, int64_t ld_src, int rows,
                                                        int cols) {
  __shared__ double tile[32][33];
  const int r0 = blockIdx.x * 32, c0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  double v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = r0 + tx, c = c0 + ty + 8 * q;
    v[q] = (r < rows && c < cols) ? src[(int64_t)r + (int64_t)c * ld_src] : 0.0;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) tile[ty + 8 * q][tx] = v[q];   // tile[c - c0][r - r0]
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = c0 + tx, r = r0 + ty + 8 * q;               // dst row c, column r
    if (r < rows && c < cols) dst[(int64_t)c + (int64_t)r * ld_dst] = tile[tx][ty + 8 * q];
  }
}

// W = L^-1 V for the thin covariate block V = [X_L | y] (n x P) and the
// lower-triangular inverse factor (N x N, ld N): a matrix-vector-shaped
// product bound by reading L^-1's lower triangle once, so it runs split over
// k on the vector units.  Workgroup (r, s) takes rows 64 r .. 64 r + 63 and
// k in [TA_KC s, TA_KC s + TA_KC), clipped to k <= row; each wave walks every
// fourth k, so a wave's loads are one 512-byte column segment.  Partial sums
// go to part[s] (N x P, ld N); chunks entirely above a row tile are skipped,
// and tri_apply_sum_kernel adds, in chunk order, exactly the chunks that
// reach each row tile.
constexpr int TA_KC = 256;

template <int P>
__global__ __launch_bounds__(256) void tri_apply_partial_kernel(const double* __restrict__ Li, int N, int n,
                                                                const double* __restrict__ XL, int64_t ld_xl,
                                                                const double* __restrict__ y,
                                                                double* __restrict__ part) {
  __shared__ double v[TA_KC * P];       // v[kk * P + j] = V[k0 + kk][j]; then the group sums
  const int i0 = blockIdx.x * 64, s = blockIdx.y, k0 = s * TA_KC;
  if (k0 > i0 + 63) return;
  const int t = threadIdx.x, r = t & 63, g = t >> 6;
  static_assert(TA_KC == 256, "one staged k per thread and column");
  {
    double x[P];
#pragma unroll
    for (int j = 0; j < P; ++j)
      x[j] = (k0 + t >= n) ? 0.0 : (j < P - 1) ? XL[(int64_t)(k0 + t) + (int64_t)j * ld_xl] : y[k0 + t];
#pragma unroll
    for (int j = 0; j < P; ++j) v[t * P + j] = x[j];
  }
  __syncthreads();
  const int i = i0 + r;
  const int kend = min(min(k0 + TA_KC, i0 + 64), N);
  double acc[P];
#pragma unroll
  for (int j = 0; j < P; ++j) acc[j] = 0.0;
  // eight loads in flight per thread, then their products
  for (int kb = k0 + g; kb < kend; kb += 32) {
    double a[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = kb + 4 * u;
      a[u] = (k < kend && k <= i) ? Li[(int64_t)i + (int64_t)k * N] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int kk = kb + 4 * u - k0;
      if (kb + 4 * u < kend) {
#pragma unroll
        for (int j = 0; j < P; ++j) acc[j] = fma(a[u], v[kk * P + j], acc[j]);
      }
    }
  }
  __syncthreads();   // v is reused for the four groups' sums
#pragma unroll
  for (int j = 0; j < P; ++j) v[(g * 64 + r) * P + j] = acc[j];
  __syncthreads();
  if (g == 0) {
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const double x = ((acc[j] + v[(64 + r) * P + j]) + v[(128 + r) * P + j]) + v[(192 + r) * P + j];
      part[(int64_t)s * N * P + (int64_t)j * N + i] = x;
    }
  }
}

// Row-wise sums of the chunks that reach a row tile.
__device__ __forceinline__ double tri_apply_row(const double* __restrict__ part, int64_t total, int64_t idx, int i) {
  const int last = (i / 64 * 64 + 63) / TA_KC;   // chunks s <= last reach row tile i / 64
  double x = 0.0;
  for (int s = 0; s <= last; ++s) x += part[(int64_t)s * total + idx];
  return x;
}

__global__ void tri_apply_sum_kernel(const double* __restrict__ part, int N, int P, double* __restrict__ W) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)N * P;
  for (; idx < total; idx += (int64_t)gridDim.x * blockDim.x) {
    W[idx] = tri_apply_row(part, total, idx, (int)(idx % N));
  }
}

// 1 / sqrt(d) to full double precision: the hardware estimate (relative error
// below 2^-22) and one third-order step, r (1 + e / 2 + 3 e^2 / 8) with
// e = 1 - d r^2.  (A dependent FP64 fma takes 20 cycles, a multiplication or
// addition 8: one such step is shorter than two of Newton's.)
__device__ __forceinline__ double fast_rsqrt(double d) {
  const double r = __builtin_amdgcn_rsq(d);
  const double e = __builtin_fma(-(d * r), r, 1.0);
  return __builtin_fma(r * e, 0.375 * e + 0.5, r);
}

// The value that lane k of the wave holds, in scalar registers.
__device__ __forceinline__ double lane_value(double x, int k) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), k), hi = __builtin_amdgcn_readlane(__double2hiint(x), k);
  return __hiloint2double(hi, lo);
}

// One diagonal block of the blocked factorization, entirely on chip.
//
// The lower triangle of the NB_LEAF x NB_LEAF block (128 x 128 doubles) sits in
// LDS as 8 x 8 blocks of 16 x 16 and is factored panel by panel (16 columns); the
// inverse is formed row block by row block behind it.
//   Panel p: up to three waves, each with the 16 rows of the diagonal block in
//     lanes 0..15 (factored by every wave alike, so none waits for another; the
//     first wave stores them once all have loaded them) and
//     48 of the rows below in the others, a row's 16 values in registers.  Step j
//     scales column j by 1 / sqrt(pivot) and subtracts its products with
//     L[k][j], read from lane k.  Rows 128..143 of each panel are the identity's:
//     against the block they become L_pp^-T, the inverse of the diagonal block.
//   Look-ahead: all waves update block column p + 1 with panel p.
//   Then the panel waves factor panel p + 1 while the others update the block
//     columns after it and form row block p of the inverse,
//       X[p][j] = -X[p][p] sum_{k=j..p-1} L[p][k] X[k][j]   (j < p),
//     on v_mfma_f64_16x16x4f64, whose accumulator layout is its B operand's, so the
//     sum goes into the last product without leaving the registers.
// Finished blocks are written to A (with zeros above the diagonal) and Ainv
// (which holds them already; ld) at once.  A non-positive or NaN pivot sets *info = row0 + j + 1 if
// *info is still 0 (the 1-based global pivot; blocks run in order, so the first
// failure wins).
//
// The chain of 128 pivots bounds it: 27 us a block (54 us with one wave per
// diagonal block exchanging columns through LDS, a separate solve of the rows
// below and the inverse formed afterwards).  A panel takes 2 us, about 250 cycles
// a pivot for some 50 instructions; the first loads take 3 us.

typedef double l4_t __attribute__((ext_vector_type(4)));

constexpr int LT = 16;                 // inner block size
constexpr int LNB = NB_LEAF / LT;      // inner blocks per side
constexpr int LROWS = NB_LEAF + LT;    // the block's rows and the identity's
constexpr int LD = LROWS + 1;          // LDS column stride: odd, so 16 lanes reading along a row hit 16 banks
constexpr int LPR = 64 - LT;           // rows below the diagonal block per panel wave
static_assert(NB_LEAF % LT == 0 && LNB == 8, "eight waves share the look-ahead blocks");

__device__ __forceinline__ double* leaf_blk(double* S, int bi, int bj) { return S + (LT * bj) * LD + LT * bi; }

// acc += op(A) op(B) for 16 x 16 blocks on v_mfma_f64_16x16x4f64.  A element
// (r, k) at pa[r * ars + k * aks], B element (k, c) at pb[k * bks + c * bcs];
// neg negates A.  Lane l supplies A[l % 16][4 s + l / 16] and
// B[4 s + l / 16][l % 16]; the accumulator holds D[l / 16 + 4 t][l % 16].
__device__ __forceinline__ void leaf_mma16(l4_t& acc, const double* pa, int ars, int aks, const double* pb, int bks,
                                           int bcs, bool neg, int lane) {
  const int r = lane & 15, q = lane >> 4;
  double a[4], b[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    a[s] = pa[r * ars + (4 * s + q) * aks];
    b[s] = pb[(4 * s + q) * bks + r * bcs];
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(neg ? -a[s] : a[s], b[s], acc, 0, 0, 0);
}
__device__ __forceinline__ l4_t leaf_ld_acc(const double* p, int lane) {
  const int c = lane & 15, q = lane >> 4;
  return l4_t{p[q + c * LD], p[q + 4 + c * LD], p[q + 8 + c * LD], p[q + 12 + c * LD]};
}
__device__ __forceinline__ void leaf_st_acc(double* p, l4_t v, int lane) {
  const int c = lane & 15, q = lane >> 4;
  p[q + c * LD] = v[0];
  p[q + 4 + c * LD] = v[1];
  p[q + 8 + c * LD] = v[2];
  p[q + 12 + c * LD] = v[3];
}

// Panel waves that panel p needs for its rows below the diagonal block.
__device__ __forceinline__ int leaf_panel_waves(int p) { return (LROWS - LT * (p + 1) + LPR - 1) / LPR; }

// Panel p by wave `wave` of its panel waves: its rows below the diagonal block
// are stored.  The block's own rows, in lanes 0..15 of every panel wave, stay in
// x, their pivots in own: another wave may only now be loading them from LDS, so
// they are stored by leaf_store_diag, past the next barrier.  Returns the first
// non-positive pivot (1-based within the leaf) or 0.
__device__ __forceinline__ int leaf_panel(double* S, int p, int wave, int lane, double (&x)[LT], double& own) {
  const int row = LT * p + (lane < LT ? lane : lane + LPR * wave);   // past the last row: a spare one, not stored
  double* P = S + (LT * p) * LD + min(row, LROWS);
#pragma unroll
  for (int k = 0; k < LT; ++k) x[k] = P[k * LD];
  double d = lane_value(x[0], 0);   // the pivot; lane j keeps its own
  own = 0.0;
#pragma unroll
  for (int j = 0; j < LT; ++j) {
    own = (lane == j) ? d : own;
    const double r = fast_rsqrt(d);
    // the next pivot from this column before it is scaled, so that its root does not wait for the column
    if (j + 1 < LT) {
      const double a = lane_value(x[j], j + 1) * r;
      d = __builtin_fma(-a, a, lane_value(x[j + 1], j + 1));
    }
    x[j] *= r;
    // five lane reads, then their five products: a product right behind its read waits for it
#pragma unroll
    for (int k0 = j + 1; k0 < LT; k0 += 5) {
      double l[5];
#pragma unroll
      for (int u = 0; u < 5; ++u) l[u] = lane_value(x[j], k0 + u < LT ? k0 + u : LT - 1);
      asm volatile("" ::"s"(l[0]), "s"(l[1]), "s"(l[2]), "s"(l[3]), "s"(l[4]));
#pragma unroll
      for (int u = 0; u < 5; ++u) {
        if (k0 + u >= LT) break;
        x[k0 + u] = __builtin_fma(-x[j], l[u], x[k0 + u]);
        asm volatile("" : "+v"(x[k0 + u]));   // formed here: put off to its use, it would hold its l in scalar registers
      }
    }
  }
  const unsigned bads = (unsigned)__ballot(!(own > 0.0)) & 0xffffu;
  const int bad = bads ? LT * p + __ffs(bads) : 0;
  if (lane >= LT && row < LROWS) {
#pragma unroll
    for (int k = 0; k < LT; ++k) P[k * LD] = x[k];
  }
  return bad;
}

// Panel p's diagonal block, by one of its panel waves (its upper triangle is not read again).
__device__ __forceinline__ void leaf_store_diag(double* S, int p, int lane, const double (&x)[LT], double own) {
  if (lane >= LT) return;
  double* P = S + (LT * p) * LD + LT * p + lane;
#pragma unroll
  for (int k = 0; k < LT; ++k) P[k * LD] = x[k];
  P[lane * LD] = sqrt(own);
}

// What waves other than the panel's do once panel p is final (wave w of n):
// the trailing update of block columns p + 2.., row block p of the inverse, and
// the stores of both results.
__device__ __forceinline__ void leaf_behind(double* S, double* A, double* Ainv, int64_t ld, int p, int w, int n,
                                            int lane) {
  const int c16 = lane & 15, q = lane >> 4;
  const int nb = LNB - 2 - p;   // block columns left to update
  const int tasks = p + (nb > 0 ? nb * (nb + 1) / 2 : 0);
  for (int task = w; task < tasks; task += n) {
    if (task < p) {   // X[p][j], the longest sum first
      const int j = task;
      l4_t acc = {0.0, 0.0, 0.0, 0.0};
      leaf_mma16(acc, leaf_blk(S, p, j), 1, LD, leaf_blk(S, LNB, j), LD, 1, false, lane);
      for (int k = j + 1; k < p; ++k) leaf_mma16(acc, leaf_blk(S, p, k), 1, LD, leaf_blk(S, j, k), 1, LD, false, lane);
      l4_t x = {0.0, 0.0, 0.0, 0.0};
      const double* D = leaf_blk(S, LNB, p) + c16 * LD;   // row c16 of X[p][p]
#pragma unroll
      for (int s = 0; s < 4; ++s)
        x = __builtin_amdgcn_mfma_f64_16x16x4f64(-D[4 * s + q], acc[s], x, 0, 0, 0);
      leaf_st_acc(leaf_blk(S, j, p), x, lane);   // kept above the diagonal, where the factor has nothing
      double* o = Ainv + (LT * p + q) + (int64_t)(LT * j + c16) * ld;
#pragma unroll
      for (int t = 0; t < 4; ++t) o[4 * t] = x[t];
    } else {          // A[i][c] -= L[i][p] L[c][p]^T
      int c = 0, rem = task - p;
      while (rem >= nb - c) {
        rem -= nb - c;
        ++c;
      }
      const int bc = p + 2 + c, bi = bc + rem;
      double* C = leaf_blk(S, bi, bc);
      l4_t acc = leaf_ld_acc(C, lane);
      leaf_mma16(acc, leaf_blk(S, bi, p), 1, LD, leaf_blk(S, bc, p), LD, 1, true, lane);
      leaf_st_acc(C, acc, lane);
    }
  }
  // block column p of the factor (zeros above its diagonal), the inverse's diagonal block
  for (int c = w; c < LT; c += n) {
    const int col = LT * p + c;
    for (int r = lane; r < NB_LEAF; r += 64) A[(int64_t)r + (int64_t)col * ld] = (r >= col) ? S[r + col * LD] : 0.0;
    if (lane >= c && lane < LT) Ainv[(int64_t)(LT * p + lane) + (int64_t)col * ld] = S[NB_LEAF + c + (LT * p + lane) * LD];
  }
}

__global__ __launch_bounds__(512) void leaf_potrf_trtri_kernel(double* __restrict__ A, double* __restrict__ Ainv,
                                                               int64_t ld, int row0, int* __restrict__ info) {
  __shared__ __align__(16) double S[NB_LEAF * LD];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  {  // all loads first, then the LDS stores: one memory latency instead of one per element
    constexpr int PER = NB_LEAF * NB_LEAF / 512;
    static_assert(512 % NB_LEAF == 0, "a thread keeps its row");
    const int r = t % NB_LEAF, c0 = t / NB_LEAF;
    double v[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int c = c0 + q * (512 / NB_LEAF);
      v[q] = (r >= c / LT * LT) ? A[(int64_t)r + (int64_t)c * ld] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int c = c0 + q * (512 / NB_LEAF);
      if (r >= c / LT * LT) S[r + c * LD] = v[q];
    }
    for (int f = t; f < LT * NB_LEAF; f += 512) {
      const int e = f % LT, c = f / LT;
      S[NB_LEAF + e + c * LD] = (e == c % LT) ? 1.0 : 0.0;
    }
  }
  __syncthreads();
  int bad = 0;   // meaningful in wave 0
  double x[LT], own = 0.0;   // a panel wave's values of its last panel
#pragma unroll
  for (int k = 0; k < LT; ++k) x[k] = 0.0;
  if (wave < leaf_panel_waves(0)) bad = leaf_panel(S, 0, wave, lane, x, own);
  __syncthreads();
  for (int p = 0; p < LNB - 1; ++p) {
    if (wave == 0) leaf_store_diag(S, p, lane, x, own);   // read from the next barrier on
    const int bi = p + 1 + wave;
    if (bi < LNB) {   // A[i][p + 1] -= L[i][p] L[p + 1][p]^T
      double* C = leaf_blk(S, bi, p + 1);
      l4_t acc = leaf_ld_acc(C, lane);
      leaf_mma16(acc, leaf_blk(S, bi, p), 1, LD, leaf_blk(S, p + 1, p), LD, 1, true, lane);
      leaf_st_acc(C, acc, lane);
    }
    __syncthreads();
    const int np = leaf_panel_waves(p + 1);
    if (wave < np) {
      const int b = leaf_panel(S, p + 1, wave, lane, x, own);
      if (bad == 0) bad = b;
    } else {
      leaf_behind(S, A, Ainv, ld, p, wave - np, LNB - np, lane);
    }
    __syncthreads();
  }
  if (wave == 0) leaf_store_diag(S, LNB - 1, lane, x, own);
  __syncthreads();
  leaf_behind(S, A, Ainv, ld, LNB - 1, wave, LNB, lane);
  if (wave == 0 && lane == 0 && bad != 0 && *info == 0) *info = row0 + bad;
}

// Strips of a product with a triangular inverse, in place: S <- alpha Li S for
// the w x w lower-triangular Li (column-major, ld) and a w x 16 strip S per
// workgroup, either columns of a column-major matrix (ROWS false) or rows of one
// (ROWS true: S^T <- alpha S^T Li^T).  The strip sits in LDS; each of the eight
// waves forms 16-row blocks of the result, Li's fragments read straight from
// memory sixteen k steps ahead.  For the small nodes of the factorization, whose
// products have few tiles and are bound by latency: in place there is no copy of
// the operand, and a node of 128 columns has w / 16 workgroups that each wait for
// memory twice, instead of four that walked eight k stages.  A node of 128 rows
// and columns: 7 us for each strip product and 10 us for the other two in one
// launch, where a copy and four 64 x 64-tile products took 65 us.  With 256
// threads a workgroup a study of 10,000 samples took 1 ms longer.
template <int W, bool ROWS>
__global__ __launch_bounds__(512) void tri_strip_kernel(const double* __restrict__ Li, int64_t ld, double* Sg, int w,
                                                        double alpha) {
  constexpr int NB = 16, PF = 16, LS = NB + 1;
  __shared__ double Ss[W * LS];   // Ss[k * LS + c]
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int c16 = lane & 15, q = lane >> 4;
  double* Sb = ROWS ? Sg + blockIdx.x * NB : Sg + (int64_t)blockIdx.x * NB * ld;
  if (ROWS) {   // 16 consecutive rows of each column
    double v[W / 32];
#pragma unroll
    for (int u = 0; u < W / 32; ++u) {
      const int k = (t >> 4) + 32 * u;
      v[u] = (k < w) ? Sb[(t & 15) + (int64_t)k * ld] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < W / 32; ++u) {
      const int k = (t >> 4) + 32 * u;
      if (k < w) Ss[k * LS + (t & 15)] = v[u];
    }
  } else {      // columns, w long
    for (int c = wave; c < NB; c += 8) {
      double v[W / 64];
#pragma unroll
      for (int u = 0; u < W / 64; ++u) {
        const int k = lane + 64 * u;
        v[u] = (k < w) ? Sb[k + (int64_t)c * ld] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < W / 64; ++u) {
        const int k = lane + 64 * u;
        if (k < w) Ss[k * LS + c] = v[u];
      }
    }
  }
  __syncthreads();
  const int nb = w / 16;   // a multiple of eight
  for (int u = 0; u < nb / 8; ++u) {
    const int b = (u & 1) ? u * 8 + 7 - wave : u * 8 + wave;   // snake: the sums get longer with b
    const double* Lr = Li + 16 * b + c16;   // A element (r, k) at Lr[k ld]
    const int steps = 4 * (b + 1);          // k < 16 (b + 1), four a step
    l4_t acc = {0.0, 0.0, 0.0, 0.0};
    double a[PF], an[PF];
#pragma unroll
    for (int f = 0; f < PF; ++f) a[f] = (f < steps) ? Lr[(int64_t)(4 * f + q) * ld] : 0.0;
    for (int s0 = 0; s0 < steps; s0 += PF) {
#pragma unroll
      for (int f = 0; f < PF; ++f) an[f] = (s0 + PF + f < steps) ? Lr[(int64_t)(4 * (s0 + PF + f) + q) * ld] : 0.0;
#pragma unroll
      for (int f = 0; f < PF; ++f)
        if (s0 + f < steps)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[f], Ss[(4 * (s0 + f) + q) * LS + c16], acc, 0, 0, 0);
#pragma unroll
      for (int f = 0; f < PF; ++f) a[f] = an[f];
    }
    // the strip's values are all in LDS: the result may overwrite them in memory
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = 16 * b + q + 4 * e;
      Sb[ROWS ? c16 + (int64_t)k * ld : k + (int64_t)c16 * ld] = alpha * acc[e];
    }
  }
}

// G[j][k] = sum_r W[r][j] * W[r][k] for j >= k (p x p, both triangles written);
// one workgroup per (j, k) pair, fixed-order tree reduction.
__global__ __launch_bounds__(256) void gram_kernel(const double* __restrict__ W, int N, int p, double* __restrict__ G) {
  __shared__ double red[256];
  int pair = blockIdx.x;
  int j = 0;
  while ((j + 1) * (j + 2) / 2 <= pair) ++j;
  int k = pair - j * (j + 1) / 2;
  double s = 0.0;
  const double* wj = W + (int64_t)j * N;
  const double* wk = W + (int64_t)k * N;
  for (int r = threadIdx.x; r < N; r += 256) s += wj[r] * wk[r];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    G[j + k * p] = red[0];
    G[k + j * p] = red[0];
  }
}

// Layout of the small per-study constants used by the per-SNP solve.
//   Lt  : q x q lower Cholesky factor of S_TL (q = p - 1), column-major
//   zT  : q      Lt^-1 r~_T
//   c   : 1      y~^T y~
//   qres: 1      c - zT^T zT   (residual of y~ on X~_L)
struct SmallLayout {
  static __host__ __device__ int Lt(int) { return 0; }
  static __host__ __device__ int zT(int p) { return (p - 1) * (p - 1); }
  static __host__ __device__ int c(int p) { return (p - 1) * (p - 1) + (p - 1); }
  static __host__ __device__ int qres(int p) { return c(p) + 1; }
  static __host__ __device__ int size(int p) { return qres(p) + 1; }
};

// Relative pivot floor of the covariate factorization: X_L counts as rank
// deficient when a squared pivot of S_TL falls to 2^-40 of its diagonal entry
// or below (exactly collinear covariates leave a rounding residual of either
// sign, about 1e-16 of it).
constexpr double RANK_REL = 9.094947017729282e-13;  // 2^-40

// Single-thread factorization of S_TL = G[0:q, 0:q] and the hoisted
// right-hand side.  Sets *info_rank = j + 1 for the first pivot at or below
// the floor.
__device__ inline void small_factor(const double* G, int p, double* __restrict__ small, int* __restrict__ info_rank) {
  const int q = p - 1;
  double* Lt = small + SmallLayout::Lt(p);
  double* zT = small + SmallLayout::zT(p);
  for (int j = 0; j < q; ++j) {
    double d = G[j + j * p];
    for (int k = 0; k < j; ++k) d -= Lt[j + k * q] * Lt[j + k * q];
    if (!(d > RANK_REL * G[j + j * p]) && *info_rank == 0) *info_rank = j + 1;
    d = sqrt(d);
    Lt[j + j * q] = d;
    for (int i = j + 1; i < q; ++i) {
      double s = G[i + j * p];
      for (int k = 0; k < j; ++k) s -= Lt[i + k * q] * Lt[j + k * q];
      Lt[i + j * q] = s / d;
    }
    for (int i = 0; i < j; ++i) Lt[i + j * q] = 0.0;
  }
  double zz = 0.0;
  for (int j = 0; j < q; ++j) {
    double s = G[j + q * p];
    for (int k = 0; k < j; ++k) s -= Lt[j + k * q] * zT[k];
    zT[j] = s / Lt[j + j * q];
    zz += zT[j] * zT[j];
  }
  const double c = G[q + q * p];
  small[SmallLayout::c(p)] = c;
  small[SmallLayout::qres(p)] = c - zz;
}

__global__ void small_factor_kernel(const double* __restrict__ G, int p, double* __restrict__ small,
                                    int* __restrict__ info_rank) {
  if (threadIdx.x == 0 && blockIdx.x == 0) small_factor(G, p, small, info_rank);
}

// tri_apply_sum_kernel, gram_kernel and small_factor_kernel in one launch by one
// workgroup, for studies of up to COV_MAX padded rows, whose three launches take
// longer than their work: W from its partial sums, its Gram matrix (a wave per
// pair in turn), the factor.
constexpr int COV_MAX = 2048;

__global__ __launch_bounds__(1024) void covariates_kernel(const double* __restrict__ part, int N, int p,
                                                          double* __restrict__ W, double* __restrict__ G,
                                                          double* __restrict__ small, int* __restrict__ info_rank) {
  __shared__ double g[20 * 20];
  const int64_t total = (int64_t)N * p;
  for (int64_t idx = threadIdx.x; idx < total; idx += 1024) W[idx] = tri_apply_row(part, total, idx, (int)(idx % N));
  __syncthreads();   // the workgroup's own stores to W are visible to it
  const int lane = threadIdx.x & 63, pairs = p * (p + 1) / 2;
  for (int pair = threadIdx.x >> 6; pair < pairs; pair += 16) {
    int j = 0;
    while ((j + 1) * (j + 2) / 2 <= pair) ++j;
    const int k = pair - j * (j + 1) / 2;
    double s = 0.0;
    for (int r = lane; r < N; r += 64) s += W[r + (int64_t)j * N] * W[r + (int64_t)k * N];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) {
      g[j + k * p] = s;
      g[k + j * p] = s;
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < p * p; e += 1024) G[e] = g[e];
  if (threadIdx.x == 0) small_factor(g, p, small, info_rank);
}

}  // namespace gls

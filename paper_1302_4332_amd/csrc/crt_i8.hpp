// FP64-accurate products of FP64 matrices on the integer matrix cores, through
// the Chinese remainder theorem (the modular form of the Ozaki scheme: Ozaki,
// Uchino and Imamura's Ozaki scheme II).
//
// Row i of op(A) and column j of op(B) are scaled by powers of two so that their
// 2-norms lie in [2^61, 2^62) and rounded to integers a_ik, b_kj.  Then
//     |sum_k a_ik b_kj| <= ||a_i|| ||b_j|| < 2^124.01 < P / 2,
// P the product of sixteen coprime moduli m_p <= 256, so the integer sum is known
// from its residues: sixteen int8 products of the residues (|r| <= 128, summed
// exactly in int32 for K <= CRT_MAX_K), one per modulus, give t_p = sum q_p mod m_p with
// q_p = (P / m_p)^-1 mod m_p, and
//     sum / P = sum_p t_p / m_p  mod 1,
// evaluated to 2^-70 of P in two exact FP64 sums.
//
// The rounding errors are those of the inputs, at most 2^-62 of their row's
// (column's) norm an element, and one of the result.  The bound is normwise:
//     |error| <= 2^-53 |result| + (2^-61 sqrt(K) + 2^-66) ||a_i|| ||b_j||
// (with independent roundings about 2^-62 ||a_i|| ||b_j||), where FP64 accumulation
// has a rounding of every partial sum: 2^-53 sum_k |sum_{l<=k} a_il b_lj|, for vectors
// without structure about 2^-55 ||a_i|| ||b_j||.  Where the large entries of row and
// column do not meet, sum_k |a_ik b_kj| can be far below the norms' product, and an
// element far below its vector's norm keeps fewer than its 53 bits; the
// factorization's own error is bounded by such norms.  Bringing M's diagonal to
// one scale (diagonal_scale_kernel) makes that bound one of each entry of A22 -
// L21 L21^T; it does not bound the spread within a row of L^-1 of an
// ill-conditioned M.
//
// Modelled on the CPU for the four products of a node (kinships of 300 and 2,000
// markers, n = 1,600, h2 = 0.1 to 0.999) the error is 0.42 to 0.59 times 2^-53 of the
// result, rms, and that of an FP64 library product 0.44 to 34 times; at 2^-58 of the
// norms, which fifteen moduli allow, it was 0.48 to 12.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_f64.hpp"
#include "lds_dma.hpp"
#include "ozaki_i8.hpp"

namespace gls {

constexpr int CRT_P = 16;
constexpr int CRT_M[CRT_P] = {256, 251, 247, 243, 241, 239, 235, 233, 229, 227, 223, 217, 211, 199, 197, 193};
constexpr int CRT_NORM = 62;        // norms below 2^62
constexpr int CRT_MAX_K = 1 << 16;  // longest sum: below 2^30, and its recombination below 2^24
constexpr int CRT_NAN = 1 << 30;    // exponent of a vector with a NaN or an infinity

constexpr int crt_gcd(int a, int b) { return b ? crt_gcd(b, a % b) : a; }
constexpr bool crt_coprime() {
  for (int i = 0; i < CRT_P; ++i)
    for (int j = 0; j < i; ++j)
      if (crt_gcd(CRT_M[i], CRT_M[j]) != 1) return false;
  return true;
}
static_assert(crt_coprime(), "moduli");

struct CrtTables {
  int q[CRT_P];          // (P / m)^-1 mod m
  double hi[CRT_P];      // 1 / m = (hi + lo 2^-40) 2^-40 up to 2^-81, hi and lo integers
  double lo[CRT_P];
  int pow16[CRT_P][4];   // 2^(16 j) mod m, symmetric
};
constexpr CrtTables crt_tables() {
  CrtTables t{};
  for (int p = 0; p < CRT_P; ++p) {
    const int m = CRT_M[p];
    int r = 1;
    for (int o = 0; o < CRT_P; ++o)
      if (o != p) r = r * (CRT_M[o] % m) % m;
    for (int x = 0; x < m; ++x)
      if (r * x % m == 1) t.q[p] = x > m / 2 ? x - m : x;
    const unsigned __int128 one = (unsigned __int128)1 << 80;
    const unsigned __int128 inv = (one + m / 2) / m;   // 2^80 / m rounded
    const unsigned __int128 hi = (inv + ((unsigned __int128)1 << 39)) >> 40;
    t.hi[p] = (double)(unsigned long long)hi;
    t.lo[p] = (double)((long long)(inv - (hi << 40)));
    int w = 1;
    for (int j = 0; j < 4; ++j) {
      t.pow16[p][j] = w > m / 2 ? w - m : w;
      w = (int)((long long)w * 65536 % m);
    }
  }
  return t;
}
constexpr CrtTables CRT_T = crt_tables();
// P = 2^125.2: exact in 128 bits, then one rounding.
constexpr unsigned __int128 crt_product() {
  unsigned __int128 a = 1;
  for (int p = 0; p < CRT_P; ++p) a *= (unsigned)CRT_M[p];
  return a;
}
static_assert(crt_product() >> 125 == 1 && (crt_product() - ((unsigned __int128)1 << 125)) >> 122 != 0,
              "P / 2 above 2^124.16, the largest sum's bound");
constexpr double crt_P() { return (double)crt_product(); }

// One operand: vectors (rows of op(A) or columns of op(B)) in groups of 16, k in
// blocks of 64; plane p holds unit (k block, group) at (kb G + g) KB, in the
// matrix instruction's operand order (see ozaki_i8.hpp).  count groups of them,
// from planes on, are the operand: all G, or the columns that a product takes at a
// time (crt_columns), whose first is column d0 of the whole op(B).
struct CrtOperand {
  int8_t* planes;
  int64_t stride;   // bytes per plane
  int* ex;          // ||vector|| < 2^ex
  int G, KB, count, d0;
};

// Exponents.  Vector v of the matrix X (column-major, ld): row v (ROWS) or column
// v, elements k0(v) <= k < k1(v) (lower: of a lower-triangular matrix whose row or
// column d0 is X's first).
//
// ROWS, first part: for 64 rows and 256 columns the largest magnitude's exponent
// and the sum of squares scaled by it.
__global__ __launch_bounds__(256) void crt_row_norm_kernel(const double* __restrict__ X, int64_t ld, int rows, int K,
                                                           int lower, int d0, double* __restrict__ part_ss,
                                                           int* __restrict__ part_e) {
  __shared__ double red[256];
  __shared__ int re[64];
  const int i0 = blockIdx.x * 64, k0 = blockIdx.y * 256;
  const int r = threadIdx.x & 63, g = threadIdx.x >> 6, i = i0 + r;
  if (lower && k0 > d0 + i0 + 63) return;
  const int kend = i < rows ? (lower ? min(K, d0 + i + 1) : K) : 0;
  double x[64], m = 0.0;
#pragma unroll
  for (int u = 0; u < 64; ++u) {
    const int k = k0 + g + 4 * u;
    x[u] = (k < kend) ? X[(int64_t)i + (int64_t)k * ld] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < 64; ++u) {
    const double a = fabs(x[u]);
    m = (a > m || !(a < __builtin_inf())) ? a : m;   // a NaN or an infinity stays
    if (!(m < __builtin_inf())) m = __builtin_inf();
  }
  red[threadIdx.x] = m;
  __syncthreads();
  if (g == 0) {
    m = fmax(fmax(red[r], red[64 + r]), fmax(red[128 + r], red[192 + r]));
    int e = 0;
    if (m > 0.0 && m < __builtin_inf()) frexp(m, &e);
    re[r] = (m < __builtin_inf()) ? e : CRT_NAN;
  }
  __syncthreads();
  const int e = re[r];
  double s = 0.0;
  if (e != CRT_NAN) {
#pragma unroll
    for (int u = 0; u < 64; ++u) {
      const double y = ldexp(x[u], -e);
      s += y * y;
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (g == 0 && i < rows) {
    const int chunks_rows = (rows + 63) / 64 * 64;
    part_ss[(int64_t)blockIdx.y * chunks_rows + i] = red[r] + red[64 + r] + red[128 + r] + red[192 + r];
    part_e[(int64_t)blockIdx.y * chunks_rows + i] = e;
  }
}

// Exponent of a norm from the exponent e of its largest element's chunk and the scaled sum of squares.
__device__ __forceinline__ int crt_exponent(double ss, int e) {
  if (e == CRT_NAN) return CRT_NAN;
  if (!(ss > 0.0)) return 0;
  int f;
  frexp(sqrt(ss) * (1.0 + 1e-14), &f);
  return e + f;
}

// ROWS, second part: ex[i] from the chunks that reach row i.
__global__ __launch_bounds__(256) void crt_row_exp_kernel(const double* __restrict__ part_ss,
                                                          const int* __restrict__ part_e, int rows, int K, int lower,
                                                          int d0, int* __restrict__ ex) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= rows) return;
  const int R = (rows + 63) / 64 * 64;
  const int n = lower ? min((K + 255) / 256, (d0 + i / 64 * 64 + 63) / 256 + 1) : (K + 255) / 256;
  int e = -100000;
  bool any = false;
  for (int s = 0; s < n; ++s) {
    const int f = part_e[(int64_t)s * R + i];
    if (f == CRT_NAN || part_ss[(int64_t)s * R + i] > 0.0) {
      e = max(e, f);
      any = true;
    }
  }
  double ss = 0.0;
  if (any && e != CRT_NAN)
    for (int s = 0; s < n; ++s) {
      const double v = part_ss[(int64_t)s * R + i];
      if (v > 0.0) ss += ldexp(v, 2 * (part_e[(int64_t)s * R + i] - e));
    }
  ex[i] = any ? crt_exponent(ss, e) : 0;
}

// Columns: one wave per column.
__global__ __launch_bounds__(256) void crt_col_exp_kernel(const double* __restrict__ X, int64_t ld, int K, int cols,
                                                          int lower, int d0, int* __restrict__ ex) {
  const int lane = threadIdx.x & 63, j = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= cols) return;
  const double* c = X + (int64_t)j * ld;
  const int kb = lower ? d0 + j : 0;
  double m = 0.0;
#pragma unroll 4
  for (int k = kb + lane; k < K; k += 64) {
    const double a = fabs(c[k]);
    m = (a > m || !(a < __builtin_inf())) ? a : m;
    if (!(m < __builtin_inf())) m = __builtin_inf();
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  if (!(m < __builtin_inf())) {
    if (lane == 0) ex[j] = CRT_NAN;
    return;
  }
  int e = 0;
  if (m > 0.0) frexp(m, &e);
  double s = 0.0;
#pragma unroll 4
  for (int k = kb + lane; k < K; k += 64) {
    const double y = ldexp(c[k], -e);
    s += y * y;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) ex[j] = crt_exponent(s, e);
}

// Byte t of w <- r as int8, for the whole number off = r + 128 in [0, 255]
// (v_cvt_pk_u8_f32); xor the finished word with 0x80808080.
__device__ __forceinline__ uint32_t crt_byte(float off, int t, uint32_t w) {
  return __builtin_amdgcn_cvt_pk_u8_f32(off, t, w);
}

// A lane's 16 elements as residues of every modulus, into its 16 bytes of each
// plane's unit.  The integer (below 2^62) is cut into four signed 16-bit pieces, so
// that its residue is a sum below 2^24 (2^15 + 125 (2^15 + 2^15 + 2^14) + 128 at most)
// that FP32 holds exactly; the quotient, below 53,300, is off by 2^-23 of itself at most
// before it is rounded, which leaves |r| <= 0.507 m, and at most 0.505 m = 126 for m =
// 251.  The byte for m = 256 is the integer's lowest.
__device__ __forceinline__ void crt_store_unit(const double (&x)[16], int e, int8_t* o, int64_t stride) {
  float c[16][4];
  uint32_t low[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int b = 0; b < 16; ++b) {
    long long v = (e == CRT_NAN) ? 0 : __double2ll_rn(ldexp(x[b], CRT_NORM - e));
    low[b >> 2] |= (uint32_t)((int)v & 255) << (8 * (b & 3));
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int d = (int)(int16_t)(v & 65535);
      v = (v - d) >> 16;
      c[b][j] = (float)(j == 0 ? d + 128 : d);
    }
    c[b][3] = (float)(int)v;
  }
  *reinterpret_cast<uint4*>(o) = make_uint4(low[0], low[1], low[2], low[3]);
#pragma unroll
  for (int p = 1; p < CRT_P; ++p) {
    const float m = (float)CRT_M[p], inv = 1.0f / (float)CRT_M[p];
    const float k1 = (float)CRT_T.pow16[p][1], k2 = (float)CRT_T.pow16[p][2], k3 = (float)CRT_T.pow16[p][3];
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int b = 0; b < 16; ++b) {
      const float s = fmaf(c[b][3], k3, fmaf(c[b][2], k2, fmaf(c[b][1], k1, c[b][0])));   // + 128
      w[b >> 2] = crt_byte(fmaf(-rintf(fmaf(s, inv, -128.0f * inv)), m, s), b & 3, w[b >> 2]);
    }
    *reinterpret_cast<uint4*>(o + p * stride) =
        make_uint4(w[0] ^ 0x80808080u, w[1] ^ 0x80808080u, w[2] ^ 0x80808080u, w[3] ^ 0x80808080u);
  }
}

// Tile of the product kernel: k blocks are taken in or left out for whole tiles.
constexpr int CRT_BM = 192, CRT_BN = 192, CRT_THREADS = 256;
static_assert(CRT_BM == CRT_BN, "one trim of the triangles for rows and columns");

// Residues of 64 rows x 64 k (ROWS).  lower: zeros past the diagonal, up to the tile's last k block.
__global__ __launch_bounds__(256) void crt_rows_kernel(const double* __restrict__ X, int64_t ld, int rows, int K,
                                                       int lower, CrtOperand op) {
  const int kb = blockIdx.x, i0 = blockIdx.y * 64;
  const int d0 = op.d0;   // a multiple of CRT_BN = CRT_BM
  if (lower && kb * 64 > d0 + (i0 + 63) / CRT_BM * CRT_BM + CRT_BM - 1) return;
  const int r = threadIdx.x & 63, kq = threadIdx.x >> 6, i = i0 + r;
  const int g = i >> 4;
  if (g >= op.G) return;
  double x[16];
#pragma unroll
  for (int b = 0; b < 16; ++b) {
    const int k = kb * 64 + kq * 16 + b;
    x[b] = (i < rows && k < K && !(lower && k > d0 + i)) ? X[(int64_t)i + (int64_t)k * ld] : 0.0;
  }
  crt_store_unit(x, i < rows ? op.ex[i] : 0, op.planes + ((int64_t)kb * op.G + g) * 1024 + 16 * (kq * 16 + (r & 15)),
                 op.stride);
}

// Residues of 16 columns x 64 k per wave (columns).  lower: zeros before the diagonal, from the tile's first k block on.
__global__ __launch_bounds__(256) void crt_cols_kernel(const double* __restrict__ X, int64_t ld, int K, int cols,
                                                       int lower, CrtOperand op) {
  const int g = blockIdx.x, lane = threadIdx.x & 63;
  const int kb = blockIdx.y * 4 + (threadIdx.x >> 6);
  const int d0 = op.d0;
  if (kb >= op.KB || (lower && kb * 64 + 63 < d0 + g * 16 / CRT_BN * CRT_BN)) return;
  const int j = g * 16 + (lane & 15), k0 = kb * 64 + (lane >> 4) * 16;
  double x[16];
  const double* c = X + (int64_t)j * ld + k0;
#pragma unroll
  for (int b = 0; b < 16; ++b) x[b] = (j < cols && k0 + b < K && !(lower && k0 + b < d0 + j)) ? c[b] : 0.0;
  crt_store_unit(x, j < cols ? op.ex[j] : 0, op.planes + ((int64_t)kb * op.G + g) * 1024 + 16 * lane, op.stride);
}

struct CrtArgs {
  CrtOperand a, b;
  int M, N, K;         // result rows and columns, sum length; columns [b.d0, b.d0 + N) of the whole result
  int a_lower;         // op(A)[i, k] = 0 for k > i
  int b_lower;         // op(B)[k, j] = 0 for k < j
  int b_upper;         // op(B)[k, j] = 0 for k > j
  int c_lower;         // only 16 x 16 tiles that reach the lower part of C
  uint32_t* out;       // residues t_p: plane p, 16 x 16 tile (row group rg, column group cg) at (cg a.count + rg) 64 dwords
  int64_t out_stride;  // dwords per plane
  // crt_finish_kernel: C = alpha op(A) op(B) + beta Cin
  double alpha, beta;
  const double* Cin; int64_t ldcin;
  double* C; int64_t ldc;
};

// One modulus's product (blockIdx.y): 192 x 192 tiles, four waves of 96 x 96 (6 x 6
// accumulators), stages of 64 k from global memory into a ring of three LDS
// buffers, two workgroups to a compute unit.  At w = 5,000 sixteen triangular
// products take 1.10 ms (1,800 TOPS).
// XCD groups: one row tile x 16 column tiles, and 4 x 8 where the sums start at the
// columns' diagonal (w = 5,000: 0.95-1.01 ms against 1.03-1.57 with 4 x 8, and
// 1.02 against 1.19).
__host__ __device__ inline int crt_map_gm(const CrtArgs& g) { return g.b_lower ? 4 : 1; }
__host__ __device__ inline int crt_map_gn(const CrtArgs& g) { return g.b_lower ? 8 : 16; }

__global__ __launch_bounds__(CRT_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void crt_gemm_kernel(CrtArgs g) {
  constexpr int NS = 3, NW = 4, U = 12, F = 6, STAGE = 2 * U * 1024, NLD = 2 * U / NW;
  static_assert(NLD * NW == 2 * U && NLD % 2 == 0, "loads");
  __shared__ __align__(1024) int8_t smem[NS * STAGE];
  const int p = blockIdx.y;
  int ti, tj;
  {
    GemmArgs m{};
    m.map_gm = crt_map_gm(g);
    m.map_gn = crt_map_gn(g);
    m.map_slots = 512;
    m.map_desc = g.a_lower | g.c_lower;
    // rows are dealt to the XCDs anew for each modulus: with some tens of row tiles some XCDs get a row more
    const int bid = (blockIdx.x & ~7) | ((blockIdx.x + p) & 7);
    if (!XcdMap::tile(m, bid, (g.M + CRT_BM - 1) / CRT_BM, (g.N + CRT_BN - 1) / CRT_BN, &ti, &tj)) return;
  }
  const int i0 = ti * CRT_BM, j0 = g.b.d0 + tj * CRT_BN;
  if (g.c_lower && i0 + CRT_BM - 1 < j0) return;
  int k0 = 0, k1 = g.a.KB;
  if (g.a_lower) k1 = imin(k1, (i0 + CRT_BM + 63) / 64);
  if (g.b_upper) k1 = imin(k1, (j0 + CRT_BN + 63) / 64);
  if (g.b_lower) k0 = j0 / 64;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave & 1, wc = wave >> 1;
  const int ga0 = ti * U, gb0 = tj * U;
  const int8_t* A = g.a.planes + p * g.a.stride;
  const int8_t* B = g.b.planes + p * g.b.stride;
  const uint32_t lds0 = lds_address(smem), voff = 16 * lane;
  int at[NLD];   // this wave's units within a k block: A's, then B's (groups past the end: the last one's, dropped)
#pragma unroll
  for (int q = 0; q < NLD; ++q) {
    const int u = q * NW + wave;
    at[q] = (q < NLD / 2 ? imin(ga0 + u, g.a.count - 1) : imin(gb0 + u - U, g.b.count - 1)) * 1024;
  }
  const int64_t sa = (int64_t)g.a.G * 1024, sb = (int64_t)g.b.G * 1024;
  auto issue = [&](int kb) {
    const uint32_t base = lds0 + (uint32_t)((kb - k0) % NS * STAGE);
    const int8_t *a = A + kb * sa, *b = B + kb * sb;
#pragma unroll
    for (int q = 0; q < NLD; ++q)
      lds_load16_sv((q < NLD / 2 ? a : b) + at[q], voff, base + (uint32_t)((q * NW + wave) * 1024));
  };
  i4_t acc[F][F];
#pragma unroll
  for (int a = 0; a < F; ++a)
#pragma unroll
    for (int c = 0; c < F; ++c) acc[a][c] = i4_t{0, 0, 0, 0};
  for (int q = 0; q < NS - 1; ++q)
    if (k0 + q < k1) issue(k0 + q);
  const int oa = wr * F * 1024 + 16 * lane, ob = (U + wc * F) * 1024 + 16 * lane;
  for (int kb = k0; kb < k1; ++kb) {
    wait_stages<NLD>(imin(k1 - 1 - kb, NS - 2));
    __syncthreads();
    if (kb + NS - 1 < k1) issue(kb + NS - 1);
    const int8_t* st = smem + (kb - k0) % NS * STAGE;
    i4_t bf[F];
#pragma unroll
    for (int c = 0; c < F; ++c) bf[c] = *reinterpret_cast<const i4_t*>(st + ob + c * 1024);
#pragma unroll
    for (int a = 0; a < F; ++a) {
      const i4_t af = *reinterpret_cast<const i4_t*>(st + oa + a * 1024);
#pragma unroll
      for (int c = 0; c < F; ++c) acc[a][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af, bf[c], acc[a][c], 0, 0, 0);
    }
  }
  // t_p = q_p acc mod m, from acc's high and low parts (FP32 holds every step exactly; the odd moduli as in
  // crt_store_unit)
  const int m = CRT_M[p], q = CRT_T.q[p];
  int qh = q * 16384 % m;
  qh = qh > m / 2 ? qh - m : qh < -(m / 2) ? qh + m : qh;
  const float mf = (float)m, inv = 1.0f / mf, ql = (float)q, qhf = (float)qh;
  uint32_t* out = g.out + p * g.out_stride;
#pragma unroll
  for (int a = 0; a < F; ++a) {
    const int rg = ga0 + wr * F + a;
    if (rg >= g.a.count) continue;
#pragma unroll
    for (int c = 0; c < F; ++c) {
      const int cg = gb0 + wc * F + c;
      if (cg >= g.b.count || (g.c_lower && rg < cg + g.b.d0 / 16)) continue;
      uint32_t w = 0;
      if (p == 0) {
#pragma unroll
        for (int t = 0; t < 4; ++t) w |= (uint32_t)(acc[a][c][t] * q & 255) << (8 * t);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int v = acc[a][c][t];
          const float s = fmaf((float)(v >> 14), qhf, fmaf((float)(v & 16383), ql, 128.0f));
          w = crt_byte(fmaf(-rintf(fmaf(s, inv, -128.0f * inv)), mf, s), t, w);
        }
        w ^= 0x80808080u;
      }
      out[((int64_t)cg * g.a.count + rg) * 64 + lane] = w;
    }
  }
}

// C from the residues.  A wave takes 16 x 16 tiles in turn; lane l holds rows
// 4 (l / 16) + t of column l % 16, as the matrix instruction left them.
__device__ __forceinline__ void crt_value(const uint32_t* __restrict__ at, int64_t stride, double (&v)[4]) {
  uint32_t w[CRT_P];
#pragma unroll
  for (int p = 0; p < CRT_P; ++p) w[p] = at[p * stride];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int p = 0; p < CRT_P; ++p) {
      const double r = (double)(int)(int8_t)(w[p] >> (8 * t));
      s1 = fma(r, CRT_T.hi[p], s1);   // exact: integers below 2^49
      s2 = fma(r, CRT_T.lo[p], s2);
    }
    // the fraction modulo 1, in units of 2^-40, with the low parts' carry
    const double s = s1 - 0x1p40 * rint((s1 + s2 * 0x1p-40) * 0x1p-40);
    v[t] = fma(s2, 0x1p-40, s) * 0x1p-40;
  }
}

__global__ __launch_bounds__(256) void crt_finish_kernel(CrtArgs g) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cg = blockIdx.y;
  const int j = cg * 16 + (lane & 15);
  const int ej = j < g.N ? g.b.ex[j] : 0;
  for (int rg = blockIdx.x * 4 + wave; rg < g.a.count; rg += gridDim.x * 4) {
    if (g.c_lower && rg < cg + g.b.d0 / 16) continue;
    double v[4];
    crt_value(g.out + ((int64_t)cg * g.a.count + rg) * 64 + lane, g.out_stride, v);
    const int i = rg * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (i + t >= g.M || j >= g.N) continue;
      const int ei = g.a.ex[i + t];
      double x = ldexp(v[t] * crt_P(), ei + ej - 2 * CRT_NORM) * g.alpha;
      if (ei == CRT_NAN || ej == CRT_NAN) x = __builtin_nan("");
      if (g.beta != 0.0) x += g.beta * g.Cin[(int64_t)(i + t) + (int64_t)j * g.ldcin];
      g.C[(int64_t)(i + t) + (int64_t)j * g.ldc] = x;
    }
  }
}

}  // namespace gls

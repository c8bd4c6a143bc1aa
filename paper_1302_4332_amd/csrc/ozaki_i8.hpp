// FP64-accurate per-block product on the integer matrix cores, for SNP values
// that are whole numbers (genotype dosages), held as FP64, bytes or packed
// 2-bit codes.
//
// Each row i of L^-1 is rounded to an 8 S-bit fixed-point number and split into
// S signed base-256 digits (the slicing of Ozaki, Ogita, Oishi and Rump's
// error-free matrix product transformation, with balanced digits):
//     L^-1[i, k] = 2^(e_i - 8 S + 1) * sum_{s<S} a_s[i, k] * 256^s  +  r_ik,
//     -128 <= a_s <= 127,  |r_ik| <= 2^(e_i - 8 S),  max_k |L^-1[i, k]| <= 0.99 * 2^e_i.
// Whole numbers x with |x| <= 127 are exact in int8, so
//     (L^-1 X)[i, j] = sum_s 2^(e_i - 8 S + 1) 256^s (a_s X)[i, j]   (+ r)
// where each a_s X is an exact int32 sum (n * 128 * max|x| < 2^31), and there is
// one FP64 rounding per digit instead of one per sample.  The rounding r is
// relative to the row's largest entry (2^(e_i - 1) at most below it), not to the
// entry itself:
//   S = 8 (FP64 handles): entries down to 2^-10 of 2^e_i are exact, any other is
//     off by 2^-64 of it at most.  Against sums in 64-bit significands the whitened
//     values are off by 0.12 to 0.7 times as much as those of FP64 sums (kinships
//     of 500 to 2,000 markers, n = 800 to 5,000, h2 = 0.1 to 0.999; seven digits: 0.4
//     to 6 times).
//   S = 7 (GLS_INT8_EMU): 2^-56 of 2^e_i, the bound of eight truncated 7-bit slices
//     with an eighth less work.
//
// Operands are kept in the order the matrix instruction reads them.  A unit is
// 1 KB: 16 rows (of L^-1) or 16 SNPs times 64 k, byte b of lane l being element
// (l % 16, 16 (l / 16) + b), which is v_mfma_i32_16x16x64_i8's A (and B) operand
// layout (checked on gfx950 with known operands).  Every load from global memory
// to LDS is then a contiguous 1 KB, and every fragment read from LDS one
// contiguous, conflict-free 1 KB without address arithmetic.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_f64.hpp"
#include "lds_dma.hpp"

namespace gls {

constexpr int OZ_DIGITS_FP64 = 8, OZ_DIGITS_EMU = 7;
constexpr int OZ_UNIT = 1024;                        // bytes of a unit
constexpr int OZ_BM = 32, OZ_BK = 64;                // rows of a product tile and k per stage
constexpr int OZ_STRIPS = OZ_BM / 16;
constexpr int OZ_TM = 64;                            // rows of a tile of the sliced factor

// Bytes of one (row tile, k block) of the factor sliced into S digits.
constexpr int oz_atile(int S) { return OZ_TM / 16 * S * OZ_UNIT; }

// Bytes of the sliced factor: row tile t holds the k blocks 0..t that reach the lower triangle.
inline size_t oz_factor_bytes(int64_t N, int S) {
  const int64_t T = N / OZ_TM;
  return (size_t)(T * (T + 1) / 2) * oz_atile(S);
}

typedef int i4_t __attribute__((ext_vector_type(4)));

// Largest |Li[i, k]| over k in [256 s, 256 s + 256), k <= i: part[s N + i].
// Workgroup (row block, s): 64 rows, four waves over k.
__global__ __launch_bounds__(256) void row_max_kernel(const double* __restrict__ Li, int N, double* __restrict__ part) {
  __shared__ double red[256];
  const int i0 = blockIdx.x * 64, k0 = blockIdx.y * 256;
  if (k0 > i0 + 63) return;
  const int r = threadIdx.x & 63, g = threadIdx.x >> 6, i = i0 + r;
  double m = 0.0;
  const int kend = min(k0 + 256, i0 + 64);
#pragma unroll 8
  for (int k = k0 + g; k < kend; k += 4) m = fmax(m, fabs(Li[(int64_t)i + (int64_t)k * N]));
  red[threadIdx.x] = m;
  __syncthreads();
  if (g == 0)
    part[(int64_t)blockIdx.y * N + i] = fmax(fmax(red[r], red[64 + r]), fmax(red[128 + r], red[192 + r]));
}

// The digits of a 64 x 64 block of L^-1 (row tile ti, k block kb <= ti), and
// the rows' exponents: ex[i] with max_k |Li[i, k]| <= 0.99 * 2^ex[i], so that the
// top digit stays within [-128, 127] after the lower digits' carries.  Thread
// (row r, k group kq) reads 16 consecutive k of its row (coalesced over rows)
// and writes its lane's 16 bytes of each digit's unit.
template <int S>
__global__ __launch_bounds__(256) void slice_factor_kernel(const double* __restrict__ Li, int N,
                                                           const double* __restrict__ part, int* __restrict__ ex,
                                                           int8_t* __restrict__ out) {
  const int ti = blockIdx.y, kb = blockIdx.x;
  if (kb > ti) return;
  const int r = threadIdx.x & 63, kq = threadIdx.x >> 6;
  const int i = ti * 64 + r;
  double x[16];
#pragma unroll
  for (int b = 0; b < 16; ++b) x[b] = Li[(int64_t)i + (int64_t)(kb * 64 + kq * 16 + b) * N];
  double m = 0.0;
  for (int s = 0; s <= (ti * 64 + 63) / 256; ++s) m = fmax(m, part[(int64_t)s * N + i]);
  int e = 0;
  if (m > 0.0 && frexp(m, &e) > 0.99) ++e;
  if (kb == 0 && kq == 0) ex[i] = e;
  uint32_t w[S][4];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q) w[s][q] = 0u;
#pragma unroll
  for (int b = 0; b < 16; ++b) {
    long long q = __double2ll_rn(ldexp(x[b], 8 * S - 1 - e));   // below 0.99 * 2^(8 S - 1)
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int d = (int)(int8_t)(q & 255);
      q = (q - d) >> 8;
      w[s][b >> 2] |= (uint32_t)(d & 255) << (8 * (b & 3));
    }
  }
  int8_t* o = out + ((int64_t)ti * (ti + 1) / 2 + kb) * oz_atile(S) + (r >> 4) * (S * OZ_UNIT) +
              16 * (kq * 16 + (r & 15));
#pragma unroll
  for (int s = 0; s < S; ++s)
    *reinterpret_cast<uint4*>(o + s * OZ_UNIT) = make_uint4(w[s][0], w[s][1], w[s][2], w[s][3]);
}

// *ok = 1 if M's diagonal spans a factor of at most 256, else 0.  The digits are
// fixed-point at the scale of their row of L^-1, whose columns go with
// M_jj^-1/2: over wildly different scales a SNP that is zero at the dominant
// samples would lose the others' low bits, and FP64 handles then form every
// product in FP64.
__global__ __launch_bounds__(1024) void diagonal_range_kernel(const double* __restrict__ Phi, int64_t ld_phi, int n,
                                                              double h2, int* __restrict__ ok) {
  __shared__ double lo[16], hi[16];
  double a = __builtin_inf(), b = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) {
    const double d = h2 * Phi[(int64_t)i * (ld_phi + 1)] + (1.0 - h2);
    a = fmin(a, d);
    b = fmax(b, d);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    a = fmin(a, __shfl_xor(a, off, 64));
    b = fmax(b, __shfl_xor(b, off, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    lo[threadIdx.x >> 6] = a;
    hi[threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) {
      a = fmin(a, lo[w]);
      b = fmax(b, hi[w]);
    }
    *ok = (b <= 256.0 * a) ? 1 : 0;
  }
}

// Packed dosages: four 2-bit codes per byte, sample k of a column in bits
// [2 (k % 4), 2 (k % 4) + 2) of the column's byte k / 4; code value = dosage
// (0..3).  Bits of the last byte past row n - 1 are ignored.
__device__ __forceinline__ uint32_t unpack_quad(const uint8_t* __restrict__ G2, int64_t ldg, int n, int q, int j) {
  const int k0 = 4 * q;
  if (k0 >= n) return 0u;
  const uint32_t b = G2[(int64_t)j * ldg + q];
  uint32_t w = (b & 3u) | ((b & 0x0cu) << 6) | ((b & 0x30u) << 12) | ((b & 0xc0u) << 18);
  const int rem = n - k0;
  if (rem < 4) w &= (1u << (8 * rem)) - 1u;
  return w;   // byte t = dosage of row k0 + t
}

// Where a block's int8 operand and its column flags come from.
enum { OZ_F64 = 0, OZ_F64_ALIGNED = 1, OZ_U8 = 2, OZ_U2 = 3 };

// A block's SNP values as units [k block][SNP group of 16] (Jb groups).  flags
// (nullptr: none are needed) receives, for every k chunk c and SNP group, the SNPs
// with a value in the chunk that is not a whole number of magnitude
// at most xmax (ColFlags; all SNPs if *ok is 0).  A wave whose SNPs are all flagged stops: their results come
// from the FP64 product.  Workgroup (group, chunk of chunk_kb k blocks), four
// waves over the chunk's k blocks; a lane holds its 16 bytes' values, so FP64
// columns are read as whole 128-byte lines.  The waves first look at four values of
// each SNP, the same ones: a group of imputed SNPs mostly ends there, having read
// 8 KB instead of a k block a wave.
template <int SRC>
__global__ __launch_bounds__(256) void pack_units_kernel(const void* __restrict__ src, int64_t ld, int n, int nkb,
                                                         int mb, int Jb, int chunk_kb, int xmax,
                                                         uint8_t* __restrict__ out, int* __restrict__ flags,
                                                         const int* __restrict__ ok_study) {
  __shared__ int seen[4];
  const int jb = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = jb * 16 + (lane & 15), kq = lane >> 4;
  const bool col = j < mb;
  const unsigned cols = (mb - jb * 16 >= 16) ? 0xffffu : (1u << (mb - jb * 16)) - 1u;
  const int kb1 = min(nkb, (int)(blockIdx.y + 1) * chunk_kb);
  unsigned bad = (flags && !*ok_study) ? cols : 0u;   // flagged columns (wave-uniform)
  if constexpr (SRC == OZ_F64 || SRC == OZ_F64_ALIGNED) {
    const int k = blockIdx.y * chunk_kb * 64 + kq * 16;
    const double x = (col && k < n) ? static_cast<const double*>(src)[(int64_t)j * ld + k] : 0.0;
    const int v = (int)x;   // saturates; NaN gives 0
    const unsigned long long m = __ballot(!((double)v == x && v <= xmax && v >= -xmax));
    bad |= (unsigned)((m | (m >> 16) | (m >> 32) | (m >> 48)) & 0xffffu);
  }
  if (bad != cols) for (int kb = blockIdx.y * chunk_kb + wave; kb < kb1; kb += 4) {
    const int k0 = kb * 64 + kq * 16;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if constexpr (SRC == OZ_F64 || SRC == OZ_F64_ALIGNED) {
      double x[16];
#pragma unroll
      for (int b = 0; b < 16; ++b) x[b] = 0.0;
      if (col) {
        const double* p = static_cast<const double*>(src) + (int64_t)j * ld + k0;
        if (k0 + 16 <= n) {
          if (SRC == OZ_F64_ALIGNED) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              const double2 v = reinterpret_cast<const double2*>(p)[q];
              x[2 * q] = v.x;
              x[2 * q + 1] = v.y;
            }
          } else {
#pragma unroll
            for (int b = 0; b < 16; ++b) x[b] = p[b];
          }
        } else {
#pragma unroll
          for (int b = 0; b < 16; ++b)
            if (k0 + b < n) x[b] = p[b];
        }
      }
      bool ok = true;
#pragma unroll
      for (int b = 0; b < 16; ++b) {
        const int v = (int)x[b];   // saturates; NaN gives 0
        ok = ok && (double)v == x[b] && v <= xmax && v >= -xmax;
        w[b >> 2] |= (uint32_t)(v & 255) << (8 * (b & 3));
      }
      const unsigned long long m = __ballot(!ok);
      bad |= (unsigned)((m | (m >> 16) | (m >> 32) | (m >> 48)) & 0xffffu);
      if (bad == cols) break;
    } else if constexpr (SRC == OZ_U8) {
      if (col && k0 < n) {
        const uint8_t* p = static_cast<const uint8_t*>(src) + (int64_t)j * ld + k0;
        if (k0 + 16 <= n) {
          __builtin_memcpy(w, p, 16);
        } else {
#pragma unroll
          for (int b = 0; b < 16; ++b)   // all in flight: one after another they took 12 us
            if (k0 + b < n) w[b >> 2] |= (uint32_t)p[b] << (8 * (b & 3));
        }
      }
      if (flags) {
        bool ok = true;
#pragma unroll
        for (int b = 0; b < 16; ++b) ok = ok && (int)((w[b >> 2] >> (8 * (b & 3))) & 255u) <= xmax;
        const unsigned long long m = __ballot(!ok);
        bad |= (unsigned)((m | (m >> 16) | (m >> 32) | (m >> 48)) & 0xffffu);
        if (bad == cols) break;
      }
    } else {
      if (col) {
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = unpack_quad(static_cast<const uint8_t*>(src), ld, n, k0 / 4 + q, j);
      }
    }
    *reinterpret_cast<uint4*>(out + ((int64_t)kb * Jb + jb) * OZ_UNIT + 16 * lane) = make_uint4(w[0], w[1], w[2], w[3]);
  }
  if (flags) {
    if (lane == 0) seen[wave] = (int)bad;
    __syncthreads();
    if (threadIdx.x == 0) flags[(int64_t)blockIdx.y * Jb + jb] = seen[0] | seen[1] | seen[2] | seen[3];
  }
}

// The two products' columns of a block, from its flags: words, the flags of a single
// chunk, and the lists of the columns that the integer (whole) and the FP64 product
// (f64) form.  Products that formed every tile of the block with one of their
// columns did each other's work where the two kinds are mixed: 8,192 SNPs at n =
// 10,000 with one whole in 64 took 15.7 ms, where the FP64 product of all of them
// takes 13.3, and now take 13.8; with every other one whole 8.1.  One workgroup, a
// group of 16 columns a thread at a time, 5 us.  Blocks of few SNPs do without (see
// split_columns).
constexpr int CL_THREADS = 1024;

__global__ __launch_bounds__(CL_THREADS) void columns_kernel(ColFlags flags, int mb, int* __restrict__ words,
                                                             int* __restrict__ whole, int* __restrict__ f64) {
  __shared__ int sums[CL_THREADS / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int before = 0;   // flagged columns of the groups below g0
  for (int g0 = 0; g0 < flags.groups; g0 += CL_THREADS) {
    const int g = g0 + t;
    const int w = g < flags.groups ? flags.word(g) : 0;   // no bits past the last column
    const int own = __popc(w);
    int sum = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(sum, off, 64);
      if (lane >= off) sum += o;
    }
    if (lane == 63) sums[wave] = sum;
    __syncthreads();
    int r = before + sum - own;   // flagged columns before this group's next one
    for (int o = 0; o < CL_THREADS / 64; ++o) {
      if (o < wave) r += sums[o];
      before += sums[o];
    }
    if (g < flags.groups) {
      words[g] = w;
      const int c1 = min(16, mb - 16 * g);
      for (int c = 0; c < c1; ++c) {
        const int j = 16 * g + c;
        if ((w >> c) & 1) f64[1 + r++] = j;
        else whole[1 + j - r] = j;
      }
    }
    __syncthreads();   // sums is written again
  }
  if (t == 0) {
    f64[0] = before;
    whole[0] = mb - before;
  }
}

// Columns of a block widened (or copied) into the zero-padded FP64 buffer out
// (ld ldo, rows n..rows-1 zero): every column, or with flags only the flagged
// ones, or with a list the listed ones, one after another.  Workgroup (x, y): rows
// [WIDEN_ROWS y, ...) of columns x, x + gridDim.x, ...
constexpr int WIDEN_ROWS = 2048;

template <int SRC>
__global__ __launch_bounds__(256) void widen_columns_kernel(const void* __restrict__ src, int64_t ld, int n, int rows,
                                                            int mb, double* __restrict__ out, int64_t ldo,
                                                            ColFlags flags, ColList cols) {
  const int count = cols.count(mb);
  for (int i = blockIdx.x; i < count; i += gridDim.x) {
    const int j = cols[i];
    if (flags.at && !flags.flagged(j)) continue;
    double* o = out + (int64_t)i * ldo;
    const int k1 = min(rows, (int)(blockIdx.y + 1) * WIDEN_ROWS);
#pragma unroll 4
    for (int k = blockIdx.y * WIDEN_ROWS + threadIdx.x; k < k1; k += 256) {
      double v = 0.0;
      if (k < n) {
        if constexpr (SRC == OZ_U8) v = (double)static_cast<const uint8_t*>(src)[(int64_t)k + (int64_t)j * ld];
        else if constexpr (SRC == OZ_U2)
          v = (double)((static_cast<const uint8_t*>(src)[(int64_t)j * ld + (k >> 2)] >> (2 * (k & 3))) & 3);
        else v = static_cast<const double*>(src)[(int64_t)k + (int64_t)j * ld];
      }
      o[k] = v;
    }
  }
}

struct OzArgs {
  const int8_t* A;        // sliced factor: row tile t's k blocks 0..t of oz_atile(S) bytes
  const int* ex;          // row exponents
  const uint8_t* B;       // units [k block][Jb]
  int Jb;                 // SNP groups of 16
  int N, Mt, ncols;       // Mt row tiles of OZ_BM
  ColList cols;           // the columns to form, if there are as many as range says
  ColRange range;
  ColFlags flags;         // without a list: flagged columns are left out (at == nullptr: none)
  // per-SNP sums (red_q > 0): red_part[(t red_q + q) ncols + j] as in GemmArgs, over row tile t of OZ_BM rows
  const double* W; int64_t ldw;
  double* red_part;
  int red_q;
  double* C; int64_t ldc; // red_q == 0: the product itself, N x ncols FP64
};

// Sums over a wave's four rows of 16 lanes, two values or pairs of them at a time:
// the value's two halves change places between registers, without the LDS port.
// add_rows16: in even rows a's sums of rows (r, r + 1), in odd ones b's of (r - 1, r);
// add_rows32: in lanes 0..31 a's sums of lanes (l, l + 32), in the others b's.
__device__ __forceinline__ double add_rows16(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double add_rows32(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// A workgroup of four waves owns 32 rows x 192 SNPs with seven digits, 32 x 160 with
// eight (26 KB a stage either way): wave w takes the 16-row
// strip w & 1 and the half w >> 1 of the SNPs with all the digits, 7 x 6 or 8 x 5
// accumulators of 16 x 16 (168 or 160 registers; two waves per SIMD).  Per 64-deep
// stage it reads thirteen 1 KB fragments for 42 or 40 MFMAs; sixteen waves of
// 4 x 4 accumulators on a 32 x 256 tile read eight for 16 and kept the LDS port
// busy for longer than the MFMA pipes.  Stages move straight from global memory
// into a ring of three LDS buffers, two ahead of the MFMAs.
//
// What bounds it (n = 10,000, 8,192 SNPs: eight digits 2.5 ms, 2,600 TOPS; seven 2.2 ms):
// with seven digits the MFMA pipes were busy 58% of the launch and the clock fell to
// 2.1 GHz under its power (with all-zero SNPs 2.0 of 2.3 ms).  The rest is waits
// after the stage barrier, which is why two workgroups with barriers of their own
// share a compute unit: one workgroup of eight waves (64 rows) had its pipes busy
// 48% and took 2.6 ms.  XCD groups of 4 x 8 tiles; 2 x 16 and 4 x 16 are equal
// within noise, 8 x 4 and 8 x 8 6% slower.
//
// A wave's accumulator element t of lane l is row 4 (l / 16) + t, SNP l % 16 of
// its 16 x 16 block, so a sum over the rows is four values of the lane and two
// exchanges between lanes.  Through the LDS port those were most of the epilogue: n =
// 3,968, 3,094 SNPs as bytes, p = 20 376 -> 335 us, p = 4 197 -> 188; n = 2,503, 1,001
// SNPs, p = 8 70.6 -> 65.0.
constexpr int OZ_THREADS = 256, OZ_STAGES = 3;
constexpr int oz_bn(int S) { return S == 7 ? 192 : 160; }
constexpr int OZ_MAP_GM = 4, OZ_MAP_GN = 8;

template <int S>
__global__ __launch_bounds__(OZ_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ozaki_i8_kernel(OzArgs g) {
  constexpr int NW = OZ_THREADS / 64, NS = OZ_STAGES, BN = oz_bn(S);
  constexpr int BU = BN / 16, FC = BU / 2;              // SNP groups per tile and per wave
  constexpr int AU = OZ_STRIPS * S, STAGE = (AU + BU) * OZ_UNIT;
  constexpr int NLD = (AU + BU + NW - 1) / NW, FULL = AU + BU - (NLD - 1) * NW;   // loads a stage; waves < FULL do NLD, the others one less
  constexpr int QC = 10;                                   // sums per pass of the epilogue's LDS exchange
  static_assert(NS * STAGE <= 80 * 1024 && OZ_STRIPS * QC * BN * 8 <= NS * STAGE, "LDS");
  __shared__ __align__(1024) int8_t smem[NS * STAGE];

  int ti, tj;
  {
    GemmArgs m{};
    m.map_gm = OZ_MAP_GM;
    m.map_gn = OZ_MAP_GN;
    m.map_slots = 512;
    m.map_desc = 1;
    if (!XcdMap::tile(m, blockIdx.x, g.Mt, (g.ncols + BN - 1) / BN, &ti, &tj)) return;
  }
  const int nk = ti * OZ_BM / OZ_TM + 1;   // lower triangular factor
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ws = wave & 1, wc = wave >> 1;
  const int j0 = tj * BN;
  const int count = g.cols.count(g.ncols);
  if (j0 >= count || (g.cols.at && !g.range.holds(count))) return;
  const ColList cols = g.cols.or_all(count, g.ncols);

  const int8_t* Abase = g.A + (int64_t)(nk - 1) * nk / 2 * oz_atile(S) + ti % (OZ_TM / OZ_BM) * (AU * OZ_UNIT);
  const uint32_t lds0 = lds_address(smem);
  // Lane offsets of this wave's loads: within A's unit, or of the lane's SNP and k within B's k block (SNPs past the
  // end: the last one, dropped).
  uint32_t voff[NLD];
#pragma unroll
  for (int q = 0; q < NLD; ++q) {
    const int u = q * NW + wave;
    voff[q] = 16 * lane;
    if (u >= AU) {
      const int j = cols[imin(j0 + (u - AU) * 16 + (lane & 15), count - 1)];
      voff[q] = (uint32_t)((j >> 4) * OZ_UNIT + 16 * ((lane >> 4) * 16 + (j & 15)));
    }
  }
  auto issue = [&](int kb) {
    const uint32_t base = lds0 + (uint32_t)((kb % NS) * STAGE);
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
      const int u = q * NW + wave;
      if (u >= AU + BU) break;       // wave-uniform: A's units, then B's
      const void* p = (u < AU) ? (const void*)(Abase + (int64_t)kb * oz_atile(S) + u * OZ_UNIT)
                               : (const void*)(g.B + (int64_t)kb * g.Jb * OZ_UNIT);
      lds_load16_sv(p, voff[q], base + (uint32_t)(u * OZ_UNIT));
    }
  };
  for (int q = 0; q < NS - 1; ++q)
    if (q < nk) issue(q);

  i4_t acc[S][FC];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int c = 0; c < FC; ++c) acc[s][c] = i4_t{0, 0, 0, 0};

  const int oa = ws * S * OZ_UNIT + 16 * lane, ob = (AU + wc * FC) * OZ_UNIT + 16 * lane;
  for (int it = 0; it < nk; ++it) {
    if (wave < FULL) wait_stages<NLD>(min(nk - 1 - it, NS - 2));   // this wave's loads of stage it have landed ...
    else wait_stages<NLD - 1>(min(nk - 1 - it, NS - 2));
    __syncthreads();                              // ... and every wave's; stage (it - 1) % NS is free
    if (it + NS - 1 < nk) issue(it + NS - 1);
    const int8_t* st = smem + (it % NS) * STAGE;
    i4_t bf[FC];
#pragma unroll
    for (int c = 0; c < FC; ++c) bf[c] = *reinterpret_cast<const i4_t*>(st + ob + c * OZ_UNIT);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const i4_t af = *reinterpret_cast<const i4_t*>(st + oa + s * OZ_UNIT);
#pragma unroll
      for (int c = 0; c < FC; ++c) acc[s][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af, bf[c], acc[s][c], 0, 0, 0);
    }
  }

  // the digits' sums, smallest first: one FP64 rounding each, then an exact scaling
  const int i = ti * OZ_BM + ws * 16 + 4 * (lane >> 4);   // the lane's first row
  const int4 e = *reinterpret_cast<const int4*>(g.ex + i);
  double v[FC][4];
#pragma unroll
  for (int c = 0; c < FC; ++c)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      double x = (double)acc[0][c][t];
#pragma unroll
      for (int s = 1; s < S; ++s) x = fma(x, 1.0 / 256.0, (double)acc[s][c][t]);
      v[c][t] = ldexp(x, (t == 0 ? e.x : t == 1 ? e.y : t == 2 ? e.z : e.w) - 7);
    }
  if (g.red_q == 0) {
#pragma unroll
    for (int c = 0; c < FC; ++c) {
      const int j = j0 + (wc * FC + c) * 16 + (lane & 15);
      if (j >= count) continue;
      double2* o = reinterpret_cast<double2*>(g.C + (int64_t)i + (int64_t)cols[j] * g.ldc);
      o[0] = double2{v[c][0], v[c][1]};
      o[1] = double2{v[c][2], v[c][3]};
    }
    return;
  }
  double* red = reinterpret_cast<double*>(smem);   // [strip][QC][192]
  for (int q0 = 0; q0 < g.red_q; q0 += QC) {
    const int qn = min(QC, g.red_q - q0);
    __syncthreads();   // every wave is done with the ring (or with the previous pass)
    for (int qq = 0; qq < qn; ++qq) {
      const int q = q0 + qq;
      const bool norm = q == g.red_q - 1;
      double w[4] = {0.0, 0.0, 0.0, 0.0};
      if (!norm) {
#pragma unroll
        for (int t = 0; t < 4; ++t) w[t] = g.W[(int64_t)(i + t) + (int64_t)q * g.ldw];
      }
      // four SNP groups at a time, whose sums end in the four rows of lanes (past the last group: spare ones)
#pragma unroll
      for (int c0 = 0; c0 < FC; c0 += 4) {
        double x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int c = c0 + u < FC ? c0 + u : FC - 1;
          x[u] = 0.0;
#pragma unroll
          for (int t = 0; t < 4; ++t) x[u] += v[c][t] * (norm ? v[c][t] : w[t]);
        }
        const double s = add_rows32(add_rows16(x[0], x[1]), add_rows16(x[2], x[3]));
        const int c = c0 + (lane >> 4);
        if (c < FC) red[(ws * QC + qq) * BN + (wc * FC + c) * 16 + (lane & 15)] = s;
      }
    }
    __syncthreads();
    for (int f = threadIdx.x; f < qn * BN; f += OZ_THREADS) {   // the strips in order
      const int qq = f / BN, jl = f % BN;
      const double* r = red + qq * BN + jl;
      if (j0 + jl < count)
        g.red_part[(int64_t)(ti * g.red_q + q0 + qq) * g.ncols + cols[j0 + jl]] =
            r[0] + r[QC * BN];
    }
  }
}

// The same product, bitwise, for few SNPs: 32 rows x 64 SNPs per workgroup, eight
// waves of a 16-row strip each (wave & 1) that share the sum over k four ways
// (every fourth k block), so that a row tile's chain of stages is a quarter as
// long and there are no stage barriers: a wave reads its fragments straight from
// memory, the next block's ahead of this one's MFMAs.  The int32 sums are exact, so
// adding the four in LDS in any order gives the same integers; the FP64 steps are
// those of ozaki_i8_kernel.  Up to 512 tiles (two rounds of workgroups), or 256 and
// 384 where there are few stages to share; beyond, the larger tiles' fewer reads
// win.  Times of a block of whole numbers, this kernel's over the other's (n: tiles
// ratio ...): 600: 190 0.88, 247 1.01, 380 1.11, 494 1.18;  1,024: 256 0.83, 320 1.07,
// 448 1.12;  1,500: 282 0.91, 376 1.04, 470 1.06;  2,048: 384 0.94, 512 1.03, 640 1.18;
// 4,096: 256 0.68, 512 0.93, 640 1.16;  8,192: 512 0.78, 768 1.13.
constexpr int OZS_BN = 64, OZS_THREADS = 512, OZS_SPLIT = 4;
inline int small_whole_tiles(int Mt) { return Mt <= 32 ? 256 : Mt <= 64 ? 384 : 512; }

template <int S>
__global__ __launch_bounds__(OZS_THREADS) void ozaki_i8_small_kernel(OzArgs g) {
  constexpr int FC = OZS_BN / 16, QC = 10;
  static_assert(2 * OZS_SPLIT * 64 == OZS_THREADS && FC == OZS_SPLIT, "a wave forms one 16 x 16 block at the end");
  __shared__ int sums[2 * S * FC * 256];           // [strip][digit][SNP group][element][lane]
  __shared__ double red[2 * QC * OZS_BN];
  __shared__ int any;
  const int ti = gridDim.y - 1 - blockIdx.y, tj = blockIdx.x;
  const int j0 = tj * OZS_BN;
  const int count = g.cols.count(g.ncols);
  if (j0 >= count || (g.cols.at && !g.range.holds(count))) return;
  const ColList cols = g.cols.or_all(count, g.ncols);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ws = wave & 1, wk = wave >> 1;
  if (threadIdx.x == 0) any = g.flags.at == nullptr;
  __syncthreads();
  if (g.flags.at && threadIdx.x < OZS_BN && j0 + (int)threadIdx.x < g.ncols &&
      !g.flags.flagged(j0 + threadIdx.x))
    any = 1;
  for (int e = threadIdx.x; e < 2 * S * FC * 256; e += OZS_THREADS) sums[e] = 0;
  __syncthreads();
  if (!any) return;

  const int nk = ti * OZ_BM / OZ_TM + 1;
  const int8_t* A = g.A + (int64_t)(nk - 1) * nk / 2 * oz_atile(S) + ((ti % (OZ_TM / OZ_BM)) * OZ_STRIPS + ws) * (S * OZ_UNIT) +
                    16 * lane;
  uint32_t ob[FC];   // the lane's SNPs and k within a k block of B (SNPs past the end: the last one, dropped)
#pragma unroll
  for (int c = 0; c < FC; ++c) {
    const int j = cols[imin(j0 + 16 * c + (lane & 15), count - 1)];
    ob[c] = (uint32_t)((j >> 4) * OZ_UNIT + 16 * ((lane >> 4) * 16 + (j & 15)));
  }
  i4_t a[2][S], b[2][FC];
  auto load = [&](int kb, int buf) {
#pragma unroll
    for (int s = 0; s < S; ++s) a[buf][s] = *reinterpret_cast<const i4_t*>(A + (int64_t)kb * oz_atile(S) + s * OZ_UNIT);
#pragma unroll
    for (int c = 0; c < FC; ++c)
      b[buf][c] = *reinterpret_cast<const i4_t*>(g.B + (int64_t)kb * g.Jb * OZ_UNIT + ob[c]);
  };
  i4_t acc[S][FC];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int c = 0; c < FC; ++c) acc[s][c] = i4_t{0, 0, 0, 0};
  auto mma = [&](int buf) {
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int c = 0; c < FC; ++c)
        acc[s][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[buf][s], b[buf][c], acc[s][c], 0, 0, 0);
  };
  if (wk < nk) load(wk, 0);
  for (int kb = wk; kb < nk; kb += 2 * OZS_SPLIT) {
    if (kb + OZS_SPLIT < nk) load(kb + OZS_SPLIT, 1);
    mma(0);
    if (kb + 2 * OZS_SPLIT < nk) load(kb + 2 * OZS_SPLIT, 0);
    if (kb + OZS_SPLIT < nk) mma(1);
  }
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int c = 0; c < FC; ++c)
#pragma unroll
      for (int t = 0; t < 4; ++t) atomicAdd(&sums[((ws * S + s) * FC + c) * 256 + t * 64 + lane], acc[s][c][t]);
  __syncthreads();

  // wave (strip ws, SNP group wk)
  const int i = ti * OZ_BM + ws * 16 + 4 * (lane >> 4);
  const int4 e = *reinterpret_cast<const int4*>(g.ex + i);
  double v[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int* at = sums + (ws * S * FC + wk) * 256 + t * 64 + lane;
    double x = (double)at[0];
#pragma unroll
    for (int s = 1; s < S; ++s) x = fma(x, 1.0 / 256.0, (double)at[s * FC * 256]);
    v[t] = ldexp(x, (t == 0 ? e.x : t == 1 ? e.y : t == 2 ? e.z : e.w) - 7);
  }
  if (g.red_q == 0) {
    const int j = j0 + wk * 16 + (lane & 15);
    if (j >= count || (g.flags.at && g.flags.flagged(j))) return;
    double2* o = reinterpret_cast<double2*>(g.C + (int64_t)i + (int64_t)cols[j] * g.ldc);
    o[0] = double2{v[0], v[1]};
    o[1] = double2{v[2], v[3]};
    return;
  }
  for (int q0 = 0; q0 < g.red_q; q0 += QC) {
    const int qn = min(QC, g.red_q - q0);
    __syncthreads();
    for (int qq = 0; qq < qn; ++qq) {
      const int q = q0 + qq;
      const bool norm = q == g.red_q - 1;
      double w[4] = {0.0, 0.0, 0.0, 0.0};
      if (!norm) {
#pragma unroll
        for (int t = 0; t < 4; ++t) w[t] = g.W[(int64_t)(i + t) + (int64_t)q * g.ldw];
      }
      double x = 0.0;
#pragma unroll
      for (int t = 0; t < 4; ++t) x += v[t] * (norm ? v[t] : w[t]);
      x += __shfl_xor(x, 16, 64);
      x += __shfl_xor(x, 32, 64);
      if (lane < 16) red[(ws * QC + qq) * OZS_BN + wk * 16 + lane] = x;
    }
    __syncthreads();
    for (int f = threadIdx.x; f < qn * OZS_BN; f += OZS_THREADS) {
      const int qq = f / OZS_BN, jl = f % OZS_BN;
      if (j0 + jl < count)
        g.red_part[(int64_t)(ti * g.red_q + q0 + qq) * g.ncols + cols[j0 + jl]] =
            red[qq * OZS_BN + jl] + red[(QC + qq) * OZS_BN + jl];
    }
  }
}

}  // namespace gls

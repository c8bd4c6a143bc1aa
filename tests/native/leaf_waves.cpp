// Runs leaf_potrf_trtri_kernel's own source on the CPU, its waves in a given
// order.  Every lane is a coroutine; a wave runs on until all of its lanes wait at
// a workgroup barrier, then the next wave of the order does.  Cross-lane
// instructions wait for the wave's 64 lanes.  A result that depends on the order
// means that waves share LDS words with no barrier between their accesses.
//
//   leaf_waves ORDER < A > L and its inverse     (ORDER: the eight waves, e.g.
//   76543210; A, L, L^-1: 128 x 128 doubles, column-major)
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#define __global__ static
#define __device__
#define __host__
#define __forceinline__ inline
#define __shared__ static
#define __align__(n)
#define __launch_bounds__(n)
#define ext_vector_type(n) vector_size(8 * (n))

using std::max;
using std::min;
struct double2 {
  double x, y;
};
struct Index {
  unsigned x, y, z;
};
static const Index blockIdx{0, 0, 0}, gridDim{1, 1, 1}, blockDim{512, 1, 1};

constexpr int THREADS = 512, LANES = 64, WAVES = THREADS / LANES;

struct Lane {
  ucontext_t ctx;
  std::vector<char> stack;
  int tid = 0;
  int calls = 0;            // cross-lane instructions begun
  bool at_barrier = false, done = false;
};
static Lane lanes[THREADS];
static Lane* self = nullptr;
static ucontext_t scheduler;
static char mail[WAVES][2][LANES][64];   // operands of a wave's last two cross-lane instructions
static int arrived[WAVES][2];

static void yield() { swapcontext(&self->ctx, &scheduler); }
static Index thread_index() { return Index{(unsigned)self->tid, 0, 0}; }
#define threadIdx thread_index()

static void __syncthreads() {
  self->at_barrier = true;
  while (self->at_barrier) yield();
}

// Hands in this lane's operand and waits for the other lanes of its wave.
template <typename T>
static const char (*exchange(const T& v))[64] {
  static_assert(sizeof(T) <= 64, "operand");
  const int w = self->tid / LANES, slot = self->calls++ & 1;
  std::memcpy(mail[w][slot][self->tid % LANES], &v, sizeof v);
  const int full = (self->calls + 1) / 2 * LANES;   // arrivals at this slot once the wave is here
  ++arrived[w][slot];
  while (arrived[w][slot] < full) yield();
  return mail[w][slot];
}
template <typename T>
static T lane_operand(const char (*m)[64], int lane) {
  T v;
  std::memcpy(&v, m[lane], sizeof v);
  return v;
}

static int __builtin_amdgcn_readlane_(int v, int k) { return lane_operand<int>(exchange(v), k); }
#define __builtin_amdgcn_readlane __builtin_amdgcn_readlane_
static int readfirstlane_(int v) { return lane_operand<int>(exchange(v), 0); }
#define __builtin_amdgcn_readfirstlane readfirstlane_
static unsigned long long __ballot(bool b) {
  const char(*m)[64] = exchange<int>(b);
  unsigned long long r = 0;
  for (int l = 0; l < LANES; ++l) r |= (unsigned long long)(lane_operand<int>(m, l) != 0) << l;
  return r;
}
template <typename T>
static T __shfl_xor(T v, int mask, int) {
  return lane_operand<T>(exchange(v), (self->tid % LANES) ^ mask);
}
static int __ffs(unsigned v) { return __builtin_ffs((int)v); }
static double rsq_(double d) { return 1.0 / std::sqrt(d); }
#define __builtin_amdgcn_rsq rsq_
static int __double2loint(double x) {
  uint64_t u;
  std::memcpy(&u, &x, 8);
  return (int)(uint32_t)u;
}
static int __double2hiint(double x) {
  uint64_t u;
  std::memcpy(&u, &x, 8);
  return (int)(u >> 32);
}
static double __hiloint2double(int hi, int lo) {
  const uint64_t u = (uint64_t)(uint32_t)hi << 32 | (uint32_t)lo;
  double x;
  std::memcpy(&x, &u, 8);
  return x;
}
typedef double vec4 __attribute__((vector_size(32)));
struct AB {
  double a, b;
};
// lane l: A[l % 16][l / 16], B[l / 16][l % 16]; result element t: D[l / 16 + 4 t][l % 16]
static vec4 mfma_(double a, double b, vec4 c, int, int, int) {
  const char(*m)[64] = exchange(AB{a, b});
  const int l = self->tid % LANES;
  for (int k = 0; k < 4; ++k)
    for (int t = 0; t < 4; ++t)
      c[t] = std::fma(lane_operand<AB>(m, 16 * k + l / 16 + 4 * t).a, lane_operand<AB>(m, 16 * k + l % 16).b, c[t]);
  return c;
}
#define __builtin_amdgcn_mfma_f64_16x16x4f64 mfma_

#include "setup_kernels.hpp"   // without its inline asm, which only pins values to registers

static double A[128 * 128], Ainv[128 * 128];
static int info = 0;
static void lane_main() {
  gls::leaf_potrf_trtri_kernel(A, Ainv, 128, 0, &info);
  self->done = true;
  for (;;) yield();
}

int main(int argc, char** argv) {
  if (argc != 2 || std::strlen(argv[1]) != WAVES || std::fread(A, 8, 128 * 128, stdin) != 128 * 128) return 2;
  for (int t = 0; t < THREADS; ++t) {
    Lane& l = lanes[t];
    l.tid = t;
    l.stack.resize(64 * 1024);
    getcontext(&l.ctx);
    l.ctx.uc_stack.ss_sp = l.stack.data();
    l.ctx.uc_stack.ss_size = l.stack.size();
    l.ctx.uc_link = &scheduler;
    makecontext(&l.ctx, lane_main, 0);
  }
  for (;;) {
    for (int o = 0; o < WAVES; ++o) {
      Lane* w = lanes + LANES * (argv[1][o] - '0');
      auto waits = [](const Lane& l) { return l.at_barrier || l.done; };
      while (!std::all_of(w, w + LANES, waits))
        for (int l = 0; l < LANES; ++l)
          if (!waits(w[l])) {
            self = w + l;
            swapcontext(&scheduler, &self->ctx);
          }
    }
    if (std::all_of(lanes, lanes + THREADS, [](const Lane& l) { return l.done; })) break;
    for (Lane& l : lanes) l.at_barrier = false;
  }
  if (info != 0) return 3;
  std::fwrite(A, 8, 128 * 128, stdout);
  std::fwrite(Ainv, 8, 128 * 128, stdout);
  return 0;
}

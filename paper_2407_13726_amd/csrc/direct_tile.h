// Tiles of trmm_direct.hip and ttm_direct.hip, whose wavefronts take both operands straight from memory: what a lane reads of a window of 16
// values of the reduction index, how a window is multiplied, where the results are -- and how the wavefronts of a workgroup add up theirs.
#pragma once
#include "split3.h"

namespace dastac {

constexpr int kWin = 16;  // values of the reduction index per window

// 32 rows by 32 columns in single precision on the bf16 matrix cores, operands split in three in registers (split3.h; two accumulators).  Lane l: row and
// column l % 32 and, of a window, the values 8 (l / 32) .. + 7.
struct SplitTile {
  typedef float Type, Sum;  // of the operands and results; in which wavefronts add up
  static constexpr bool kSplit = true;
  static constexpr int kSets = 1;
  static constexpr int kRows = 32, kOwn = 8, kRegs = 16, kCols = 1;
  struct Raw {
    float u[8], b[kCols][8];
  };
  struct Sums {
    f16v hi, lo;
  };
  __device__ static int row(int lane) { return lane & 31; }
  __device__ static int first(int lane) { return 8 * (lane >> 5); }
  __device__ static int column(int lane, int) { return lane & 31; }
  __device__ static void load(const float *p, float (&o)[8]) {
    const f4a x = *reinterpret_cast<const f4u *>(p), y = *reinterpret_cast<const f4u *>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = x[e], o[4 + e] = y[e];
  }
  __device__ static void clear(Sums &s) {
#pragma unroll
    for (int v = 0; v < 16; ++v) s.hi[v] = 0.0f, s.lo[v] = 0.0f;
  }
  // next() requests the next window, when the raw values are used up
  template <typename F>
  __device__ static void multiply(const Raw &o, Sums &s, F next) {
    const Parts a = split3x8(o.u);
    const Parts b = split3x8(o.b[0]);
    __builtin_amdgcn_sched_barrier(0);
    next();
    s.lo = mma_bf16(a.v[2], b.v[0], s.lo);
    s.hi = mma_bf16(a.v[0], b.v[0], s.hi);
    s.lo = mma_bf16(a.v[0], b.v[2], s.lo);
    s.lo = mma_bf16(a.v[1], b.v[1], s.lo);
    s.lo = mma_bf16(a.v[1], b.v[0], s.lo);
    s.lo = mma_bf16(a.v[0], b.v[1], s.lo);
  }
  // the same window on the fp32 instructions
  __device__ static void plain(const Raw &o, Sums &s) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s.hi = __builtin_amdgcn_mfma_f32_32x32x2f32(o.u[e], o.b[0][e], s.hi, 0, 0, 0);
  }
  // false: not all of this lane's sums are finite
  __device__ static bool finish(Sums &s) {
    float z = 0.0f;
    s.hi += s.lo;
#pragma unroll
    for (int v = 0; v < 16; ++v) z = __builtin_fmaf(s.hi[v], 0.0f, z);
    s.hi *= kSplitDown;
    return z == z;
  }
  __device__ static float at(const Sums &s, int v) { return s.hi[v]; }
  __device__ static void add(Sums &s, int v, float x) { s.hi[v] += x; }
  __device__ static int row_of(int v, int lane) { return 8 * (v / 4) + 4 * (lane >> 5) + v % 4; }
  __device__ static int col_of(int, int lane) { return lane & 31; }
};

// What v_mfma_f32_16x16x4_f32 and v_mfma_f64_16x16x4_f64 differ in.
template <typename A>
struct Native16;
template <>
struct Native16<float> {
  typedef f4a acc;
  __device__ static acc mma(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row_of(int v, int lane) { return 4 * (lane >> 4) + v; }
};
template <>
struct Native16<double> {
  typedef d4v acc;
  __device__ static acc mma(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row_of(int v, int lane) { return 4 * v + (lane >> 4); }
};
__device__ inline void load4(const float *p, float (&o)[4]) {
  const f4a x = *reinterpret_cast<const f4u *>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = x[e];
}
__device__ inline void load4(const double *p, double (&o)[4]) {
  const d2a x = *reinterpret_cast<const d2u *>(p), y = *reinterpret_cast<const d2u *>(p + 2);
  o[0] = x[0], o[1] = x[1], o[2] = y[0], o[3] = y[1];
}

// 16 rows by 32 columns, two results side by side, of operands T on the instructions that add up in A.  Lane l: row l % 16 and the values 4 (l / 16) ..
// + 3 of a window; columns l % 16 and 16 + l % 16.  Single precision keeps eight sums where it adds up in itself, one for each instruction of two
// windows, and wavefronts add up in double precision, so that sums are no further off than the split's (TRMM n=1000, m=32 against 64 bits: one sum 1.3e-7,
// four 6.7e-8, the split 7.4e-8).
template <typename T, typename A>
struct NativeTile {
  typedef T Type;
  typedef double Sum;
  static constexpr bool kSplit = false;
  static constexpr int kRows = 16, kOwn = 4, kRegs = 8, kCols = 2;
  static constexpr int kSets = sizeof(A) == 4 ? 8 : 1;
  struct Raw {
    T u[4], b[kCols][4];
  };
  struct Sums {
    typename Native16<A>::acc v[2][kSets];
  };
  __device__ static int row(int lane) { return lane & 15; }
  __device__ static int first(int lane) { return 4 * (lane >> 4); }
  __device__ static int column(int lane, int c) { return 16 * c + (lane & 15); }
  __device__ static void load(const T *p, T (&o)[4]) { load4(p, o); }
  __device__ static void clear(Sums &s) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int e = 0; e < kSets; ++e)
#pragma unroll
        for (int v = 0; v < 4; ++v) s.v[c][e][v] = A(0);
  }
  __device__ static void plain(const Raw &o, Sums &s, int odd = 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        auto &acc = s.v[c][kSets == 1 ? 0 : e + 4 * odd];
        acc = Native16<A>::mma(o.u[e], o.b[c][e], acc);
      }
  }
  template <typename F>
  __device__ static void multiply(const Raw &o, Sums &s, F next, int odd = 0) {
    const Raw own = o;
    next();
    plain(own, s, odd);
  }
  __device__ static bool finish(Sums &s) {
    A z = A(0);
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      if (kSets == 8) {
#pragma unroll
        for (int e = 0; e < 4; ++e) s.v[v / 4][e][v % 4] += s.v[v / 4][e + kSets / 2][v % 4];
      }
#pragma unroll
      for (int e = 0; e < (kSets + 1) / 2; ++e) z = __builtin_elementwise_fma(s.v[v / 4][e][v % 4], A(0), z);
    }
    return z == z;
  }
  __device__ static double at(const Sums &s, int v) {
    double x = s.v[v / 4][0][v % 4];
#pragma unroll
    for (int e = 1; e < kSets / 2; ++e) x += s.v[v / 4][e][v % 4];
    return x;
  }
  __device__ static void add(Sums &s, int v, T x) { s.v[v / 4][0][v % 4] += x; }
  __device__ static int row_of(int v, int lane) { return Native16<A>::row_of(v % 4, lane); }
  __device__ static int col_of(int v, int lane) { return 16 * (v / 4) + (lane & 15); }
};

// Adds up the sums number 0 .. REGS-1 of all WX wavefronts, at(v) a lane, and hands them to put(v, sum), each to one wavefront: the upper half of the
// wavefronts leave their sums, the lower half add their own, then all add up the slots.
// (One wavefront hands its own to put.)
template <int WX, int REGS, typename T, typename At, typename Put>
__device__ __attribute__((always_inline)) inline void add_up(int wave, int lane, At at, Put put) {
  if constexpr (WX == 1) {
#pragma unroll
    for (int v = 0; v < REGS; ++v) put(v, at(v));
    return;
  }
  constexpr int kSlots = WX > 1 ? WX / 2 : 1;
  __shared__ T slots[kSlots][REGS * 64];
  T *mine = slots[wave % kSlots];
  if (wave >= kSlots) {
#pragma unroll
    for (int v = 0; v < REGS; ++v) mine[v * 64 + lane] = at(v);
  }
  __syncthreads();
  if (wave < kSlots) {
#pragma unroll
    for (int v = 0; v < REGS; ++v) mine[v * 64 + lane] += at(v);
  }
  __syncthreads();
#pragma unroll
  for (int v0 = 0; v0 < REGS; v0 += WX) {
    const int v = v0 + wave;
    if (REGS % WX != 0 && v >= REGS) return;
    T sum = slots[0][v * 64 + lane];
#pragma unroll
    for (int s = 1; s < kSlots; ++s) sum += slots[s][v * 64 + lane];
    put(v, sum);
  }
}

}  // namespace dastac

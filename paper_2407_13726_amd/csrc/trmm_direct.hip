// C := U B for small products in one launch: every wavefront takes operands straight from memory, every tile of C is written once.
//
// A workgroup owns 32 (fp64: 16) rows by 32 columns of C; its WX wavefronts take every WX-th window of 16 values of k, from the row
// block's first row to n, and add their sums up through LDS.  Nothing is staged and nothing cleared, and equal calls give equal bits.  A lane reads 32
// contiguous bytes of its own packed row and its column of B's rows.  In single precision both are split in three bf16 parts in registers
// (split3.h; two accumulators, so that the error is that of the 64 x 64 tiles of trmm.hip).
// The last window is moved back to end with the matrix; what it repeats, and what lies left of the diagonal, is made zero in U.
//
// Bound by latency (windows of a wavefront one after the other) and, in single precision, by the vector instructions of the split; the tiles of
// trmm.hip, which share what they split, take over for larger products (run_tiles there).
// us a call, before (two launches) and here: fp32 n=256, m=100 9.4, 4.0; n=1000, m=100 13.0, 7.4; n=2000, m=200 21.1, 15.3; fp64 n=500, m=200 10.7,
// 5.7; n=1500, m=100 18.1, 12.7.  Two windows on their way instead of one: slower (fp32 spills, fp64 n=1500, m=100 14.5).
#include "split3.h"

using namespace dastac;

namespace {

constexpr int kWin = 16;  // values of k per window

template <typename T>
struct Rows;

// Lane l: row l % 32 and, of a window, the values 8 (l / 32) .. + 7; column l % 32.
template <>
struct Rows<float> {
  static constexpr int kRows = 32, kOwn = 8, kRegs = 16, kCols = 1;
  struct Raw {
    float u[8], b[8][kCols];
  };
  struct Sums {
    f16v hi, lo;
  };
  __device__ static int row(int lane) { return lane & 31; }
  __device__ static int first(int lane) { return 8 * (lane >> 5); }
  __device__ static int column(int lane, int) { return lane & 31; }
  __device__ static void load_u(const float *p, Raw &o) {
    const f4a x = *reinterpret_cast<const f4u *>(p), y = *reinterpret_cast<const f4u *>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) o.u[e] = x[e], o.u[4 + e] = y[e];
  }
  __device__ static void clear(Sums &s) {
#pragma unroll
    for (int v = 0; v < 16; ++v) s.hi[v] = 0.0f, s.lo[v] = 0.0f;
  }
  // next() requests the next window, when the raw values are used up
  template <typename F>
  __device__ static void multiply(const Raw &o, Sums &s, F next) {
    const Parts a = split3x8(o.u);
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = o.b[e][0];
    const Parts b = split3x8(x);
    __builtin_amdgcn_sched_barrier(0);
    next();
    s.lo = mma_bf16(a.v[2], b.v[0], s.lo);
    s.hi = mma_bf16(a.v[0], b.v[0], s.hi);
    s.lo = mma_bf16(a.v[0], b.v[2], s.lo);
    s.lo = mma_bf16(a.v[1], b.v[1], s.lo);
    s.lo = mma_bf16(a.v[1], b.v[0], s.lo);
    s.lo = mma_bf16(a.v[0], b.v[1], s.lo);
  }
  __device__ static void plain(const Raw &o, Sums &s) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s.hi = __builtin_amdgcn_mfma_f32_32x32x2f32(o.u[e], o.b[e][0], s.hi, 0, 0, 0);
  }
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

// v_mfma_f64_16x16x4_f64, two side by side.  Lane l: row l % 16 and the values 4 (l / 16) .. + 3; columns l % 16 and 16 + l % 16.
template <>
struct Rows<double> {
  static constexpr int kRows = 16, kOwn = 4, kRegs = 8, kCols = 2;
  struct Raw {
    double u[4], b[4][kCols];
  };
  struct Sums {
    d4v v[2];
  };
  __device__ static int row(int lane) { return lane & 15; }
  __device__ static int first(int lane) { return 4 * (lane >> 4); }
  __device__ static int column(int lane, int c) { return 16 * c + (lane & 15); }
  __device__ static void load_u(const double *p, Raw &o) {
    const d2a x = *reinterpret_cast<const d2u *>(p), y = *reinterpret_cast<const d2u *>(p + 2);
    o.u[0] = x[0], o.u[1] = x[1], o.u[2] = y[0], o.u[3] = y[1];
  }
  __device__ static void clear(Sums &s) { s.v[0] = s.v[1] = d4v{0.0, 0.0, 0.0, 0.0}; }
  __device__ static void plain(const Raw &o, Sums &s) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < 2; ++c) s.v[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.u[e], o.b[e][c], s.v[c], 0, 0, 0);
  }
  template <typename F>
  __device__ static void multiply(const Raw &o, Sums &s, F next) {
    const Raw own = o;
    next();
    plain(own, s);
  }
  __device__ static bool finish(Sums &s) {
    double z = 0.0;
#pragma unroll
    for (int v = 0; v < 8; ++v) z = __builtin_fma(s.v[v / 4][v % 4], 0.0, z);
    return z == z;
  }
  __device__ static double at(const Sums &s, int v) { return s.v[v / 4][v % 4]; }
  __device__ static void add(Sums &s, int v, double x) { s.v[v / 4][v % 4] += x; }
  __device__ static int row_of(int v, int lane) { return 4 * (v % 4) + (lane >> 4); }
  __device__ static int col_of(int v, int lane) { return 16 * (v / 4) + (lane & 15); }
};

template <typename T, int WX>
__global__ __launch_bounds__(64 * WX) __attribute__((amdgpu_waves_per_eu(4, 4)))
void trmm_direct_kernel(int n, int m, const T *__restrict__ U, const T *__restrict__ B, int64_t ldb, T *__restrict__ C, int64_t ldc, int ncb) {
  typedef Rows<T> S;
  constexpr int kSlots = WX / 2;
  __shared__ T slots[kSlots][S::kRegs * 64];
  // Row blocks are dealt to the eight XCDs in turn, longest first, the column blocks of one are neighbours there: they read the same rows of U.
  const int xcd = blockIdx.x & 7, slot = (int)(blockIdx.x >> 3);
  const int i0 = uniform32(S::kRows * (8 * (slot / ncb) + xcd)), c0 = uniform32(32 * (slot % ncb));
  if (i0 >= n) return;
  const int lane = threadIdx.x & 63, wave = uniform32(threadIdx.x >> 6);
  const int i = i0 + S::row(lane) < n ? i0 + S::row(lane) : n - 1;
  const T *const urow = U + (tri_row_start(n, i) - i + S::first(lane));  // element k of this lane's row is U(i, k + first)
  const T *bcol[S::kCols];
#pragma unroll
  for (int c = 0; c < S::kCols; ++c) {
    const int col = c0 + S::column(lane, c) < m ? c0 + S::column(lane, c) : m - 1;
    bcol[c] = B + (int64_t)S::first(lane) * ldb + col;
  }
  const int windows = (n - i0 + kWin - 1) / kWin;
  auto begins = [&](int w) { return i0 + kWin * w; };                                      // the window's own values of k
  auto start = [&](int w) { return begins(w) + kWin <= n ? begins(w) : n - kWin; };      // where it is read
  auto load = [&](int w, typename S::Raw &o) __attribute__((always_inline)) {
    const int k = start(w);
    S::load_u(urow + k, o);
#pragma unroll
    for (int e = 0; e < S::kOwn; ++e)
#pragma unroll
      for (int c = 0; c < S::kCols; ++c) o.b[e][c] = bcol[c][(int64_t)(k + e) * ldb];
  };
  auto meets_edge = [&](int w) { return w < S::kRows / kWin || begins(w) != start(w); };
  auto mask = [&](int w, int least, typename S::Raw &o) __attribute__((always_inline)) {  // U's values left of `least` and of the window's own
    const int k = start(w) + S::first(lane), from = least > begins(w) ? least : begins(w);
#pragma unroll
    for (int e = 0; e < S::kOwn; ++e) o.u[e] = k + e < from ? T(0) : o.u[e];
  };
  typename S::Sums acc;
  S::clear(acc);
  typename S::Raw raw;
  if (wave < windows) load(wave, raw);
  for (int w = wave; w < windows; w += WX) {
    if (meets_edge(w)) mask(w, i, raw);
    S::multiply(raw, acc, [&] { load(w + WX < windows ? w + WX : w, raw); });
  }
  // Operands that the split cannot hold, results that are not finite, or a zero left of the diagonal that met a non-finite row of B: once more
  // on the instructions of the type, what meets the diagonal element by element.
  if (!__all(S::finish(acc))) {
    S::clear(acc);
    for (int w = wave; w < windows; w += WX) {
      if (w < S::kRows / kWin) {
        for (int k = begins(w); k < begins(w) + kWin && k < n; ++k)
#pragma unroll
          for (int v = 0; v < S::kRegs; ++v) {
            const int r = i0 + S::row_of(v, lane), col = c0 + S::col_of(v, lane);
            if (r <= k && r < n && col < m) S::add(acc, v, U[tri_row_start(n, r) - r + k] * B[(int64_t)k * ldb + col]);
          }
      } else {
        load(w, raw);
        if (begins(w) != start(w)) {
          const int k = start(w) + S::first(lane);
          mask(w, 0, raw);
#pragma unroll
          for (int e = 0; e < S::kOwn; ++e)
#pragma unroll
            for (int c = 0; c < S::kCols; ++c) raw.b[e][c] = k + e < begins(w) ? T(0) : raw.b[e][c];
        }
        S::plain(raw, acc);
      }
    }
  }
  // the upper half of the wavefronts leave their sums, the lower half add their own, then all add up the slots and write
  T *mine = slots[wave % kSlots];
  if (wave >= kSlots) {
#pragma unroll
    for (int v = 0; v < S::kRegs; ++v) mine[v * 64 + lane] = S::at(acc, v);
  }
  __syncthreads();
  if (wave < kSlots) {
#pragma unroll
    for (int v = 0; v < S::kRegs; ++v) mine[v * 64 + lane] += S::at(acc, v);
  }
  __syncthreads();
  if (wave >= S::kRegs) return;
#pragma unroll
  for (int v0 = 0; v0 < S::kRegs; v0 += WX) {
    const int v = v0 + wave;
    if (v >= S::kRegs) break;
    T sum = slots[0][v * 64 + lane];
#pragma unroll
    for (int s = 1; s < kSlots; ++s) sum += slots[s][v * 64 + lane];
    const int r = i0 + S::row_of(v, lane), col = c0 + S::col_of(v, lane);
    if (r < n && col < m) C[(int64_t)r * ldc + col] = sum;
  }
}

template <typename T, int WX>
int launch(int64_t n, int64_t m, const T *U, const T *B, int64_t ldb, T *C, int64_t ldc, hipStream_t st) {
  const int64_t nrb = ceil_div(ceil_div(n, Rows<T>::kRows), 8) * 8, ncb = ceil_div(m, 32);
  trmm_direct_kernel<T, WX><<<(unsigned)(nrb * ncb), 64 * WX, 0, st>>>((int)n, (int)m, U, B, ldb, C, ldc, (int)ncb);
  return launch_status();
}

// Sixteen wavefronts shorten a workgroup's chain of windows while few workgroups share a compute unit, eight waste less of it otherwise (us, eight and
// sixteen: fp32 n=3000, m=100, 376 workgroups 21.8, 17.5; m=200, 658 25.5, 27.7; n=1000, m=200, 224 8.1, 7.5; m=400, 416 9.8, 10.9; fp64 n=1500, m=64, 188
// 11.9, 12.3; m=100, 376 15.4, 12.7; m=200, 658 18.5, 21.3).
template <typename T>
int run(int64_t n, int64_t m, const T *U, const T *B, int64_t ldb, T *C, int64_t ldc, void *stream) {
  const int64_t groups = ceil_div(n, Rows<T>::kRows) * ceil_div(m, 32);
  const bool wide = sizeof(T) == 4 ? n >= 500 && groups <= 512 && groups <= n / 4 + 100 : n >= 1000 && groups > 256 && groups <= 512;
  return wide ? launch<T, 16>(n, m, U, B, ldb, C, ldc, (hipStream_t)stream) : launch<T, 8>(n, m, U, B, ldb, C, ldc, (hipStream_t)stream);
}

}  // namespace

int dastac::trmm_direct(int64_t n, int64_t m, const float *U, const float *B, int64_t ldb, float *C, int64_t ldc, void *stream) {
  return run(n, m, U, B, ldb, C, ldc, stream);
}
int dastac::trmm_direct(int64_t n, int64_t m, const double *U, const double *B, int64_t ldb, double *C, int64_t ldc, void *stream) {
  return run(n, m, U, B, ldb, C, ldc, stream);
}

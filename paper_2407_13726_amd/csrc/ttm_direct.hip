// The running example for few packed rows in one layer: Ap[p, k] = sum_l Bp[p, l] C[k, l], operands straight from memory (ttm.hip has the rule, and the
// kernels for more rows).
//
// A workgroup owns 32 (fp64: 16) packed rows by 32 columns; its WX wavefronts take every WX-th window of 16 values of l and add their sums up through LDS,
// where a workgroup of ttm.hip walks all of l in one chain of staged steps.  A lane reads 32 contiguous bytes of its own row of Bp and of C.  In single
// precision both are split in three bf16 parts in registers (split3.h, two accumulators, as in ttm.hip).  The last window is moved back to end with l;
// what it repeats is made zero.  Bound by latency: us a call, before and here:
// fp32 n=24, Q=K=500 23.2, 5.2; n=60, Q=250, K=60 12.4, 4.0; n=90, Q=K=100 9.1, 4.2; fp64 n=24, Q=K=500 57.6, 11.2; n=40, Q=260, K=112 28.4, 4.3.
#include "split3.h"

using namespace dastac;

namespace {

constexpr int kWin = 16;  // values of l per window

template <typename T>
struct Rows;

// Lane t: row and column t % 32 and, of a window, the values 8 (t / 32) .. + 7.
template <>
struct Rows<float> {
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
  __device__ static void plain(const Raw &o, Sums &s) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s.hi = __builtin_amdgcn_mfma_f32_32x32x2f32(o.u[e], o.b[0][e], s.hi, 0, 0, 0);
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
  __device__ static int row_of(int v, int lane) { return 8 * (v / 4) + 4 * (lane >> 5) + v % 4; }
  __device__ static int col_of(int, int lane) { return lane & 31; }
};

// v_mfma_f64_16x16x4_f64, two side by side.  Lane t: row t % 16 and the values 4 (t / 16) .. + 3; columns t % 16 and 16 + t % 16.
template <>
struct Rows<double> {
  static constexpr int kRows = 16, kOwn = 4, kRegs = 8, kCols = 2;
  struct Raw {
    double u[4], b[kCols][4];
  };
  struct Sums {
    d4v v[2];
  };
  __device__ static int row(int lane) { return lane & 15; }
  __device__ static int first(int lane) { return 4 * (lane >> 4); }
  __device__ static int column(int lane, int c) { return 16 * c + (lane & 15); }
  __device__ static void load(const double *p, double (&o)[4]) {
    const d2a x = *reinterpret_cast<const d2u *>(p), y = *reinterpret_cast<const d2u *>(p + 2);
    o[0] = x[0], o[1] = x[1], o[2] = y[0], o[3] = y[1];
  }
  __device__ static void clear(Sums &s) { s.v[0] = s.v[1] = d4v{0.0, 0.0, 0.0, 0.0}; }
  __device__ static void plain(const Raw &o, Sums &s) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < 2; ++c) s.v[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.u[e], o.b[c][e], s.v[c], 0, 0, 0);
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
  __device__ static int row_of(int v, int lane) { return 4 * (v % 4) + (lane >> 4); }
  __device__ static int col_of(int v, int lane) { return 16 * (v / 4) + (lane & 15); }
};

template <typename T, int WX>
__global__ __launch_bounds__(64 * WX) __attribute__((amdgpu_waves_per_eu(4, 4)))
void ttm_direct_kernel(int rows, int Q, int K, const T *__restrict__ Bp, const T *__restrict__ C, int64_t ldc, T *__restrict__ Ap, int ncb) {
  typedef Rows<T> S;
  constexpr int kSlots = WX / 2;
  __shared__ T slots[kSlots][S::kRegs * 64];
  const int p0 = uniform32(S::kRows * (int)(blockIdx.x / (unsigned)ncb)), c0 = uniform32(32 * (int)(blockIdx.x % (unsigned)ncb));
  const int lane = threadIdx.x & 63, wave = uniform32(threadIdx.x >> 6);
  const int p = p0 + S::row(lane) < rows ? p0 + S::row(lane) : rows - 1;  // rows and columns past the last are read as the last and not written
  const T *const brow = Bp + ((int64_t)p * Q + S::first(lane));
  const T *crow[S::kCols];
#pragma unroll
  for (int c = 0; c < S::kCols; ++c) {
    const int col = c0 + S::column(lane, c) < K ? c0 + S::column(lane, c) : K - 1;
    crow[c] = C + ((int64_t)col * ldc + S::first(lane));
  }
  const int windows = (Q + kWin - 1) / kWin;
  auto start = [&](int w) { return kWin * w + kWin <= Q ? kWin * w : Q - kWin; };  // where window w is read
  auto load = [&](int w, typename S::Raw &o) __attribute__((always_inline)) {
    const int l = start(w);
    S::load(brow + l, o.u);
#pragma unroll
    for (int c = 0; c < S::kCols; ++c) S::load(crow[c] + l, o.b[c]);
  };
  auto mask = [&](int w, typename S::Raw &o) __attribute__((always_inline)) {  // what the window before has had
    const int own = kWin * w - start(w) - S::first(lane);
#pragma unroll
    for (int e = 0; e < S::kOwn; ++e) {
      o.u[e] = e < own ? T(0) : o.u[e];
#pragma unroll
      for (int c = 0; c < S::kCols; ++c) o.b[c][e] = e < own ? T(0) : o.b[c][e];
    }
  };
  typename S::Sums acc;
  S::clear(acc);
  typename S::Raw raw;
  if (wave < windows) load(wave, raw);
  for (int w = wave; w < windows; w += WX) {
    if (kWin * w != start(w)) mask(w, raw);
    S::multiply(raw, acc, [&] { load(w + WX < windows ? w + WX : w, raw); });
  }
  // operands that the split cannot hold, or results that are not finite: once more on the fp32 instructions
  if (sizeof(T) == 4 && !__all(S::finish(acc))) {
    S::clear(acc);
    for (int w = wave; w < windows; w += WX) {
      load(w, raw);
      if (kWin * w != start(w)) mask(w, raw);
      S::plain(raw, acc);
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
    const int r = p0 + S::row_of(v, lane), col = c0 + S::col_of(v, lane);
    if (r < rows && col < K) Ap[(int64_t)r * K + col] = sum;
  }
}

template <typename T, int WX>
int launch(int64_t rows, int64_t Q, int64_t K, const T *Bp, const T *C, int64_t ldc, T *Ap, hipStream_t st) {
  const int64_t ncb = ceil_div(K, 32);
  ttm_direct_kernel<T, WX><<<(unsigned)(ceil_div(rows, Rows<T>::kRows) * ncb), 64 * WX, 0, st>>>((int)rows, (int)Q, (int)K, Bp, C, ldc, Ap, (int)ncb);
  return launch_status();
}

// Two wavefronts where there are few windows or many workgroups to fill the chip, else four (us, two and four: fp32 n=90, Q=K=100, 512 workgroups 5.1,
// 4.2; n=130, Q=500, K=40, 534 12.0, 13.8; n=130, Q=K=64 4.7, 5.3; fp64 n=90, Q=300, K=32, 256 6.2, 4.9; Q=K=100, 1024 6.6, 7.5).
template <typename T>
int run(int64_t rows, int64_t Q, int64_t K, const T *Bp, const T *C, int64_t ldc, T *Ap, void *stream) {
  const int64_t groups = ceil_div(rows, Rows<T>::kRows) * ceil_div(K, 32);
  return Q <= 3 * kWin || groups > 512 ? launch<T, 2>(rows, Q, K, Bp, C, ldc, Ap, (hipStream_t)stream)
                                       : launch<T, 4>(rows, Q, K, Bp, C, ldc, Ap, (hipStream_t)stream);
}

}  // namespace

int dastac::ttm_direct(int64_t rows, int64_t Q, int64_t K, const float *Bp, const float *C, int64_t ldc, float *Ap, void *stream) {
  return run(rows, Q, K, Bp, C, ldc, Ap, stream);
}
int dastac::ttm_direct(int64_t rows, int64_t Q, int64_t K, const double *Bp, const double *C, int64_t ldc, double *Ap, void *stream) {
  return run(rows, Q, K, Bp, C, ldc, Ap, stream);
}

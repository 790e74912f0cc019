// The running example for few packed rows in one layer: Ap[p, k] = sum_l Bp[p, l] C[k, l], operands straight from memory (ttm.hip has the rule, and the
// kernels for more rows).
//
// A workgroup owns 32 or 16 packed rows by 32 columns; its WX wavefronts take every WX-th window of 16 values of l and add their sums up through LDS,
// where a workgroup of ttm.hip walks all of l in one chain of staged steps.  A lane reads a few consecutive elements of its own row of Bp and of C
// (direct_tile.h).  Single precision splits both in three bf16 parts in registers, with two accumulators, as ttm.hip does -- and where that kernel keeps to the
// type's own products (Q <= 32 in one layer), so does this one, with sums in double precision: a product of two floats is exact there.  The last window is moved
// back to end with l; what it repeats is made zero.  Bound by latency: us a call, before and here:
// fp32 n=24, Q=K=500 23.2, 5.2; n=60, Q=250, K=60 12.4, 4.0; n=90, Q=K=100 9.1, 4.2; n=60, Q=32, K=500 5.4, 5.2 (split 5.2); fp64 n=24, Q=K=500 57.6, 11.2;
// n=40, Q=260, K=112 28.4, 4.3.
#include "direct_tile.h"

using namespace dastac;

namespace {

template <typename S, int WX, typename T = typename S::Type>
__global__ __launch_bounds__(64 * WX) __attribute__((amdgpu_waves_per_eu(4, 4)))
void ttm_direct_kernel(int rows, int Q, int K, const T *__restrict__ Bp, const T *__restrict__ C, int64_t ldc, T *__restrict__ Ap, int ncb) {
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
  if (S::kSplit && !__all(S::finish(acc))) {
    S::clear(acc);
    for (int w = wave; w < windows; w += WX) {
      load(w, raw);
      if (kWin * w != start(w)) mask(w, raw);
      S::plain(raw, acc);
    }
  }
  add_up<WX, S::kRegs, typename S::Sum>(
      wave, lane, [&](int v) { return S::at(acc, v); },
      [&](int v, typename S::Sum sum) {
        const int r = p0 + S::row_of(v, lane), col = c0 + S::col_of(v, lane);
        if (r < rows && col < K) Ap[(int64_t)r * K + col] = (T)sum;
      });
}

template <typename S, int WX, typename T = typename S::Type>
int launch(int64_t rows, int64_t Q, int64_t K, const T *Bp, const T *C, int64_t ldc, T *Ap, hipStream_t st) {
  const int64_t ncb = ceil_div(K, 32);
  ttm_direct_kernel<S, WX><<<(unsigned)(ceil_div(rows, S::kRows) * ncb), 64 * WX, 0, st>>>((int)rows, (int)Q, (int)K, Bp, C, ldc, Ap, (int)ncb);
  return launch_status();
}

// One wavefront where two windows are all there is and workgroups are many (fp32 n=60, Q=32, K=500 5.2 us, with two 5.8).  Two where there are few windows or many workgroups to fill the chip, else four (us, two and four: fp32 n=90, Q=K=100, 512 workgroups 5.1,
// 4.2; n=130, Q=500, K=40, 534 12.0, 13.8; n=130, Q=K=64 4.7, 5.3; fp64 n=90, Q=300, K=32, 256 6.2, 4.9; Q=K=100, 1024 6.6, 7.5).
template <typename S, typename T = typename S::Type>
int run(int64_t rows, int64_t Q, int64_t K, const T *Bp, const T *C, int64_t ldc, T *Ap, void *stream) {
  const int64_t groups = ceil_div(rows, S::kRows) * ceil_div(K, 32);
  if (!S::kSplit && sizeof(T) == 4 && groups > 1024) return launch<S, 1>(rows, Q, K, Bp, C, ldc, Ap, (hipStream_t)stream);
  return Q <= 3 * kWin || groups > 512 ? launch<S, 2>(rows, Q, K, Bp, C, ldc, Ap, (hipStream_t)stream)
                                       : launch<S, 4>(rows, Q, K, Bp, C, ldc, Ap, (hipStream_t)stream);
}

}  // namespace

int dastac::ttm_direct(int64_t rows, int64_t Q, int64_t K, const float *Bp, const float *C, int64_t ldc, float *Ap, void *stream) {
  return Q <= 2 * kWin && ceil_div(rows, 64) * ceil_div(K, 128) <= 256 ? run<NativeTile<float, double>>(rows, Q, K, Bp, C, ldc, Ap, stream)
                                       : run<SplitTile>(rows, Q, K, Bp, C, ldc, Ap, stream);
}
int dastac::ttm_direct(int64_t rows, int64_t Q, int64_t K, const double *Bp, const double *C, int64_t ldc, double *Ap, void *stream) {
  return run<NativeTile<double, double>>(rows, Q, K, Bp, C, ldc, Ap, stream);
}

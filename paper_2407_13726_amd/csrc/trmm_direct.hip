// C := U B for small products in one launch: every wavefront takes operands straight from memory, every tile of C is written once.
//
// A workgroup owns 32 or 16 rows by 32 columns of C; its WX wavefronts take every WX-th window of 16 values of k, from the row
// block's first row to n, and add their sums up through LDS.  Nothing is staged and nothing cleared, and equal calls give equal bits.  A lane reads a few
// consecutive elements of its own packed row and its column of B's rows (direct_tile.h).  With more than 32 columns single precision splits both in three
// bf16 parts in registers, with two accumulators, so that the error is that of the 64 x 64 tiles of trmm.hip; up to 32 columns, which run on the fp32
// instructions there, they do so here, so that a sum of one term is its rounded product.
// The last window is moved back to end with the matrix; what it repeats, and what lies left of the diagonal, is made zero in U.
//
// Bound by latency (windows of a wavefront one after the other) and, where operands are split, by the vector instructions of the split; the tiles of
// trmm.hip, which share what they split, take over for larger products (run_tiles there).
// us a call, before (two launches) and here: fp32 n=256, m=100 9.4, 4.0; n=1000, m=100 13.0, 7.4; n=2000, m=200 21.1, 15.3; up to 32 columns n=1000, m=20 9.6,
// 6.9 (split 7.3); n=1500, m=20 11.3, 8.5 (split 9.3); fp64 n=500, m=200 10.7, 5.7; n=1500, m=100 18.1, 12.7.  Two windows on their way instead of
// one: slower (fp32 spills, fp64 n=1500, m=100 14.5).  Up to 32 columns with sums in double precision (error 6.7e-8 at n=1000, here 5.9e-8): n=1000 8.0 us, n=2048
// 13.1; with four sums a column 6.3 and 9.6, error at n=2048 8.9e-8, here 7.2e-8.
#include "direct_tile.h"

using namespace dastac;

namespace {

template <typename S, int WX, typename T = typename S::Type>
__global__ __launch_bounds__(64 * WX) __attribute__((amdgpu_waves_per_eu(4, 4)))
void trmm_direct_kernel(int n, int m, const T *__restrict__ U, const T *__restrict__ B, int64_t ldb, T *__restrict__ C, int64_t ldc, int ncb) {
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
    S::load(urow + k, o.u);
#pragma unroll
    for (int e = 0; e < S::kOwn; ++e)
#pragma unroll
      for (int c = 0; c < S::kCols; ++c) o.b[c][e] = bcol[c][(int64_t)(k + e) * ldb];
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
  auto step = [&](int w, auto... odd) __attribute__((always_inline)) {
    if (meets_edge(w)) mask(w, i, raw);
    S::multiply(raw, acc, [&] { load(w + WX < windows ? w + WX : w, raw); }, odd...);
  };
  if constexpr (S::kSets == 1) {
    for (int w = wave; w < windows; w += WX) step(w);
  } else {
    for (int w = wave; w < windows; w += 2 * WX) {
      step(w, 0);
      if (w + WX < windows) step(w + WX, 1);
    }
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
            for (int c = 0; c < S::kCols; ++c) raw.b[c][e] = k + e < begins(w) ? T(0) : raw.b[c][e];
        }
        S::plain(raw, acc);
      }
    }
  }
  add_up<WX, S::kRegs, typename S::Sum>(
      wave, lane, [&](int v) { return S::at(acc, v); },
      [&](int v, typename S::Sum sum) {
        const int r = i0 + S::row_of(v, lane), col = c0 + S::col_of(v, lane);
        if (r < n && col < m) C[(int64_t)r * ldc + col] = (T)sum;
      });
}

template <typename S, int WX, typename T = typename S::Type>
int launch(int64_t n, int64_t m, const T *U, const T *B, int64_t ldb, T *C, int64_t ldc, hipStream_t st) {
  const int64_t nrb = ceil_div(ceil_div(n, S::kRows), 8) * 8, ncb = ceil_div(m, 32);
  trmm_direct_kernel<S, WX><<<(unsigned)(nrb * ncb), 64 * WX, 0, st>>>((int)n, (int)m, U, B, ldb, C, ldc, (int)ncb);
  return launch_status();
}

// Sixteen wavefronts shorten a workgroup's chain of windows while few workgroups share a compute unit; eight waste less of it otherwise.  Up to 32 columns in
// single precision the length of the chain decides (us, four, eight and sixteen: n=64, m=8 2.8, 2.9, 3.5; n=200 3.6, 3.9, 4.3; n=400 4.5, 4.5, 4.9;
// n=1000 7.4, 6.8, 7.0; n=1400 9.2, 8.3, 8.2; n=2500 13.3 with eight, 10.9); else it is (us, eight and sixteen) fp32 n=3000, m=100, 376 workgroups 21.8, 17.5;
// m=200, 658 25.5, 27.7; n=1000, m=200, 224 8.1, 7.5; m=400, 416 9.8, 10.9; fp64 n=1500, m=64, 188 11.9, 12.3; m=100, 376 15.4, 12.7; m=200, 658 18.5, 21.3.
template <typename S, typename T = typename S::Type>
int run(int64_t n, int64_t m, const T *U, const T *B, int64_t ldb, T *C, int64_t ldc, void *stream) {
  const int64_t groups = ceil_div(n, S::kRows) * ceil_div(m, 32);
  if (S::kSets > 1 && n <= 200) return launch<S, 4>(n, m, U, B, ldb, C, ldc, (hipStream_t)stream);
  const bool wide = S::kSets > 1 ? n > 1200 : (S::kSplit ? n >= 500 && groups <= 512 && groups <= n / 4 + 100 : n >= 1000 && groups > 256 && groups <= 512);
  return wide ? launch<S, 16>(n, m, U, B, ldb, C, ldc, (hipStream_t)stream) : launch<S, 8>(n, m, U, B, ldb, C, ldc, (hipStream_t)stream);
}

}  // namespace

int dastac::trmm_direct(int64_t n, int64_t m, const float *U, const float *B, int64_t ldb, float *C, int64_t ldc, void *stream) {
  return m <= 32 ? run<NativeTile<float, float>>(n, m, U, B, ldb, C, ldc, stream) : run<SplitTile>(n, m, U, B, ldb, C, ldc, stream);
}
int dastac::trmm_direct(int64_t n, int64_t m, const double *U, const double *B, int64_t ldb, double *C, int64_t ldc, void *stream) {
  return run<NativeTile<double, double>>(n, m, U, B, ldb, C, ldc, stream);
}

// Band SpMV over diagonal-major packed storage:
//
//   y(i) := sum_{d=-w..w, 0<=i+d<n} D(d,i) * x(i+d)
//
// The rule is the strided-band structure of Section 6.4 with unit stride and 2w+1 summands
// (w=0 is Table 2's SpMV_D).  Each diagonal is one summand with its own densely packed n-slot
// buffer (Section 4, per-summand buffers), addressed by band_offset(d,i) = (d+w)*n + i, so lane l of
// a wavefront reads slot i0+l of every diagonal: 2w+1 perfectly contiguous streams, each element
// used exactly once.  They are read with non-temporal loads (measured: about 15 % faster than
// cached loads, which evict x from L2 for nothing), one row per lane (measured faster than two or
// four rows per lane at this shape).  x is the only reused operand; its 2w+1-wide window per lane
// overlaps the neighbours' windows almost completely and is served by the vector L1 cache
// (staging it in LDS behind a workgroup barrier measured slower, because the barrier delays the
// issue of the diagonal loads).
//
// Padding slots (column outside the matrix) are never used for their value: interior lanes cannot
// reach one, and the w lanes at either end select by the column predicate.
#include "common.h"

using namespace dastac;

namespace {

constexpr int kBlock = 256;
// Diagonals read at a time where their number is not known at compile time, and by the first and last rows of any: one at a time, the chain of 2w+1
// latencies was the time of small calls and the tail of large ones (us, before and now: fp32 w=3, n=4194304 37.8, 24.7; w=11, n=500000 21, 9.1; w=23, n=20000
// 23.6, 6.6; w=32, n=4194304 307, 179; w=16, whose interior rows are unrolled, n=4194304 94.5, 89; fp64 w=5, n=4194304 79, 72; w=20, n=20000 24.6, 7.1).
constexpr int kAhead = 8;

// acc + the products of N diagonals' slots (n apart) with consecutive elements of x, all reads requested first
template <int N, typename T>
__device__ inline T add_diagonals(T acc, const T *d, int64_t n, const T *x) {
  T a[N], b[N];
#pragma unroll
  for (int u = 0; u < N; ++u) a[u] = __builtin_nontemporal_load(d + (int64_t)u * n), b[u] = x[u];
#pragma unroll
  for (int u = 0; u < N; ++u) acc += a[u] * b[u];
  return acc;
}

// W >= 0: half-width known at compile time (fully unrolled); W < 0: run-time half-width `w`.
// With 33 streams per lane, four wavefronts per SIMD keep as much in flight as the memory system takes; the
// eight that the register count allows put more rows of more diagonals in flight at once and measured 2 % slower
// (n = 2^22: 97.6 -> 95.5 us; three: 95.0, five: 96.7, two: 102.9), so the widest instantiation is held to four.
template <int W, typename T>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(W == 16 ? 4 : 1, W == 16 ? 4 : 8)))
void band_kernel(int64_t n, int w, const T *__restrict__ D,
                                                      const T *__restrict__ x, T *__restrict__ y) {
  const int hw = W >= 0 ? W : w;
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const T *d = D + i;
  T acc = T(0);
  if (i >= hw && i + hw < n) {  // interior row: every column exists
    const T *xw = x + (i - hw);
    if (W >= 0) {
#pragma unroll
      for (int dd = 0; dd <= 2 * (W >= 0 ? W : 0); ++dd)
        acc += __builtin_nontemporal_load(d + (int64_t)dd * n) * xw[dd];
    } else {
      // eight diagonals' reads at a time (one by one, each would be waited for), then at once the one to seven that are left
      const int count = 2 * hw + 1;
      int dd = 0;
      for (; dd + kAhead <= count; dd += kAhead) acc = add_diagonals<kAhead>(acc, d + (int64_t)dd * n, n, xw + dd);
      d += (int64_t)dd * n, xw += dd;
      switch (count - dd) {
        case 1: acc = add_diagonals<1>(acc, d, n, xw); break;
        case 2: acc = add_diagonals<2>(acc, d, n, xw); break;
        case 3: acc = add_diagonals<3>(acc, d, n, xw); break;
        case 4: acc = add_diagonals<4>(acc, d, n, xw); break;
        case 5: acc = add_diagonals<5>(acc, d, n, xw); break;
        case 6: acc = add_diagonals<6>(acc, d, n, xw); break;
        case 7: acc = add_diagonals<7>(acc, d, n, xw); break;
      }
    }
  } else {  // one of the first or last w rows: skip the padding slots
    const int lo = i < hw ? (int)(hw - i) : 0, hi = n - 1 - i < hw ? hw + (int)(n - 1 - i) : 2 * hw;  // diagonals whose column exists
    for (int dd = lo; dd <= hi; dd += kAhead) {
      T a[kAhead], b[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int at = dd + u <= hi ? dd + u : hi;
        a[u] = d[(int64_t)at * n], b[u] = x[i + at - hw];
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) acc = dd + u <= hi ? acc + a[u] * b[u] : acc;
    }
  }
  __builtin_nontemporal_store(acc, y + i);
}

// Element type T: float, or double (the paper's element type; same kernel, eight bytes per slot).
template <typename T>
int run(int64_t n, int64_t w, const T *D, const T *x, T *y, void *stream) {
  if (n < 0 || w < 0) return DASTAC_EINVAL;
  if (w > (1 << 20)) return DASTAC_EOVERFLOW;
  if (n > ((int64_t)1 << 40) / (2 * w + 1)) return DASTAC_EOVERFLOW;
  if (n == 0) return DASTAC_OK;
  if (!D || !x || !y) return DASTAC_ENULL;
  const int64_t sz = (int64_t)sizeof(T);
  if (overlaps(y, n * sz, D, (2 * w + 1) * n * sz) || overlaps(y, n * sz, x, n * sz)) return DASTAC_EALIAS;
  hipStream_t st = (hipStream_t)stream;
  const unsigned blocks = (unsigned)ceil_div(n, kBlock);
  switch (w) {
    case 16: band_kernel<16, T><<<blocks, kBlock, 0, st>>>(n, 16, D, x, y); break;
    case 8: band_kernel<8, T><<<blocks, kBlock, 0, st>>>(n, 8, D, x, y); break;
    case 4: band_kernel<4, T><<<blocks, kBlock, 0, st>>>(n, 4, D, x, y); break;
    case 2: band_kernel<2, T><<<blocks, kBlock, 0, st>>>(n, 2, D, x, y); break;
    case 1: band_kernel<1, T><<<blocks, kBlock, 0, st>>>(n, 1, D, x, y); break;
    case 0: band_kernel<0, T><<<blocks, kBlock, 0, st>>>(n, 0, D, x, y); break;
    default: band_kernel<-1, T><<<blocks, kBlock, 0, st>>>(n, (int)w, D, x, y);
  }
  return launch_status();
}

}  // namespace

extern "C" int dastac_band_spmv_f32(int64_t n, int64_t w, const float *D, const float *x, float *y, void *stream) {
  return run<float>(n, w, D, x, y, stream);
}

extern "C" int dastac_band_spmv_f64(int64_t n, int64_t w, const double *D, const double *x, double *y,
                                    void *stream) {
  return run<double>(n, w, D, x, y, stream);
}

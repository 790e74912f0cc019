// The launch in front of MTTKRP's kernels that add into M.
#pragma once
#include "common.h"

namespace dastac {

constexpr int kMinOrder = 3;  // slices of order 1 and 2: the last four elements of the packed buffer, where a 16-byte load has no room

// Clears M and computes those slices directly from the rule: sums of one and of three terms, which the split products of single precision would bring less close
// (2-norm of the slice's error, split and here: order 1 3.9e-8, 3.1e-8; order 2 3.74e-8, 3.65e-8; order 3 4.0e-8, with fp32 products 4.4e-8).
template <typename T, typename Index>
__global__ __launch_bounds__(256) void mttkrp_clear_kernel(Index n, Index R, const T *__restrict__ end_of_A, const T *__restrict__ Bm, int64_t ldb,
                                                           const T *__restrict__ Cm, int64_t ldc, T *__restrict__ M, int64_t ldm) {
  // one output element per thread, in turns beyond 2^31 of them
  for (Index e = (Index)blockIdx.x * 256 + threadIdx.x; e < n * R; e += (Index)gridDim.x * 256) {
    const Index i = e / R, r = e - i * R;
    T s = T(0);
    if (n - i < kMinOrder) {  // (all reads at once)
      const T *b = Bm + ((int64_t)i * ldb + r), *c = Cm + ((int64_t)i * ldc + r);
      // (added to zero: a product that is -0 leaves +0, as in every other sum)
      if (n - i == 1) {
        s += end_of_A[-1] * b[0] * c[0];
      } else {
        s += end_of_A[-4] * b[0] * c[0];
        s += end_of_A[-3] * b[0] * c[ldc];
        s += end_of_A[-2] * b[ldb] * c[ldc];
      }
    }
    M[(int64_t)i * ldm + r] = s;
  }
}
template <typename T>
inline int mttkrp_clear(int64_t n, int64_t R, const T *A, const T *B, int64_t ldb, const T *C, int64_t ldc, T *M, int64_t ldm, hipStream_t st) {
  const int64_t cb = ceil_div(n * R, 256);
  if (n * R < ((int64_t)1 << 24))  // (a division of 64 bits is 0.3 us of a launch)
    mttkrp_clear_kernel<T, unsigned><<<(unsigned)cb, 256, 0, st>>>((unsigned)n, (unsigned)R, A + tet(n), B, ldb, C, ldc, M, ldm);
  else
    mttkrp_clear_kernel<T, int64_t><<<(unsigned)(cb < (1 << 23) ? cb : 1 << 23), 256, 0, st>>>(n, R, A + tet(n), B, ldb, C, ldc, M, ldm);
  return launch_status();
}

}  // namespace dastac

// TTM over a packed upper half cube, the paper's running example (Fig. 3):
//
//   A(i,j,k) := B(i,j,l) * C(k,l),   i<=j, 0<=l<Q, 0<=k<K
//
// B stores only the pairs i<=j, each with its Q values of l back to back, at the position given
// by the printed index polynomial P_B(i,j,l) = tri(n,i,j)*Q + l (Section 3).  The output inherits
// the structure and is packed by the same rule with k in place of l (Section 3, "Data layout
// compression": input and output compression).  Pair number p = tri(n,i,j) is therefore row p of
// both buffers, and the whole contraction is ONE dense product over the packed rows,
//
//   Ap[p, k] = sum_l Bp[p, l] * C[k, l],      p = 0 .. Tri(n)-1
//
// with no structural zero left to skip and no index arithmetic beyond the row number: that is
// the point of the layout.  It runs on the matrix cores, in single and in double precision.
//
// Single precision runs as a three-part split on the bf16 matrix cores (ttm_split_kernel below).  This kernel serves double
// precision, and single precision where split_serves() declines; few rows, and in double precision few columns, go to ttm_direct.hip first (direct_serves).
//
// Tiling.  A workgroup (8 wavefronts, 2 x 4) owns 64 packed rows x 128 values of k and sweeps l in
// steps of kKT = 32 (fp32) or 16 (fp64); the 64 x kKT tile of Bp and the 128 x kKT tile of C are staged
// in LDS, double-buffered against the global loads of the next step.  Both tiles keep l contiguous, so
// in fp32 -- with lane half h taking the four consecutive l values 8t+4h..8t+4h+3 of every group of
// eight, as in the TRMM kernel -- both operands of v_mfma_f32_32x32x2_f32 are single 16-byte LDS reads
// (the per-type matrix-core pieces are those of mfma_tile.h).  Workgroups
// that share a row block (different blocks of k) get ids that are equal modulo 8, i.e. the same
// XCD, so the rows of Bp they both read come from HBM once.  About two workgroups per compute unit
// are launched; each walks a strided set of row blocks with one uninterrupted pipeline, so the
// first loads of a row block are in flight while the previous block's last step is multiplied.
#include "split3.h"
#include "mfma_tile.h"

using namespace dastac;

namespace {

// tags that pick a step's flavour at compile time
struct Whole {
  static constexpr bool value = true;
};
struct Any {
  static constexpr bool value = false;
};

template <typename T>
struct Stage {
  typename Core<T>::vec a;     // Bp: row sr of the tile, one 16-byte piece of l values
  typename Core<T>::vec c[2];  // C: rows sr and sr+64 of the tile, one 16-byte piece of l values each
};

template <typename T>
__global__ __launch_bounds__(kTileThreads) void ttm_mfma_kernel(int64_t rows, int64_t Q, int64_t K,
                                                                const T *__restrict__ Bp, const T *__restrict__ C,
                                                                int64_t ldc, T *__restrict__ Ap, int lanes, int ncb) {
  typedef Core<T> Kc;
  typedef typename Kc::vec vec;
  typedef typename Kc::uvec uvec;
  constexpr int kBM = kTileM, kBN = kTileN, kKT = Kc::kKT, kV = Kc::kVec, kP = Kc::kRowPitch;
  __shared__ __attribute__((aligned(16))) T As[2][kBM * kP];
  __shared__ __attribute__((aligned(16))) T Cs[2][kBN * kP];

  // workgroup id -> (first row block, block of k); ids equal mod 8 share an XCD.  A workgroup
  // then walks every (8*lanes)-th row block, keeping its pipeline full across blocks.
  const int L = blockIdx.x;
  const int xcd = L & 7, slot = L >> 3;
  const int cb = slot % ncb;
  const int64_t rstride = (int64_t)kBM * 8 * lanes;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 2, wc = wave & 3;  // 2x4 wavefronts: 32 rows x 32 values of k each

  // staging role: tile row tid/8 (and +64 for C), l offset kV*(tid%8)
  const int sr = tid >> 3, sl = (tid & 7) * kV;
  const int64_t c0 = (int64_t)cb * kBN;
  const bool full_c = c0 + kBN <= K;
  const int nk = (int)ceil_div(Q, kKT);

  const T *cp0 = C + (c0 + sr < K ? c0 + sr : K - 1) * ldc;
  const T *cp1 = C + (c0 + sr + 64 < K ? c0 + sr + 64 : K - 1) * ldc;

  struct Cur {  // wave-uniform cursor over the steps of this workgroup: row block, step along l
    int64_t r0;
    int kt;
    bool valid;
  };
  auto next = [&](Cur c) -> Cur {
    if (!c.valid) return c;
    if (c.kt + 1 < nk) {
      c.kt += 1;
    } else {
      c.kt = 0;
      c.r0 += rstride;
      c.valid = c.r0 < rows;
    }
    return c;
  };

  auto load_stage = [&](const Cur &cu, Stage<T> &s) {
    const int64_t l0 = (int64_t)cu.kt * kKT + sl;
    const T *ap = Bp + (cu.r0 + sr < rows ? cu.r0 + sr : rows - 1) * Q;
    if (full_c && cu.r0 + kBM <= rows && (int64_t)cu.kt * kKT + kKT <= Q) {
      s.a = *reinterpret_cast<const uvec *>(ap + l0);
      s.c[0] = *reinterpret_cast<const uvec *>(cp0 + l0);
      s.c[1] = *reinterpret_cast<const uvec *>(cp1 + l0);
    } else {  // ragged edge: zeros outside the operands
#pragma unroll
      for (int e = 0; e < kV; ++e) {
        const bool lok = l0 + e < Q;
        s.a[e] = (lok && cu.r0 + sr < rows) ? ap[l0 + e] : T(0);
        s.c[0][e] = (lok && c0 + sr < K) ? cp0[l0 + e] : T(0);
        s.c[1][e] = (lok && c0 + sr + 64 < K) ? cp1[l0 + e] : T(0);
      }
    }
  };
  auto store_stage = [&](int buf, const Stage<T> &s) {
    *reinterpret_cast<vec *>(&As[buf][sr * kP + sl]) = s.a;
    *reinterpret_cast<vec *>(&Cs[buf][sr * kP + sl]) = s.c[0];
    *reinterpret_cast<vec *>(&Cs[buf][(sr + 64) * kP + sl]) = s.c[1];
  };

  typename Kc::Acc acc;
  Kc::clear(acc);
  auto read_ops = [&](int buf, int t, typename Kc::Ops &o) {
    Kc::read_a(&As[buf][wr * 32 * kP], lane, t, o);
    Kc::read_b_rows(&Cs[buf][wc * 32 * kP], lane, t, o);
  };

  Cur cc{(int64_t)kBM * (xcd + 8 * (slot / ncb)), 0, true};  // the step being multiplied
  cc.valid = cc.r0 < rows;
  if (!cc.valid) return;
  Cur cl = cc;  // the step being loaded: one ahead
  Stage<T> st;
  typename Kc::Ops oa, ob;
  load_stage(cl, st);
  store_stage(0, st);
  __syncthreads();
  read_ops(0, 0, oa);

  // One step on LDS buffer `buf` (a literal at every call site).  The global loads of the next
  // step -- of the next row block, at a block's last step -- are in flight throughout; its LDS
  // stores and the workgroup barrier sit before the last group's matrix instructions, whose
  // operands are already in registers.  (The schedule of mfma_tile.h's sweep, run as ONE pipeline over
  // all the workgroup's row blocks.)
  // WHOLE: the step being loaded exists and lies in a whole row block of a whole column block, with Q a
  // multiple of the step (so does the step being multiplied, which comes before it): loads and the stores of
  // a finished tile then need no test and no clamped row, and the loop made of such steps holds none.
  const int64_t aoff = (int64_t)sr * Q + sl;
  auto step = [&](int buf, auto whole_tag) {
    constexpr bool WHOLE = decltype(whole_tag)::value;
    cl = next(cl);
    const bool more = WHOLE || cl.valid;
    if (WHOLE) {
      const int64_t l0 = (int64_t)cl.kt * kKT;
      st.a = *reinterpret_cast<const uvec *>(Bp + (cl.r0 * Q + l0) + aoff);
      st.c[0] = *reinterpret_cast<const uvec *>(cp0 + l0 + sl);
      st.c[1] = *reinterpret_cast<const uvec *>(cp1 + l0 + sl);
    } else if (more) {
      load_stage(cl, st);
    }
    // (Scheduling barriers keep the written order: left alone, the compiler merges the two operand register
    // sets and issues a group's LDS reads after the previous group's matrix instructions instead of before
    // them.  With two workgroups per CU and no shares, as here, the written order is 2.5 % faster.)
    read_ops(buf, 1, ob);
    __builtin_amdgcn_sched_barrier(0);
    Kc::mma(oa, acc);
    __builtin_amdgcn_sched_barrier(0);
    read_ops(buf, 2, oa);
    __builtin_amdgcn_sched_barrier(0);
    Kc::mma(ob, acc);
    __builtin_amdgcn_sched_barrier(0);
    read_ops(buf, 3, ob);
    __builtin_amdgcn_sched_barrier(0);
    Kc::mma(oa, acc);
    __builtin_amdgcn_sched_barrier(0);
    if (more) store_stage(buf ^ 1, st);
    __syncthreads();
    if (more) read_ops(buf ^ 1, 0, oa);
    __builtin_amdgcn_sched_barrier(0);
    Kc::mma(ob, acc);
    __builtin_amdgcn_sched_barrier(0);
    if (cc.kt == nk - 1) {
      Kc::for_each(acc, lane, [&](int r, int c, T v) {
        const int64_t row = cc.r0 + wr * 32 + r, col = c0 + wc * 32 + c;
        if (WHOLE || (row < rows && col < K)) Ap[row * K + col] = v;
      });
      Kc::clear(acc);
    }
    cc = next(cc);
  };
  // whole steps two at a time (all whole row blocks come before the ragged one), then the rest
  if (full_c && Q % kKT == 0) {
    auto whole = [&](const Cur &c) { return c.valid && c.r0 + kBM <= rows; };
    for (;;) {
      const Cur n1 = next(cl);
      if (!whole(n1) || !whole(next(n1))) break;
      step(0, Whole{});
      step(1, Whole{});
    }
  }
  for (;;) {
    step(0, Any{});
    if (!cc.valid) break;
    step(1, Any{});
    if (!cc.valid) break;
  }
}

// ---- single precision by the three-part split (split3.h) --------------------------------------------------------
// The same product on the bf16 matrix cores: a workgroup of WR x WC wavefronts with WM x WN sub-tiles of 32 x 32 each walks
// every (8*lanes)-th row block of its column block with one uninterrupted pipeline over (row block, step of 32 l).  Both
// operands keep l contiguous: a thread stages pieces of four l of a row, split on the way into LDS (split3.h).  The
// requests run two steps ahead of their use and the conversion one; the last twelve matrix instructions of a step stand
// behind the barrier, while the first operands of the next step come back (256 x 128 tiles: eight, below).  A ragged last step reads its pieces pulled
// back into the row and shifts them into place; rows past the last repeat it.
// One 32 x 32 sub-tile in fp32, operands straight from memory: what a sub-tile with a non-finite element is evaluated by
// again, so that Inf and NaN propagate as IEEE arithmetic has it.  A lane's four l are one load, and two groups of eight l are
// requested at once (us, n=512, Q=K=256, NaN in C: 226; one value and one group at a time 404; marked and run by the whole
// workgroup through LDS when its walk is over 294, but the barrier before that costs small calls 0.5 of 5; the call without 122).
__device__ __attribute__((noinline)) Core<float>::Acc plain_sub_tile(int64_t rows, int Q, int K, const float *Bp, const float *C, int64_t ldc,
                                                                     int64_t row0, int col0, int lane) {
  typedef Core<float> Kc;
  constexpr int kAtOnce = 2;
  Kc::Acc acc;
  Kc::clear(acc);
  const float *a = Bp + (row0 + (lane & 31) < rows ? row0 + (lane & 31) : rows - 1) * Q;
  const float *c = C + (int64_t)(col0 + (lane & 31) < K ? col0 + (lane & 31) : K - 1) * ldc;
  int l0 = 0;
#pragma unroll 1
  for (; l0 + kAtOnce * Kc::kGroup <= Q; l0 += kAtOnce * Kc::kGroup) {
    f4a x[kAtOnce], y[kAtOnce];
#pragma unroll
    for (int g = 0; g < kAtOnce; ++g) {
      const int l = l0 + g * Kc::kGroup + Kc::op_index(lane, 0);
      x[g] = *reinterpret_cast<const f4u *>(a + l), y[g] = *reinterpret_cast<const f4u *>(c + l);
    }
#pragma unroll
    for (int g = 0; g < kAtOnce; ++g) {
      Kc::Ops o;
#pragma unroll
      for (int q = 0; q < Kc::kOps; ++q) o.a[q] = x[g][q], o.b[q] = y[g][q];
      Kc::mma(o, acc);
    }
  }
#pragma unroll 1
  for (; l0 < Q; l0 += Kc::kGroup) {
    Kc::Ops o;
#pragma unroll
    for (int q = 0; q < Kc::kOps; ++q) {
      const int l = l0 + Kc::op_index(lane, q), lc = l < Q ? l : Q - 1;
      const float x = a[lc], y = c[lc];
      o.a[q] = l < Q ? x : 0.0f;
      o.b[q] = l < Q ? y : 0.0f;
    }
    Kc::mma(o, acc);
  }
  return acc;
}

template <typename G>
__global__ __launch_bounds__(G::kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void ttm_split_kernel(int64_t rows, int Q, int K, const float *__restrict__ Bp, const float *__restrict__ C, int64_t ldc,
                      float *__restrict__ Ap, int nrb, int lanes, int ncb) {
  constexpr int kBM = G::kBM, kBN = G::kBN, kKT = 32, kTh = G::kThreads, WM = G::WM, WN = G::WN;
  constexpr int kPass = kTh / 8, kPA = kBM / kPass, kPC = kBN / kPass;  // rows staged per pass; pieces per thread
  static_assert(kBM % kPass == 0 && kBN % kPass == 0, "whole passes stage a step");
  typedef unsigned short Parts16[3][(kBM + kBN) * kKT];
  __shared__ __attribute__((aligned(16))) Parts16 parts[2];

  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int cb = slot % ncb, stride = 8 * lanes;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform32(tid >> 6);
  const int wr = wave / G::WC, wc = wave % G::WC;
  const int sr = tid >> 3, sl = (tid & 7) * 4;
  const int c0 = cb * kBN, nk = (Q + kKT - 1) / kKT;

  struct Cur {  // wave-uniform: row block and step
    int rb, kt;
  };
  auto next = [&](Cur c) {  // past the last step: the last step again
    Cur d{c.kt + 1 < nk ? c.rb : c.rb + stride, c.kt + 1 < nk ? c.kt + 1 : 0};
    return d.rb < nrb ? d : c;
  };
  Cur cc{xcd + 8 * (slot / ncb), 0};  // the step being multiplied
  if (cc.rb >= nrb) return;
  int left = ((nrb - 1 - cc.rb) / stride + 1) * nk;  // steps of this workgroup

  const float *cp[kPC];
#pragma unroll
  for (int q = 0; q < kPC; ++q) cp[q] = C + (int64_t)(c0 + sr + q * kPass < K ? c0 + sr + q * kPass : K - 1) * ldc;
  unsigned aoff[kPA];  // the thread's rows within a row block, in elements
#pragma unroll
  for (int p = 0; p < kPA; ++p) aoff[p] = (unsigned)(sr + p * kPass) * (unsigned)Q;

  struct Stage {
    f4a a[kPA], c[kPC];
  };
  auto load = [&](const Cur &cu, Stage &s) __attribute__((always_inline)) {
    const int64_t r0 = (int64_t)cu.rb * kBM;
    const char *base = reinterpret_cast<const char *>(Bp + r0 * Q);
    const unsigned lim = rows - r0 > kBM ? 0xffffffffu : (unsigned)(rows - 1 - r0) * (unsigned)Q;  // the last row's offset
    const int l = cu.kt * kKT + sl < Q - 4 ? cu.kt * kKT + sl : Q - 4;
#pragma unroll
    for (int p = 0; p < kPA; ++p) s.a[p] = *reinterpret_cast<const f4u *>(base + 4u * ((aoff[p] < lim ? aoff[p] : lim) + (unsigned)l));
#pragma unroll
    for (int q = 0; q < kPC; ++q) s.c[q] = *reinterpret_cast<const f4u *>(cp[q] + l);
  };
  auto put = [&](int buf, int row, f4a v) __attribute__((always_inline)) {
    u2v h, md, lw;
    unsigned x, y, z;
    split3(v[0], v[1], x, y, z);
    h[0] = x, md[0] = y, lw[0] = z;
    split3(v[2], v[3], x, y, z);
    h[1] = x, md[1] = y, lw[1] = z;
    const int at = part_place(row, sl >> 3) + (sl & 4);
    *reinterpret_cast<u2v *>(&parts[buf][0][at]) = h;
    *reinterpret_cast<u2v *>(&parts[buf][1][at]) = md;
    *reinterpret_cast<u2v *>(&parts[buf][2][at]) = lw;
  };
  auto convert = [&](int buf, const Cur &cu, Stage &s) __attribute__((always_inline)) {
    const int past = cu.kt * kKT + sl - (Q - 4);  // by how much the pieces were pulled back
    if ((cu.kt + 1) * kKT > Q) {
      auto shift = [&](f4a v) {
        f4a w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          w[e] = past <= 0 ? v[e] : 0.0f;
#pragma unroll
          for (int x = 1; e + x < 4; ++x) w[e] = past == x ? v[e + x] : w[e];
        }
        return w;
      };
#pragma unroll
      for (int p = 0; p < kPA; ++p) s.a[p] = shift(s.a[p]);
#pragma unroll
      for (int q = 0; q < kPC; ++q) s.c[q] = shift(s.c[q]);
    }
#pragma unroll
    for (int p = 0; p < kPA; ++p) put(buf, sr + p * kPass, s.a[p]);
#pragma unroll
    for (int q = 0; q < kPC; ++q) put(buf, kBM + sr + q * kPass, s.c[q]);
  };
  struct Plane {
    u4v a[WM], b[WN];
  };
  auto read = [&](int buf, int t, int part, Plane &o) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WM; ++i)
      o.a[i] = *reinterpret_cast<const u4v *>(&parts[buf][part][part_place((wr * WM + i) * 32 + (lane & 31), 2 * t + (lane >> 5))]);
#pragma unroll
    for (int j = 0; j < WN; ++j)
      o.b[j] = *reinterpret_cast<const u4v *>(&parts[buf][part][part_place(kBM + (wc * WN + j) * 32 + (lane & 31), 2 * t + (lane >> 5))]);
  };
  Core<float>::Acc hi[WM][WN], lo[WM][WN];  // the five smaller products have an accumulator of their own
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) Core<float>::clear(hi[i][j]), Core<float>::clear(lo[i][j]);
  };
  auto mma = [&](const Plane &a, const Plane &b, bool largest) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        f16v &acc = largest ? hi[i][j].v : lo[i][j].v;
        acc = mma_bf16(a.a[i], b.b[j], acc);
      }
  };
  auto flush = [&](int rb) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const int64_t row0 = (int64_t)rb * kBM + (wr * WM + i) * 32;
        const int col0 = c0 + (wc * WN + j) * 32;
        hi[i][j].v += lo[i][j].v;
        const bool bad = Core<float>::non_finite(hi[i][j], lane, K - col0);
        hi[i][j].v *= kSplitDown;
        if (__any(bad)) hi[i][j] = plain_sub_tile(rows, Q, K, Bp, C, ldc, row0, col0, lane);
        float *out = Ap + row0 * K + col0;
        const int64_t rleft = rows - row0;
        const int cleft = K - col0;
        if (rleft >= 32) {  // scalar row addresses, one test
          if ((lane & 31) < cleft) Core<float>::for_each_at(hi[i][j], lane, out, K, [](auto p, float v) { *p = v; });
        } else {
          int l = lane;
          asm volatile("" : "+v"(l));  // (or the places of all elements are kept in registers through the loop: 244 of them where it takes 180)
          Core<float>::for_each(hi[i][j], l, [&](int r, int c, float v) {
            if (r < rleft && c < cleft) out[(int64_t)r * K + c] = v;
          });
        }
      }
    clear();
  };
  if constexpr (WM == 1) {
    Stage s0, s1;
    Plane h0, h1, md, lw;
    clear();
    Cur c1 = next(cc), c2 = next(c1);
    load(cc, s0);
    load(c1, s1);
    convert(0, cc, s0);
    __syncthreads();
    read(0, 0, 0, h0);
    auto step = [&](int buf, Stage &freed, Stage &coming) __attribute__((always_inline)) {
      load(c2, freed);
      read(buf, 0, 1, md);
      read(buf, 0, 2, lw);
      convert(buf ^ 1, c1, coming);
      mma(h0, h0, true);
      mma(h0, md, false);
      mma(md, h0, false);
      mma(md, md, false);
      read(buf, 1, 0, h1);
      mma(h0, lw, false);
      mma(lw, h0, false);
      read(buf, 1, 1, md);
      read(buf, 1, 2, lw);
      mma(h1, h1, true);
      mma(h1, md, false);
      mma(md, h1, false);
      __syncthreads();
      read(buf ^ 1, 0, 0, h0);
      mma(md, md, false);
      mma(h1, lw, false);
      mma(lw, h1, false);
      __builtin_amdgcn_sched_barrier(0);
      if (cc.kt == nk - 1) flush(cc.rb);
      cc = c1;
      c1 = c2;
      c2 = next(c2);
    };
    for (; left > 1; left -= 2) {
      step(0, s0, s1);
      step(1, s1, s0);
    }
    if (left > 0) step(0, s0, s1);
  } else {
    // Twice the matrix instructions a step and a third less to read from LDS for each, but 128 registers of sums: one set of loads on its way, converted before
    // the barrier and asked for again behind it, and three planes of operands at a time.
    Stage st;
    Plane h, m, l, g;
    clear();
    Cur c1 = next(cc), c2 = next(c1);
    load(cc, st);
    convert(0, cc, st);
    load(c1, st);
    __syncthreads();
    read(0, 0, 0, h);
    auto step = [&](int buf) __attribute__((always_inline)) {
      read(buf, 0, 1, m);
      mma(h, h, true);
      read(buf, 0, 2, l);
      mma(h, m, false);
      mma(m, h, false);
      mma(m, m, false);
      read(buf, 1, 0, g);
      mma(h, l, false);
      mma(l, h, false);
      read(buf, 1, 1, m);
      mma(g, g, true);
      read(buf, 1, 2, l);
      convert(buf ^ 1, c1, st);
      load(c2, st);
      mma(g, m, false);
      mma(m, g, false);
      mma(m, m, false);
      __syncthreads();
      read(buf ^ 1, 0, 0, h);
      mma(g, l, false);
      mma(l, g, false);
      __builtin_amdgcn_sched_barrier(0);
      if (cc.kt == nk - 1) flush(cc.rb);
      cc = c1;
      c1 = c2;
      c2 = next(c2);
    };
    for (; left > 1; left -= 2) {
      step(0);
      step(1);
    }
    if (left > 0) step(0);
  }
}

// ---- compression / decompression of the upper half cube ---------------------------------------
// One workgroup per 256-element piece of one (i,j) row of the dense n x n x Q tensor.
constexpr int kCopy = 256;

template <bool PACK, typename T>
__global__ __launch_bounds__(kCopy) void uhc_copy_kernel(int64_t n, int64_t Q, const T *__restrict__ src,
                                                         T *__restrict__ dst, int64_t pieces,
                                                         int64_t nblocks) {
  for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
    const int64_t ij = b / pieces, l = (b - ij * pieces) * kCopy + threadIdx.x;
    const int64_t i = ij / n, j = ij - i * n;
    if (l >= Q) continue;
    if (PACK) {
      if (j >= i) dst[tri_offset(n, i, j) * Q + l] = src[ij * Q + l];
    } else {
      dst[ij * Q + l] = (j >= i) ? src[tri_offset(n, i, j) * Q + l] : T(0);
    }
  }
}

inline bool uhc_ok(int64_t n, int64_t Q) {
  return n >= 0 && Q >= 1 && n <= (1 << 20) && Q <= (1 << 24) && (n == 0 || tri(n) <= ((int64_t)1 << 40) / Q);
}

// pack (dense -> packed) or unpack (packed -> dense) of the upper half cube, float or double
template <bool PACK, typename T>
int uhc_copy(int64_t n, int64_t Q, const T *src, T *dst, void *stream) {
  if (n < 0 || Q < 1) return DASTAC_EINVAL;
  if (!uhc_ok(n, Q) || n * n > ((int64_t)1 << 40) / Q) return DASTAC_EOVERFLOW;
  if (n == 0) return DASTAC_OK;
  if (!src || !dst) return DASTAC_ENULL;
  const int64_t sz = (int64_t)sizeof(T), nd = n * n * Q * sz, np = tri(n) * Q * sz;
  if (overlaps(dst, PACK ? np : nd, src, PACK ? nd : np)) return DASTAC_EALIAS;
  const int64_t pieces = ceil_div(Q, kCopy), nblocks = n * n * pieces;
  const unsigned grid = (unsigned)(nblocks < (1 << 20) ? nblocks : (1 << 20));
  uhc_copy_kernel<PACK, T><<<grid, kCopy, 0, (hipStream_t)stream>>>(n, Q, src, dst, pieces, nblocks);
  return launch_status();
}

// Few rows run straight from memory with l cut among wavefronts (ttm_direct.hip).  A workgroup of the kernels here takes a time that grows with Q, the
// direct tiles together one that grows with their number times Q, so the line is a number of direct tiles (us, here and there, fp32: 1068 tiles
// n=130, Q=250, K=100 14.4, 12.5; 1280 n=90, Q=400, K=300 20.4, 17.0; 1144 n=270, K=18, Q=228 13.9, 10.4; 1146 n=191, K=34, Q=410 19.0, 17.2; 1258 n=200, K=33,
// Q=100 8.8, 6.8; Q=256 12.9, 13.7; 2122 n=260, Q=K=60 9.5, 9.0; 2550 n=180,
// Q=200, K=150 15.8, 20.6).  Q and K above 2^20 stay here.
//
// In double precision the tiles here are 128 columns wide, so 32 columns or fewer go there with any number of rows (n=500, Q=434, K=16 310, 149; n=700, Q=32,
// K=32 50, 47).  With two column blocks the line depends on the remainder of Q by 16, for which these kernels take a whole step and the direct one
// moves a window back (us: n=150, 1416 tiles, K=33, Q=32 5.9, 6.7; Q=40 7.5, 6.0; n=200, 2514 tiles, K=64, Q=64 14.3, 15.2; Q=128 24.4, 22.9; Q=100 21.7, 13.9; n=240, 3616 tiles, K=33,
// Q=128 24.1, 30.0; Q=100 21.4, 18.1; n=300, K=48, 5644 tiles, Q=48 17.6, 23.6; Q=24 12.7, 13.0; Q=100 34, 25; Q=1000 0.77 of the time; n=257, 4146 tiles, K=46,
// Q=24 12.4, 10.8; n=700, Q=32 51, 86; Q=100 152, 120; Q=434, K=33 589, 694).
template <typename T>
bool direct_serves(int64_t rows, int64_t Q, int64_t K) {
  const int64_t tiles = ceil_div(rows, sizeof(T) == 4 ? 32 : 16) * ceil_div(K, 32);
  if (Q < 16 || Q > (1 << 20) || K > (1 << 20) || rows > (1 << 24)) return false;
  if (sizeof(T) == 4) return tiles <= 1280;
  if (K <= 32) return true;
  if (Q % 16 == 0) return tiles <= (Q < 128 ? 1280 : K <= 64 ? 2560 : 2048);
  if (K <= 48 && Q >= 64 && Q <= (tiles <= 6000 ? 1024 : 256)) return true;
  return tiles <= (K <= 48 ? 4700 : K <= 64 ? 4096 : 2048);
}

// The split's offsets within a row block are 32 bits and a piece needs four l; beyond that the fp32 matrix cores take over, and
// where one step is all there is and the tiles do not fill the chip: the split's conversion then only adds to the latency
// (us, split and fp32 cores: n=60, Q=20, K=512 6.0, 5.1; n=150, Q=20, K=100 6.1, 5.1; past one layer, n=150, Q=20, K=300, 9.7, 10.7).
// Two steps in one layer are up to 1 us slower split as well (n=30, Q=33, K=512 6.7, 5.7; Q=48, K=100 6.6, 6.8; Q=56, K=16 5.1, 5.8), but
// with half the error or less; they stay.
inline bool split_serves(int64_t rows, int64_t Q, int64_t K, const float *) {
  if (Q <= 32 && ceil_div(rows, kTileM) * ceil_div(K, kTileN) <= 256) return false;
  return Q >= 4 && Q <= (1 << 20) && K <= (1 << 20);
}
inline bool split_serves(int64_t, int64_t, int64_t, const double *) { return false; }

// Workgroups that walk one column block on each XCD, of `slots` that the chip holds at once: a walker that has to wait for another to end doubles the time.
inline int64_t walkers(int64_t slots, int64_t ncb) { return slots >= 8 * ncb ? slots / (8 * ncb) : 1; }

template <typename G>
int launch_split(int64_t rows, int64_t Q, int64_t K, const float *Bp, const float *C, int64_t ldc, float *Ap, int64_t cus, hipStream_t st) {
  const int64_t nrb = ceil_div(rows, G::kBM), ncb = ceil_div(K, G::kBN);
  if (nrb > 0x7fffffff || (nrb + 8) * ceil_div(Q, 32) > 0x7fffffff) return DASTAC_EOVERFLOW;
  int64_t lanes = walkers(G::kThreads == 512 ? cus : 2 * cus, ncb);  // one workgroup of eight wavefronts to a compute unit, or two of four
  if (lanes > ceil_div(nrb, 8)) lanes = ceil_div(nrb, 8);
  ttm_split_kernel<G><<<(unsigned)(8 * lanes * ncb), G::kThreads, 0, st>>>(rows, (int)Q, (int)K, Bp, C, ldc, Ap, (int)nrb, (int)lanes, (int)ncb);
  return launch_status();
}
// Tiles by columns: 128 x 32 and 128 x 64 where C has no more (us, before: n=300, Q=512, K=16 25, 83; n=500, Q=K=64 17, 33; n=512,
// Q=100, K=40 28, 58), else eight wavefronts on 128 x 128 or, a third less LDS traffic a product and half the barriers, on 256 x 128.  A workgroup to a compute
// unit takes whole tiles, so what counts is the rounds of tiles, and the rows past whole rounds may run straight from memory in a launch of their own.
//
// The estimate, us: 4.1, and for a round 1.46 + 0.0437 Q of 128 x 128, 3.28 + 0.0803 Q of 256 x 128 (Q in whole steps of 32), a last round that is a part f of one counted
// as 0.67 + 0.33 f; for t direct tiles in a second launch 3.1 + (9e-4 + 2.6e-5 Q) t.  Fitted to the four ways at 740 sizes (n 60 to 900, Q 10 to 900, K 65 to 900; 6 % off
// in the root mean square); its choice takes 1.004 times the best way's time, 0.92 of 128 x 128 in one launch as it was before, 1.08 at worst (n=276, Q=371, K=200 54.5, 58.4).  us, 128 x 128, with
// the rest apart, 256 x 128, with the rest apart: n=512, Q=371, K=256 175 165 179 157; n=512, Q=371, K=470 339 332 324 300; n=280, Q=256, K=128 27.8 28.8 25.1 25.0; n=276, Q=64, K=200
// 15.8 19.2 18.6 19.5; n=270, Q=64, K=256 15.9 18.5 18.9 19.3; n=204, Q=323, K=230 35.1 38.6 31.6 31.4.
//
// One and two steps of l and more output than the memory-side cache holds are bound by writing it, and 256 x 128 is faster there (why has not been taken apart; 128 x 128, 256 x 128):
// 263 MB n=512, Q=20, K=500 69, 58; 306 MB n=600, Q=10, K=424 79, 68; 493 MB n=705, Q=64, K=495 166, 155; below, 252 MB n=512, Q=24, K=480 50, 50.  With one step
// and four column blocks it turns from 430 MB on: n=777, Q=20, K=414 120, 148; n=768, Q=16, K=467 133, 158.
// What bounds many steps is power: 1.09 PFLOP/s of bf16 at n=512, Q=K=512, 0.81 of the library's.
struct Rounds {
  double us;
  int64_t rows;  // of the launch of tiles; the others run straight from memory
};
inline Rounds ttm_rounds(int64_t rows, int64_t Q, int64_t K, int64_t height, int64_t cus) {
  const double l = 32.0 * (double)ceil_div(Q, 32), us = height == 128 ? 1.46 + 0.0437 * l : 3.28 + 0.0803 * l;
  const int64_t ncb = ceil_div(K, 128), round = height * 8 * walkers(cus, ncb);
  const double layers = (double)ceil_div(8 * ncb, cus);  // more column blocks than compute units on an XCD: one after the other
  const int64_t whole = rows / round, left = rows - whole * round, direct = ceil_div(left, 32) * ceil_div(K, 32);
  Rounds r{us * layers * ((double)whole + (left ? 0.67 + 0.33 * (double)left / (double)round : 0.0)), rows};
  const double two = us * layers * (double)whole + 3.1 + (9e-4 + 2.6e-5 * (double)Q) * (double)direct;
  if (whole > 0 && left > 0 && Q >= 16 && direct <= 1280 && two < r.us) r = {two, rows - left};
  return r;
}
inline int ttm_split(int64_t rows, int64_t Q, int64_t K, const float *Bp, const float *C, int64_t ldc, float *Ap, hipStream_t st) {
  const int64_t cus = compute_units();
  if (cus < 1) return DASTAC_EHIP;
  if (K <= 32) return launch_split<Tile<4, 1, 1, 1>>(rows, Q, K, Bp, C, ldc, Ap, cus, st);
  if (K <= 64) return launch_split<Tile<4, 1, 1, 2>>(rows, Q, K, Bp, C, ldc, Ap, cus, st);
  const Rounds small = ttm_rounds(rows, Q, K, 128, cus);
  Rounds large = ttm_rounds(rows, Q, K, 256, cus);
  const int64_t out = 4 * rows * K;  // bytes
  if (Q <= 64 && out > 250000000 && (Q > 32 || out < 430000000 || ceil_div(K, 128) != 4)) large = {0.0, rows};
  const Rounds &r = large.us < small.us ? large : small;
  const int status = large.us < small.us ? launch_split<Tile<4, 2, 2, 2>>(r.rows, Q, K, Bp, C, ldc, Ap, cus, st)
                                         : launch_split<Tile<4, 2, 1, 2>>(r.rows, Q, K, Bp, C, ldc, Ap, cus, st);
  if (status != DASTAC_OK || r.rows == rows) return status;
  return ttm_direct(rows - r.rows, Q, K, Bp + r.rows * Q, C, ldc, Ap + r.rows * K, st);
}
inline int ttm_split(int64_t, int64_t, int64_t, const double *, const double *, int64_t, double *, hipStream_t) { return DASTAC_EINVAL; }

template <typename T>
int ttm_ut(int64_t n, int64_t Q, int64_t K, const T *Bp, const T *C, int64_t ldc, T *Ap, void *stream) {
  constexpr int64_t kB = (int64_t)sizeof(T);
  if (n < 0 || Q < 1 || K < 1 || ldc < Q) return DASTAC_EINVAL;
  if (!uhc_ok(n, Q) || !uhc_ok(n, K) || ld_too_large(ldc) || K > ((int64_t)1 << 40) / ldc) return DASTAC_EOVERFLOW;
  if (n == 0) return DASTAC_OK;
  if (!Bp || !C || !Ap) return DASTAC_ENULL;
  const int64_t rows = tri(n);
  if (overlaps(Ap, rows * K * kB, Bp, rows * Q * kB) || overlaps(Ap, rows * K * kB, C, view_bytes(K, ldc, Q, kB)))
    return DASTAC_EALIAS;
  if (direct_serves<T>(rows, Q, K)) return ttm_direct(rows, Q, K, Bp, C, ldc, Ap, stream);
  if (split_serves(rows, Q, K, Bp)) return ttm_split(rows, Q, K, Bp, C, ldc, Ap, (hipStream_t)stream);
  const int64_t nrb = ceil_div(rows, kTileM), ncb = ceil_div(K, kTileN);
  if (ncb > (1 << 20)) return DASTAC_EOVERFLOW;
  // about two workgroups per compute unit (256 of them), each walking a strided set of row blocks
  int64_t lanes = ceil_div(512, 8 * ncb);
  if (lanes > ceil_div(nrb, 8)) lanes = ceil_div(nrb, 8);
  const int64_t grid = 8 * lanes * ncb;
  ttm_mfma_kernel<T><<<(unsigned)grid, kTileThreads, 0, (hipStream_t)stream>>>(rows, Q, K, Bp, C, ldc, Ap, (int)lanes,
                                                                             (int)ncb);
  return launch_status();
}

}  // namespace

extern "C" {

int64_t dastac_uhc_count(int64_t n, int64_t Q) {
  if (!uhc_ok(n, Q)) return -1;
  return tri(n) * Q;
}

int64_t dastac_uhc_offset(int64_t n, int64_t Q, int64_t i, int64_t j, int64_t l) {
  if (!uhc_ok(n, Q) || i < 0 || j < i || j >= n || l < 0 || l >= Q) return -1;
  return tri_offset(n, i, j) * Q + l;
}

int dastac_pack_uhc_f32(int64_t n, int64_t Q, const float *dense, float *packed, void *stream) {
  return uhc_copy<true, float>(n, Q, dense, packed, stream);
}

int dastac_unpack_uhc_f32(int64_t n, int64_t Q, const float *packed, float *dense, void *stream) {
  return uhc_copy<false, float>(n, Q, packed, dense, stream);
}

int dastac_pack_uhc_f64(int64_t n, int64_t Q, const double *dense, double *packed, void *stream) {
  return uhc_copy<true, double>(n, Q, dense, packed, stream);
}

int dastac_unpack_uhc_f64(int64_t n, int64_t Q, const double *packed, double *dense, void *stream) {
  return uhc_copy<false, double>(n, Q, packed, dense, stream);
}

int dastac_ttm_ut_f32(int64_t n, int64_t Q, int64_t K, const float *Bp, const float *C, int64_t ldc, float *Ap,
                      void *stream) {
  return ttm_ut<float>(n, Q, K, Bp, C, ldc, Ap, stream);
}

// Double precision (the paper's element type): the same kernel on the fp64 matrix cores.
int dastac_ttm_ut_f64(int64_t n, int64_t Q, int64_t K, const double *Bp, const double *C, int64_t ldc, double *Ap,
                      void *stream) {
  return ttm_ut<double>(n, Q, K, Bp, C, ldc, Ap, stream);
}

}  // extern "C"

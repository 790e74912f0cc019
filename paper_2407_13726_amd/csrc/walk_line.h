// How MTTKRP's walks (mttkrp_walk.hip) share their work: plain C++ on whole numbers, the same on host and device.
//
// The plane (j,k) of a tensor of order n is cut into blocks of kB x kB, aligned to its lower right corner: block row q (from the bottom) holds rows
// j in [n - kB(q+1), n - kB q) and blocks p = 0..q (from the right), block p columns k in [n - kB(p+1), n - kB p); what is left of 0 is cut off.  A slice i has the
// rows j >= i, so of a block row it has kB/16 steps of sixteen rows, or those from the step that holds row i on.
//
// A block row is dealt out as runs of neighbouring blocks: as many of `run` (a power of two, four at most) as there are, then two, then one.  The line: for every group
// of columns, the block rows from the bottom, the runs of each, the steps (all slices, in order) of each run times its blocks, and kSwitch steps that nobody has, what it
// costs a workgroup to end one run and begin another, so that those who do have less.
#pragma once
#include "index_poly.h"

namespace dastac {

constexpr int kWalkers = 8;             // wavefronts of a workgroup
constexpr int kSwitch = 3 * kWalkers;   // (without it n=256, R=32 fp32 19.1 us, with it 13.1; six steps a wavefront instead of three 13.5)
constexpr int kWalkMost = 2048;         // steps of one walk of a wavefront, and so slices that it can note (a bit each)

template <int kB>
DASTAC_HD int ragged_before(int v) {  // steps of the slices that begin at rows 0..v-1 of a block row
  constexpr int kS = kB / 16;
  const int g = v / 16;
  return 16 * (kS * g - g * (g - 1) / 2) + (v % 16) * (kS - g);
}
template <int kB>
DASTAC_HD int row_steps(int n, int q) {  // steps of one block of block row q, over all slices
  const int j0 = n - kB * (q + 1);
  return j0 >= 0 ? kB / 16 * j0 + ragged_before<kB>(kB) : ragged_before<kB>(kB) - ragged_before<kB>(-j0);
}
DASTAC_HD int runs_of(int blocks, int run) { return blocks / run + (blocks & (run >> 1) ? 1 : 0) + (blocks & (run >> 2) ? 1 : 0); }
template <int kB>
DASTAC_HD int64_t row_line(int n, int q, int run) {
  return (int64_t)(q + 1) * row_steps<kB>(n, q) + kSwitch * runs_of(q + 1, run);
}
template <int kB>
DASTAC_HD int64_t group_line(int n, int run) {
  int64_t all = 0;
  for (int q = 0; q < (n + kB - 1) / kB; ++q) all += row_line<kB>(n, q, run);
  return all;
}

// What stands on the line from `at` on: steps [from, to) of each of `width` blocks p0.. of block row q, for group `group`; `next` is the place behind it, no further than
// `stop` and than kWalkMost steps a wavefront.  from == to: nothing (between two runs).
struct Run {
  int group, q, p0, width, from, to;
  int64_t next;
};
template <int kB>
DASTAC_HD Run run_at(int n, int run, int64_t group_steps, int64_t at, int64_t stop) {
  Run r;
  int64_t left = at;
  r.group = 0;
  if (left >= group_steps) {
    r.group = (int)(left / group_steps);
    left -= r.group * group_steps;
  }
  r.q = 0;
  for (int64_t line; r.q < (n + kB - 1) / kB - 1 && left >= (line = row_line<kB>(n, r.q, run)); ++r.q) left -= line;
  const int len = row_steps<kB>(n, r.q);
  r.p0 = 0, r.width = run;
  int in = (int)left;
  while (true) {
    while (r.p0 + r.width > r.q + 1) r.width >>= 1;
    if (in < r.width * len + kSwitch) break;
    in -= r.width * len + kSwitch;
    r.p0 += r.width;
  }
  const int ahead = r.width * len - in;  // steps left of this run
  r.from = r.to = 0;
  if (ahead <= 0) {
    r.next = at + ahead + kSwitch;
    return r;
  }
  r.next = at + ahead < stop ? at + ahead : stop;
  if (r.next - at > (int64_t)kWalkMost * kWalkers) r.next = at + (int64_t)kWalkMost * kWalkers;
  r.from = in / r.width, r.to = (in + (int)(r.next - at)) / r.width;
  return r;
}

// Step s of a block of block row q: slice i and step t of it (rows n - kB(q+1) + 16 t ..+15).
struct Place {
  int i, t;
};
template <int kB>
DASTAC_HD Place place_of(int n, int q, int s) {
  constexpr int kS = kB / 16;
  const int j0 = n - kB * (q + 1);
  Place p;
  if (j0 > 0 && s < kS * j0) {
    p.i = s / kS, p.t = s % kS;
    return p;
  }
  s += j0 > 0 ? -kS * j0 : ragged_before<kB>(-j0);
  int g = 0;
  while (s >= 16 * (kS - g)) s -= 16 * (kS - g), ++g;
  p.i = j0 + 16 * g + s / (kS - g), p.t = g + s % (kS - g);
  return p;
}
// the first step of slice i in the block row that begins at row j0
DASTAC_HD int first_step(int i, int j0) { return i > j0 ? (i - j0) / 16 : 0; }

}  // namespace dastac

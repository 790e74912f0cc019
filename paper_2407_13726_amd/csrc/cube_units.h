// How the third-order polynomial-regression tensor is cut into tiles of (i,j) pairs by columns k; plain C++, nothing of the runtime.
#pragma once
#include "index_poly.h"

namespace dastac {

constexpr int kCubeSub = 32;  // columns k of a tile

// ---- rows kernel: strips of NS slices i and sixteen rows j, from the group's first slice on -------------------------
// Groups of slices from the two ends share a line of workgroups: together they have as many row blocks as the first alone, or one more.
DASTAC_HD int strip_columns(int d) { return (d + 15) / 16 + 1; }
DASTAC_HD int strip_lines(int d, int NS) { return ((d + NS - 1) / NS + 1) / 2; }
// Group and row block of workgroup (x, y); false: none.
DASTAC_HD bool strip_of(int d, int NS, int x, int y, int &group, int &block) {
  const int mine = (d - NS * y + 15) / 16;
  group = x < mine ? y : (d + NS - 1) / NS - 1 - y;
  block = x < mine ? x : x - mine;
  if (x >= mine && group == y) return false;  // the group in the middle has no other
  return NS * group + 16 * block < d;
}

// ---- direct kernel: tiles of NT * 4 slices i, 8 rows j and 32 columns k --------------------------------------------
// Units: row block J (eight j), a group of 4 NT slices, 32 columns k from 8 J on (NT is 1 or 2).
constexpr int kCubeRowsD = 8;
DASTAC_HD int units_of_row_block(int d, int NT, int J) {
  const int slices = kCubeRowsD * (J + 1) < d ? kCubeRowsD * (J + 1) : d;
  return (d - kCubeRowsD * J + kCubeSub - 1) / kCubeSub * ((slices + 4 * NT - 1) / (4 * NT));
}
// Row blocks 4b..4b+3, wholly inside (b < d / 32): each has d/32 - b column blocks, the first ceil(d%32 / 8) of them one more.
DASTAC_HD int units_of_four(int d, int NT, int b) {
  const int a = d / kCubeSub - b, c = (d % kCubeSub + kCubeRowsD - 1) / kCubeRowsD;
  return (a * (16 * b + 10) + 4 * b * c + c * (c + 1) / 2) * (2 / NT);
}
DASTAC_HD int64_t direct_units(int d, int NT) {
  int64_t t = 0;
  for (int J = 0; kCubeRowsD * J < d; ++J) t += units_of_row_block(d, NT, J);
  return t;
}
struct CubeTile {
  int i0, j0, k0;
};
DASTAC_HD CubeTile direct_tile(int d, int NT, int unit) {
  int J = 0;
  while (J / 4 < d / kCubeSub && unit >= units_of_four(d, NT, J / 4)) unit -= units_of_four(d, NT, J / 4), J += 4;
  while (unit >= units_of_row_block(d, NT, J)) unit -= units_of_row_block(d, NT, J), ++J;
  const int nK = (d - kCubeRowsD * J + kCubeSub - 1) / kCubeSub;
  return CubeTile{4 * NT * (unit / nK), kCubeRowsD * J, kCubeRowsD * J + kCubeSub * (unit % nK)};
}

// ---- staged kernel: tiles of 16 slices i, 16 rows j and 32 wn columns k, wn <= 4 -----------------------------------
constexpr int kCubeRowsS = 16, kCubeSlices = 16;
DASTAC_HD int cube_weight(int wn) { return wn == 1 ? 16 : wn == 2 ? 19 : wn == 3 ? 24 : 29; }  // what a step costs
// column blocks of row block J, the chunks of at most four that they are cut into, groups of slices
DASTAC_HD int subs_of(int d, int J) { return (d - kCubeRowsS * J + kCubeSub - 1) / kCubeSub; }
DASTAC_HD int chunks_of(int nsub) { return (nsub + 3) / 4; }
DASTAC_HD int groups_of(int d, int J) { return ((kCubeRowsS * (J + 1) < d ? kCubeRowsS * (J + 1) : d) + kCubeSlices - 1) / kCubeSlices; }
DASTAC_HD int weight_of_chunks(int nsub, int nch) {
  return nsub % nch * cube_weight(nsub / nch + 1) + (nch - nsub % nch) * cube_weight(nsub / nch);
}
DASTAC_HD int64_t staged_weight(int d) {  // of one step of all units
  int64_t t = 0;
  for (int J = 0; kCubeRowsS * J < d; ++J) t += (int64_t)groups_of(d, J) * weight_of_chunks(subs_of(d, J), chunks_of(subs_of(d, J)));
  return t;
}
// Row blocks with one number of chunks follow each other, eight at a time (the first of them fewer).  f(number of chunks, first row block, end) for each run,
// until f returns true.
template <typename F>
DASTAC_HD void chunk_runs(int d, F f) {
  const int blocks = (d + kCubeRowsS - 1) / kCubeRowsS;
  int nch = (d + 4 * kCubeSub - 1) / (4 * kCubeSub), J = 0;
  while (J < blocks) {
    const int end = (d - 4 * kCubeSub * (nch - 1) + kCubeRowsS - 1) / kCubeRowsS;
    if (f(nch, J, end)) return;
    J = end, --nch;
  }
}
// Units in all, and f(tile, wn) for unit number `unit`: row block after row block (widest chunks first, so that a launch ends with small units), group, chunk.
DASTAC_HD int64_t staged_units(int d) {
  int64_t t = 0;
  chunk_runs(d, [&](int nch, int J, int end) { return t += (int64_t)nch * (end * (end + 1) / 2 - J * (J + 1) / 2), false; });
  return t;
}
template <typename F>
DASTAC_HD void staged_unit(int d, int unit, F f) {
  chunk_runs(d, [&](int nch, int J, int end) {
    const int all = nch * (end * (end + 1) / 2 - J * (J + 1) / 2);  // row block J has J + 1 groups
    if (unit >= all) return unit -= all, false;
    while (unit >= nch * (J + 1)) unit -= nch * (J + 1), ++J;
    const int nsub = subs_of(d, J), c = unit % nch, more = c < nsub % nch ? 1 : 0;
    f(CubeTile{kCubeSlices * (unit / nch), kCubeRowsS * J, kCubeRowsS * J + kCubeSub * (c * (nsub / nch) + (more ? c : nsub % nch))}, nsub / nch + more);
    return true;
  });
}
// The steps of all units (row block, group, chunk, `steps` each) stand on one line, cube_weight(wn) apart; total = staged_weight * steps is cut
// into `parts` equal parts.  f(tile, wn, s0, s1) for every unit that has steps beginning in part `part`.
template <typename F>
DASTAC_HD void staged_part(int d, int steps, int64_t total, int64_t part, int64_t parts, F f) {
  int64_t at = total * part / parts;
  const int64_t end = total * (part + 1) / parts;
  if (at >= end) return;
  // the row block and group that `at` lies in, and where on the line they begin
  int J = 0, nsub = subs_of(d, 0), nch = chunks_of(nsub);
  int64_t begin = 0, per_group = (int64_t)weight_of_chunks(nsub, nch) * steps;
  while (at >= begin + per_group * groups_of(d, J)) {
    begin += per_group * groups_of(d, J), ++J;
    nsub = subs_of(d, J), nch = chunks_of(nsub), per_group = (int64_t)weight_of_chunks(nsub, nch) * steps;
  }
  int g = (int)((at - begin) / per_group), c = 0;
  begin += g * per_group;
  while (true) {
    const int more = c < nsub % nch ? 1 : 0, wn = nsub / nch + more;
    const int64_t w = cube_weight(wn), next = begin + w * steps;
    if (at < next) {
      const int s0 = (int)((at - begin + w - 1) / w), s1 = (int)(((end < next ? end : next) - begin + w - 1) / w);
      if (s0 < s1)
        f(CubeTile{kCubeSlices * g, kCubeRowsS * J, kCubeRowsS * J + kCubeSub * (c * (nsub / nch) + (more ? c : nsub % nch))}, wn, s0, s1);
      at = next;
    }
    if (at >= end) return;
    begin = next;
    if (++c == nch) {
      c = 0;
      if (++g == groups_of(d, J)) {
        g = 0, ++J;
        if (kCubeRowsS * J >= d) return;
        nsub = subs_of(d, J), nch = chunks_of(nsub);
      }
    }
  }
}

}  // namespace dastac

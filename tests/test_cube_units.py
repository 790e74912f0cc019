"""How the third-order polynomial-regression tensor is cut into tiles: every element i<=j<=k in exactly one strip of the rows kernel, one
tile of the direct kernel, one unit of the staged one and, for every step of samples, in exactly one of its parts; closed forms of the counts against the sums."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "cube_units.h"
using namespace dastac;
// adds `by` to every element of the tile that belongs to the tensor
static void cover(std::vector<int> &seen, int d, CubeTile t, int ni, int nj, int nk, int by) {
  for (int i = t.i0; i < t.i0 + ni; ++i)
    for (int j = t.j0; j < t.j0 + nj; ++j)
      for (int k = t.k0; k < t.k0 + nk; ++k)
        if (i <= j && j <= k && k < d) seen[tet_offset(d, i, j, k)] += by;
}
static bool all(const std::vector<int> &seen, int value) {
  for (int v : seen) if (v != value) return false;
  return true;
}
int main(int, char **argv) {
  const int d = atoi(argv[1]), steps = atoi(argv[2]);
  for (int NT = 1; NT <= 2; ++NT) {
    std::vector<int> seen(tet(d), 0);
    const int64_t units = direct_units(d, NT);
    for (int64_t u = 0; u < units; ++u) {
      const CubeTile t = direct_tile(d, NT, (int)u);
      if (t.i0 >= d || t.j0 >= d || t.k0 >= d) return printf("direct: empty tile\n"), 1;
      cover(seen, d, t, 4 * NT, 8, 32, 1);
    }
    if (!all(seen, 1)) return printf("direct, NT=%d: not a partition\n", NT), 1;
  }
  for (int NS = 1; NS <= 2; ++NS) {
    std::vector<int> seen(tet(d), 0);
    for (int y = 0; y < strip_lines(d, NS); ++y)
      for (int x = 0; x < strip_columns(d); ++x) {
        int group, block;
        if (!strip_of(d, NS, x, y, group, block)) continue;
        cover(seen, d, CubeTile{NS * group, NS * group + 16 * block, NS * group + 16 * block}, NS, 16, d, 1);
      }
    if (!all(seen, 1)) return printf("rows, NS=%d: not a partition\n", NS), 1;
  }
  {
    std::vector<int> seen(tet(d), 0);
    const int64_t units = staged_units(d);
    bool inside = true;
    int calls = 0;
    for (int64_t u = 0; u < units; ++u)
      staged_unit(d, (int)u, [&](const CubeTile &t, int wn) {
        inside = inside && t.i0 < d && t.j0 < d && t.k0 < d && 1 <= wn && wn <= 4;
        cover(seen, d, t, 16, 16, 32 * wn, 1), ++calls;
      });
    if (!inside || calls != units || !all(seen, 1)) return printf("staged, units: not a partition\n"), 1;
  }
  for (int parts : {1, 7, 256}) {
    std::vector<int> seen(tet(d), 0);
    const int64_t total = staged_weight(d) * steps;
    bool inside = true;
    for (int p = 0; p < parts; ++p)
      staged_part(d, steps, total, p, parts, [&](const CubeTile &t, int wn, int s0, int s1) {
        inside = inside && 0 <= s0 && s0 < s1 && s1 <= steps && 1 <= wn && wn <= 4;
        cover(seen, d, t, 16, 16, 32 * wn, s1 - s0);
      });
    if (!inside || !all(seen, steps)) return printf("staged, %d parts: not a partition\n", parts), 1;
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("cube")
    src, exe = d / "cube.cpp", d / "cube"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2407_13726_amd", "csrc"), str(src), "-o", str(exe)])
    return str(exe)


@pytest.mark.parametrize("d,steps", [(1, 1), (3, 2), (7, 5), (8, 1), (9, 3), (15, 2), (16, 7), (17, 1), (25, 4), (31, 3), (32, 5), (33, 1), (40, 9), (63, 2), (64, 1),
                                     (65, 3), (95, 1), (104, 4), (127, 1), (128, 3), (129, 2), (160, 1), (209, 5), (257, 1)])
def test_tiles_partition_the_tensor(program, d, steps):
    subprocess.check_output([program, str(d), str(steps)])

"""How MTTKRP's walks share their work: every step of every block, slice and group of columns has one wavefront, whatever the cut."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <map>
#include <tuple>
#include "walk_line.h"
using namespace dastac;
template <int kB>
int check(int n, int run, int groups, int wgs) {
  constexpr int kS = kB / 16;
  std::map<std::tuple<int, int, int, int, int>, int> seen;
  const int64_t line = group_line<kB>(n, run), all = line * groups;
  int longest = 0;
  for (int g = 0; g < wgs; ++g) {
    int64_t at = all / wgs * g + (g < all % wgs ? g : all % wgs);
    const int64_t stop = at + all / wgs + (g < all % wgs ? 1 : 0);
    while (at < stop) {
      const Run r = run_at<kB>(n, run, line, at, stop);
      if (r.next <= at) return 1;
      at = r.next;
      if (r.from == r.to) continue;
      if (r.p0 + r.width > r.q + 1 || kWalkers % r.width) return 2;
      for (int w = 0; w < kWalkers; ++w) {
        const int parts = kWalkers / r.width, b = w % r.width, no = w / r.width;
        const int lo = r.from + (r.to - r.from) * no / parts, hi = r.from + (r.to - r.from) * (no + 1) / parts;
        if (hi - lo > kWalkMost) return 3;
        if (hi - lo > longest) longest = hi - lo;
        if (hi <= lo) continue;
        const int j0 = n - kB * (r.q + 1);
        Place p = place_of<kB>(n, r.q, lo);
        for (int s = lo; s < hi; ++s) {  // as the kernel goes on from its first step
          const Place q = place_of<kB>(n, r.q, s);
          if (p.i != q.i || p.t != q.t) return 4;
          if (++seen[std::make_tuple(r.group, r.q, r.p0 + b, p.i, p.t)] != 1) return 5;
          if (++p.t == kS) ++p.i, p.t = first_step(p.i, j0);
        }
      }
    }
  }
  int64_t want = 0;
  for (int q = 0; q < (n + kB - 1) / kB; ++q)
    for (int i = 0; i < n - kB * q; ++i)
      for (int t = first_step(i, n - kB * (q + 1)); t < kS; ++t, want += (int64_t)(q + 1) * groups) {
        const int j0 = n - kB * (q + 1) + 16 * t;
        if (j0 + 15 < i || j0 + 15 < 0) return 6;  // a step without a row
        for (int c = 0; c < groups; ++c)
          for (int p = 0; p <= q; ++p)
            if (!seen.count(std::make_tuple(c, q, p, i, t))) return 7;
      }
  if ((int64_t)seen.size() != want) return 8;
  printf("%d %lld\n", longest, (long long)want);
  return 0;
}
int main(int argc, char **argv) {
  const int kB = atoi(argv[1]), n = atoi(argv[2]), run = atoi(argv[3]), groups = atoi(argv[4]), wgs = atoi(argv[5]);
  return kB == 128 ? check<128>(n, run, groups, wgs) : check<64>(n, run, groups, wgs);
}
"""


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    d = tmp_path_factory.mktemp("line")
    src, exe = d / "line.cpp", d / "line"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2407_13726_amd", "csrc"), str(src), "-o", str(exe)])
    return lambda *a: [int(x) for x in subprocess.check_output([str(exe), *map(str, a)], text=True).split()]


@pytest.mark.parametrize("kB,n,run,groups,wgs", [
    (128, 3, 4, 1, 8), (128, 89, 4, 2, 16), (128, 127, 4, 1, 80), (128, 128, 4, 1, 80), (128, 129, 4, 3, 256), (128, 256, 4, 1, 256), (128, 257, 2, 2, 256),
    (128, 300, 4, 1, 40), (128, 400, 2, 2, 256), (128, 513, 4, 1, 256), (128, 700, 2, 1, 304), (64, 65, 4, 5, 40), (64, 127, 4, 1, 104), (64, 128, 4, 2, 256),
    (64, 180, 2, 3, 256), (64, 193, 4, 1, 8), (64, 333, 2, 1, 256), (64, 450, 4, 1, 256),
    # what the kernels launch: one block at a time but for one tile of single precision, two from n=450 on, four from n=1150 on
    (128, 111, 1, 1, 72), (128, 129, 1, 3, 112), (128, 333, 1, 1, 256), (128, 449, 1, 2, 256), (128, 450, 2, 1, 256), (128, 640, 1, 2, 256), (128, 1149, 2, 1, 256), (128, 1150, 4, 1, 256),
    (64, 65, 1, 33, 256), (64, 81, 1, 6, 80), (64, 128, 1, 3, 256), (64, 179, 1, 4, 256), (64, 229, 1, 3, 256), (64, 333, 1, 1, 256), (64, 450, 1, 1, 240), (64, 700, 1, 2, 256)])
def test_every_step_has_one_wavefront(check, kB, n, run, groups, wgs):
    longest, steps = check(kB, n, run, groups, wgs)
    if steps > 8 * wgs * 4:  # no wavefront has much more than its share
        assert longest <= 1.15 * (steps + 24 * 300) / (8 * wgs) + 2


def test_a_walk_has_an_end(check):
    """A workgroup that has everything: the walks of a single block of so many slices are cut."""
    assert check(128, 2300, 4, 1, 1)[0] == 2048

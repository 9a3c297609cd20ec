"""The map from workgroup numbers to the tiles of a matrix product, run on the host: every tile once, and no XCD
(workgroup number mod 8) with more than one tile beyond another where the tiles are dealt in runs.  And the plans that
split key ranges: within their bounds, and lists by the number of compute units alone (twice of both is split the same)."""
import os
import subprocess

import pytest

from paper_2502_02406_amd import build as B

PROGRAM = r"""
#include "lvx_internal.h"
#include "lvx_mfma.h"
#include <cstdio>
#include <vector>
int main() {
  for (int n_rt = 1; n_rt <= 300; n_rt = n_rt < 70 ? n_rt + 1 : n_rt + 37)
    for (int n_ct : {1, 2, 3, 4, 6, 8, 16, 23, 32}) {
      const long tiles = (long)n_rt * n_ct, grid = lvx::tile_grid(n_rt, n_ct);
      std::vector<int> seen(tiles, 0);
      long of_xcd[8] = {};
      for (long pid = 0; pid < grid; ++pid) {
        lvx::HeadWork w;
        if (!lvx::tile_decode(pid, n_rt, n_ct, &w)) continue;
        if (w.head < 0 || w.head >= n_rt || w.item < 0 || w.item >= n_ct) { printf("%d x %d: workgroup %ld outside\n", n_rt, n_ct, pid); return 1; }
        ++seen[(long)w.head * n_ct + w.item];
        ++of_xcd[pid % 8];
      }
      for (long t = 0; t < tiles; ++t)
        if (seen[t] != 1) { printf("%d x %d: tile %ld taken %d times\n", n_rt, n_ct, t, seen[t]); return 1; }
      long lo = of_xcd[0], hi = of_xcd[0];
      for (long x : of_xcd) { lo = x < lo ? x : lo; hi = x > hi ? x : hi; }
      if (lvx::tile_runs(n_rt, n_ct) && hi - lo > 1) { printf("%d x %d: from %ld to %ld tiles\n", n_rt, n_ct, lo, hi); return 1; }
    }
  return 0;
}
"""


def test_runs_are_even(tmp_path):
    src, exe = tmp_path / "map.hip", tmp_path / "map"
    src.write_text(PROGRAM)
    subprocess.run([B.HIPCC] + B.FLAGS + ["-I", B.CSRC, "-I", os.path.join(B.HERE, "..", "include"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


PLANS = r"""
#include "lvx_internal.h"
#include <cstdio>
int main() {
  for (int n_cu : {32, 64, 104, 128, 256})
    for (long wgs = 1; wgs <= 3 * n_cu; wgs = wgs < 40 ? wgs + 1 : wgs + wgs / 17)
      for (int n_tiles = 1; n_tiles < 5000; n_tiles = n_tiles * 5 / 4 + 1) {
        const int s = lvx::list_split(wgs, n_tiles, n_cu), t = lvx::list_split(2 * wgs, n_tiles, 2 * n_cu);
        if (s != t || s < 1 || (s > 1 && 3 * s > n_tiles)) { printf("list: %ld x %d on %d: %d and %d\n", wgs, n_tiles, n_cu, s, t); return 1; }
        if (s * wgs > 2 * n_cu && s > 2) { printf("list: %ld x %d on %d: %d\n", wgs, n_tiles, n_cu, s); return 1; }
        const lvx::TailPlan p = lvx::pick_tail(8, (int)wgs, n_tiles, n_cu, 64, 2e-6, 1e-5, 1e-7, 5e-6);
        if (p.whole < 0 || p.whole > wgs || p.parts < 1 || (p.parts > 1 && (3 * p.parts > n_tiles || p.whole == wgs))) {
          printf("tail: %ld x %d on %d: %d, %d\n", wgs, n_tiles, n_cu, p.whole, p.parts);
          return 1;
        }
      }
  return 0;
}
"""


def test_plans_scale_with_the_device(tmp_path):
    src, exe = tmp_path / "plans.hip", tmp_path / "plans"
    src.write_text(PLANS)
    subprocess.run([B.HIPCC] + B.FLAGS + ["-I", B.CSRC, "-I", os.path.join(B.HERE, "..", "include"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout

"""The order in which workgroups take whole row tiles and parts of the others (no GPU needed: the decode is host code as well): every
item once, a head's on one XCD where there are as many heads, and the whole tiles of all heads before any part, so that the parts fill
what these leave."""
import os
import subprocess
import tempfile

import pytest

from paper_2502_02406_amd import build as B

_MAIN = r"""
#include "lvx_internal.h"
#include "lvx_mfma.h"
#include <cstdio>
int main(int, char** v) {
  const int heads = atoi(v[1]), whole = atoi(v[2]), parts = atoi(v[3]);
  const long grid = lvx::tail_grid(heads, whole, parts);
  for (long pid = 0; pid < grid; ++pid) {
    lvx::HeadWork w;
    if (lvx::tail_decode(pid, heads, whole, parts, &w)) printf("%ld %d %d\n", pid, w.head, w.item);
  }
}
"""


@pytest.fixture(scope="module")
def program():
    with tempfile.TemporaryDirectory() as tmp:
        src, exe = os.path.join(tmp, "order.hip"), os.path.join(tmp, "order")
        with open(src, "w") as f:
            f.write("#include <cstdlib>\n" + _MAIN)
        r = subprocess.run([B.HIPCC] + B.FLAGS + ["-I", B.CSRC, src, "-o", exe], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        yield exe


@pytest.mark.parametrize("heads", [1, 3, 4, 8, 12, 16, 40])
@pytest.mark.parametrize("whole,parts", [(0, 7), (16, 14), (21, 6), (32, 1)])
def test_whole_tiles_first(program, heads, whole, parts):
    out = subprocess.run([program, str(heads), str(whole), str(parts)], capture_output=True, text=True, check=True, timeout=60).stdout
    taken = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert sorted((h, i) for _, h, i in taken) == [(h, i) for h in range(heads) for i in range(whole + parts)]
    if whole:
        assert max(p for p, _, i in taken if i < whole) < min(p for p, _, i in taken if i >= whole)
    if heads % 8 == 0:
        for h in range(heads):
            assert len({p % 8 for p, hh, _ in taken if hh == h}) == 1

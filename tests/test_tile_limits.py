"""Tiles of one patch at the shared-memory limits of the plan (csrc/layout.h),
on the host: what fits is decided without the bank padding and the tables,
which such a tile may carry beyond the budget."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_01654_amd", "csrc")

# (element size, budget in KiB, slots): most free blocks that fit, -1 for none.
# Each pair's entries: slots 18 a slot, rays 4, sums 8 (float32: rays and relative
# poses again in float64), 28 a slot, the larger of four rows of 16-wide columns
# and the wavefronts' partials, then cells or source blocks and B terms, 2 bytes a block.
LIMITS = {(4, 80, 43): 44, (4, 80, 44): 45, (4, 80, 45): 42, (4, 80, 46): 37, (4, 80, 47): 33, (4, 80, 48): 29,
          (4, 80, 49): 24, (4, 80, 50): 20, (4, 80, 51): 15, (4, 80, 52): 11, (4, 80, 56): -1,
          (4, 150, 64): 65, (8, 150, 58): 59, (8, 150, 59): 60, (8, 150, 60): 57, (8, 150, 61): 54, (8, 150, 62): 52,
          (8, 150, 63): 49, (8, 150, 64): 46}


def test_one_patch_tiles_fit_up_to_their_limits(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    src = tmp_path / "limits.cpp"
    src.write_text("""
#define __host__
#define __device__
#include <cstdio>
#include "layout.h"
using namespace dpvba;
int main() {
  int ts, kib, Tn;
  while (scanf("%d %d %d", &ts, &kib, &Tn) == 3) {
    int most = -1, holes = 0, over = 0;
    for (int nb = 0; nb <= Tn + 1; ++nb) {
      const bool fits = tile_fits(1, Tn, nb, ts, kib * 1024, false);
      if (fits && most != nb - 1) ++holes;
      if (fits) most = nb;
      // what the kernels take is within a compute unit's 160 KiB
      if (fits && tile_lds_bytes(1, Tn, nb, ts) > 160 * 1024 - 256) ++over;
    }
    printf("%d %d %d\\n", most, holes, over);
  }
}
""")
    exe = str(tmp_path / "limits")
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    keys = list(LIMITS)
    r = subprocess.run([exe], input="\n".join(" ".join(map(str, k)) for k in keys), capture_output=True, text=True,
                       check=True)
    rows = [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
    assert {k: row[0] for k, row in zip(keys, rows)} == LIMITS
    assert all(row[1:] == (0, 0) for row in rows)

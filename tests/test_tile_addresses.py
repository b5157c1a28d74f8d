"""Addresses of the stored tiles inside a block, up to the most tile columns a block can
have: the first entry of a tile in 64 bits (a coarsest operator of 33,616 unknowns holds
4.5 GB of FP32 tiles), everything a wave adds to it in 32.  A host program with the
kernels' own header prints them; Python's integers are the reference."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = """
#include <cstdio>
#include "hblocks.hpp"
int main() {
  using namespace dpg;
  const int sizes[] = {1, 2, 724, 725, 1024, 1051, 1364, kMaxTiles};
  for (int nt : sizes)
    for (int I : {0, 1, nt / 2, nt - 2, nt - 1})
      for (int J : {0, 1, nt / 2, nt - 2, nt - 1}) {
        if (I < 0 || J < 0 || I >= nt || J >= nt) continue;
        const TileSpan t = tile_span(I, J);
        printf("%d %d %d %lld %d %d\\n", nt, I, J, (long long)t.first, t.entries, t.step);
      }
}
"""


def _first(i, j):
    return 1024 * (j * (j - 1) // 2 + i) + 576 * j


def test_tile_addresses_of_large_blocks(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "t.hip", tmp_path / "t"
    src.write_text(SOURCE)
    subprocess.run([HIPCC, "--cuda-host-only", "-std=c++17",
                    "-I", os.path.join(ROOT, "paper_2304_01728_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True, capture_output=True)
    rows = [tuple(map(int, r.split()))
            for r in subprocess.run([str(exe)], check=True, capture_output=True,
                                    text=True).stdout.splitlines()]
    assert max(r[0] for r in rows) == 4095
    assert max(8 * r[3] for r in rows if r[0] == 1051) > 2 ** 32
    for nt, i, j, first, entries, step in rows:
        lo, hi = min(i, j), max(i, j)
        assert first == _first(lo, hi)
        assert (entries, step) == ((1024, 64) if i != j else (576, 36))
        # the last entry of the tile ends where the next one (or the block) does
        after = _first(lo + 1, hi) if lo < hi else _first(0, hi + 1)
        assert first + entries == after
        assert 15 * step + (63 if i != j else 35) < entries
        assert 8 * entries < 2 ** 31

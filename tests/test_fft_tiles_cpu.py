"""Tiles of the transform passes (csrc/fft_tiles.hpp), checked on the host: whatever tile was measured, at
whatever precision, the run-time kernels get one that they can run."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_25161_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <initializer_list>
#include "fft_tiles.hpp"
using namespace fsd;
int main() {
  for (int N = 8; N <= 256; ++N) {
    int m = N;
    for (int r : {2, 3, 5})
      while (m % r == 0) m /= r;
    if (m != 1) continue;
    for (int rb : {4, 8})
      for (int t : {0, 1, 2, 3, 4, 6, 8, 16, 32, 64}) {
        const FftTile l = line_tile(N, t, rb), g = green_tile(N, t, rb);
        const size_t lds = size_t(2 * rb) * (2 * size_t(l.size) * fft_line_stride(N, l.size, 2 * rb) + N);
        std::printf("%d %d %d %d %d %zu %d %d %zu\n", N, rb, t, l.two_step, l.size, lds, g.two_step, g.size,
                    xgreen_shm(N, g.size, 2 * rb));
      }
  }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_run_time_passes_get_tiles_they_can_run(tmp_path):
    src, exe = tmp_path / "h.cpp", tmp_path / "h"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__host__=", "-D__device__=", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    rows = [list(map(int, l.split())) for l in subprocess.run([str(exe)], check=True, capture_output=True,
                                                              text=True).stdout.split("\n") if l]
    assert len(rows) == 46 * 20  # sides, precisions and tiles
    for N, rb, t, l2, B, lds, g2, G, gshm in rows:
        if not l2:
            assert B & (B - 1) == 0 and N % B == 0 and lds <= 65536, (N, rb, t, B, lds)
        if not g2:
            # the default of two row pairs takes up to 98 KB of a CU's 160 KB
            assert 1 <= G <= 64 and gshm <= 163840, (N, rb, t, G, gshm)
        if t and not l2 and (t & (t - 1)) == 0 and N % t == 0 and B != t:
            # a measured tile gives way only where it does not fit
            assert 2 * rb * (2 * t * N + N) > 65536 - 2 * rb * 2 * t * 64, (N, rb, t, B)

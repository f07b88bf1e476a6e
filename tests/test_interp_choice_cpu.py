"""The choice between interpolation by beads and by blocks (csrc/interp_choice.hpp) against measured times."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_25161_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include "interp_choice.hpp"
int main() {
  int le, bytes, systems, n, g, P;
  while (std::scanf("%d %d %d %d %d %d", &le, &bytes, &systems, &n, &g, &P) == 6) {
    fsd::InterpChoice c(le, bytes);
    for (int k = 0; k < systems; ++k) c.add(n, g, P);
    std::printf("%d\n", int(c.by_blocks()));
  }
}
"""

# sheared, bytes, beads, grid, support: us by beads, us by blocks (MI355X)
MEASURED = [
    (0, 8, 1000, 16, 14, 10.8, 67.8), (0, 8, 3000, 64, 14, 29.2, 22.8), (0, 8, 2000, 96, 14, 34.8, 24.7),
    (0, 8, 4096, 16, 14, 27.1, 253.1), (0, 8, 4096, 24, 21, 69.7, 270.7), (0, 8, 4096, 32, 10, 14.9, 47.4),
    (0, 8, 4096, 64, 6, 7.0, 11.7), (0, 8, 4096, 128, 14, 81.5, 36.2), (0, 8, 16384, 32, 14, 104.2, 311.8),
    (0, 8, 16384, 64, 14, 119.0, 71.4), (0, 8, 40000, 48, 10, 110.1, 140.8),
    (1, 8, 4096, 128, 14, 84.2, 42.2), (1, 8, 8192, 32, 14, 57.1, 268.2), (1, 8, 16384, 48, 14, 112.5, 171.4),
    (1, 8, 16384, 96, 14, 125.0, 93.0),
    (0, 4, 4096, 48, 10, 11.5, 19.1), (0, 4, 4096, 128, 14, 35.2, 28.2), (0, 4, 8192, 32, 14, 36.0, 117.1),
    (0, 4, 16384, 96, 14, 78.8, 41.8), (0, 4, 16384, 48, 6, 16.2, 23.6),
    (1, 4, 8192, 32, 14, 36.0, 200.0), (1, 4, 16384, 96, 14, 78.2, 60.5),
]


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_choice_follows_the_measured_times(tmp_path):
    src, exe = tmp_path / "h.cpp", tmp_path / "h"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def chosen(rows):
        text = "".join(" ".join(map(str, r)) + "\n" for r in rows)
        return list(map(int, subprocess.run([str(exe)], input=text, check=True, capture_output=True,
                                            text=True).stdout.split()))

    for r, c in zip(MEASURED, chosen([(r[0], r[1], 1, *r[2:5]) for r in MEASURED])):
        beads, blocks = r[5:]
        assert (beads, blocks)[c] <= 1.29 * min(beads, blocks), r  # the worst that the rule states
    # many small systems together fill the chip with blocks where one does not
    assert chosen([(0, 8, 1, 600, 24, 14), (0, 8, 64, 600, 24, 14)]) == [0, 1]

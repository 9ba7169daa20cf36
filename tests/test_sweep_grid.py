"""The grid of the scoring sweeps, on the host: the header that the launches and the kernels share."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_23200_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "sweep_grid.h"
int main(int, char** v) {
  const int units = atoi(v[1]), chunks = atoi(v[2]);
  const bool causal = atoi(v[3]) != 0;
  const ams::SweepGrid g = ams::sweep_grid(units, chunks, causal);
  std::vector<char> sweep((size_t)units * chunks), tail(units);
  int last_row = -1, twice = 0;
  bool in_order = true;
  for (int y = 0; y < g.y; ++y)
    for (int x = 0; x < g.x; ++x) {
      int bx, by;
      ams::sweep_place(x, y, g.x, chunks, bx, by);
      in_order = in_order && by >= last_row && bx >= 0 && bx < chunks;
      last_row = by;
      if (by < units) {
        twice += sweep[(size_t)by * chunks + bx]++;
      } else if (causal) {
        const int u = ams::sweep_tail(bx, by, chunks, units);
        if (u >= 0) twice += tail[u]++;
      }
    }
  size_t n = 0, m = 0;
  for (char c : sweep) n += c;
  for (char c : tail) m += c;
  std::printf("%d %d %d %d\n", g.y, (int)in_order, twice, (int)(n == sweep.size() && m == (causal ? tail.size() : 0)));
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "grid.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "grid.cpp"), "-o", str(d / "grid")], check=True)
    return str(d / "grid")


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("units,chunks", [(1, 1), (7, 3), (32767, 1), (32768, 1), (32768, 2), (43690, 2), (43691, 2), (65535, 1),
                                          (65535, 2), (65535, 7), (300, 128)])
def test_every_chunk_and_every_tail_once_within_the_grids_rows(program, units, chunks, causal):
    """The ABI takes up to 65535 units; the rows of the tails come on top of theirs."""
    rows, in_order, twice, all_there = map(int, subprocess.run([program, str(units), str(chunks), str(causal)], check=True,
                                                               capture_output=True, text=True).stdout.split())
    assert rows <= 65535 and in_order and twice == 0 and all_there

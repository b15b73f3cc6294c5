"""Numbers of the cells of a device build (csrc/cell_numbers.h), compiled on the
host: with more than 2^31 cells no number may come out below an array's end."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# Reads the starts per block (one count for all blocks of a level, level by level) and does what the
# scan and the cells kernel do with them: the sum before each block in CellSum, then cell_number.
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "cell_numbers.h"
using namespace octgrav;
int main(int argc, char** argv) {
  const long long nb = std::atoll(argv[1]), cap = std::atoll(argv[2]);
  CellSum at = 0;
  long long exact = 0, wrong = 0, written = 0;
  for (int L = 3; L < argc; ++L) {
    const CellSum k = std::atoll(argv[L]);
    for (long long b = 0; b < nb; ++b) {
      for (long long i : {0ll, (long long)k - 1}) {  // the block's first and last start
        if (k == 0) break;
        const int c = cell_number(at) + (int)i;
        wrong += c < 0 || (c < cap) != (exact + i < cap) || (c < cap && c != exact + i);
        written += c < cap;
      }
      at += k;
      exact += k;
    }
  }
  std::printf("%lld %lld %d %lld\n", (long long)at, wrong, at > kMaxCells, written);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("cells")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", f"-I{ROOT}/paper_1005_5384_amd/csrc", "-o",
                    str(d / "p"), str(d / "p.cpp")], check=True)
    return str(d / "p")


# Starts per block of 1024 particles: all of them pairs of coincident particles, one particle per leaf
# (a cell per pair from the level that separates the pairs down to the deepest), at the number of
# particles where the count passes 2^31, and at the largest; and a tree of few cells.
@pytest.mark.parametrize("n,levels", [(3.6e8, [1] + [2] * 9 + [512] * 12 + [0]), (2 ** 31 - 1, [1] + [512] * 21),
                                      (2 ** 31 - 1, [1024] * 22), (4e6, [1, 8, 64, 300, 0])])
def test_numbers_past_every_limit(program, n, levels):
    nb = (int(n) + 1023) // 1024
    cap = min(2 * int(n) + 64, (1 << 29) - 1)  # what the build allocates at first
    out = subprocess.run([program, str(nb), str(cap), *map(str, levels)], capture_output=True, text=True,
                         check=True).stdout.split()
    total, wrong, refused, written = map(int, out)
    assert total == nb * sum(levels) and wrong == 0
    assert refused == (total >= 1 << 29) and (written > 0)
    if n != 4e6:
        assert total > np.iinfo(np.int32).max

"""The walk of a group of lanes over a CSR row (csrc/swconv_rows.hpp), run on the host over the range of int32 row
pointers: every entry once, none beyond the row, and an end, also where the row ends at the last index of 31 bits.
And the pruning step's grid: a launch the device takes (less than 2^32 threads) for every row count that is accepted."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "swconv_rows.hpp"

static_assert(swconv::prune_groups(1) == 1 && swconv::prune_groups(16) == 1 && swconv::prune_groups(17) == 2, "");
constexpr bool grid_fits(int64_t rows) {
  return (uint64_t)swconv::prune_groups(rows) * swconv::kPruneThreads < ((uint64_t)1 << 32) &&
         (swconv::prune_groups(rows) == 1 << 23 || (int64_t)swconv::prune_groups(rows) * swconv::kPruneRows >= rows);
}
static_assert(grid_fits((1 << 27) + 1) && grid_fits(1 << 28) && grid_fits(((int64_t)1 << 31) - 257), "");

int main(int, char** argv) {
  const int32_t q0 = (int32_t)atoll(argv[1]), q1 = (int32_t)atoll(argv[2]);
  const long long entries = q1 > q0 ? (long long)q1 - q0 : 0;
  long long chunks = 0, seen = 0, last = -1;
  bool ok = true;
  swconv::for_row_chunks<16>(q0, q1, [&](uint32_t i, uint32_t n) {
    if (++chunks > entries / 16 + 2) exit(2);  // a walk that does not end
    ok = ok && n == (uint32_t)entries;
    for (uint32_t lane = 0; lane < 16; lane += i + 32 < n ? 15 : 1)  // first and last lane; all of them in the last chunks
      if (i + lane < n) {
        const size_t q = (size_t)q0 + i + lane;
        ok = ok && q < (size_t)q1 && (long long)q > last;
        last = (long long)q;
      }
    seen += n - i < 16 ? n - i : 16;
  });
  return ok && seen == entries && (entries == 0 || last == q1 - 1) ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk")
    (d / "walk.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_1702_08597_amd", "csrc"),
                           str(d / "walk.cpp"), "-o", str(d / "walk")])
    return lambda q0, q1: subprocess.run([str(d / "walk"), str(q0), str(q1)], timeout=60).returncode


TOP = 2 ** 31 - 1


@pytest.mark.parametrize("q0,q1", [(0, 0), (5, 3), (0, 1), (7, 22), (7, 23), (7, 24), (3, 36), (TOP - 1, TOP), (TOP - 15, TOP),
                                   (TOP - 16, TOP), (TOP - 17, TOP), (TOP - 40, TOP), (TOP - 40, TOP - 16), (0, TOP)])
def test_every_entry_once(walk, q0, q1):
    assert walk(q0, q1) == 0

"""The row and column that the factorisation's threads keep for the entries of A and J
(csrc/row_walk.hpp), compiled for the host and compared with integer division.

* Every size of the LDS classes' workgroups and waves, every thread, every n up to 512, over
  65,536 entries (more than 160 KB of LDS hold).
* The device-memory class (1024 threads), first, middle and last thread, every n up to 512, up
  to 2^28 entries: beyond 2^22 a quotient formed in FP32 is off by one for 164 of these n.
"""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_14344_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "row_walk.hpp"
static bool walk(int rank, int size, int n, int limit) {
  subadmm::RowWalk w(rank, size, n);
  for (int t = rank; t < limit; t += size, w.next())
    if (w.row != t / n || w.col != t % n) {
      std::printf("n %d size %d entry %d: row %d column %d\n", n, size, t, w.row, w.col);
      return false;
    }
  return true;
}
int main() {
  for (int n = 1; n <= 512; ++n) {
    for (int size : {64, 128, 256, 512})
      for (int rank = 0; rank < size; ++rank)
        if (!walk(rank, size, n, 65536)) return 1;
    for (int rank : {0, 511, 1023})
      if (!walk(rank, 1024, n, 1 << 28)) return 1;
  }
  return 0;
}
"""


def test_row_and_column_of_every_entry(tmp_path):
    src = tmp_path / "walk.cpp"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(tmp_path / "walk")],
                   check=True)
    r = subprocess.run([str(tmp_path / "walk")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout

"""The rule that sends the cutoffs of bfloat16 rows to one kernel or the other, compiled by itself: a K that keeps every entry
is the same as no K, in every size."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "warp_rules.hpp"
int main() {
  const int rows[] = {1, 200, 512, 513, 800, 1627, 4000, 70000}, sizes[] = {1, 8, 64, 65, 400, 513, 4096, 24576, 24577, 32768, 32769, 65536, 65537, 152064};
  for (int r : rows)
    for (int V : sizes) {
      const int off[] = {0, -1, V, V + 1, 1 << 30};
      for (int k : off) {
        if (sv::rows_in_registers(r, V, 1, &k) != sv::rows_in_registers(r, V, 1, off)) { std::printf("%d x %d, K = %d\n", r, V, k); return 1; }
        const int mixed[] = {0, k};
        if (sv::rows_in_registers(r, V, 2, mixed) != sv::rows_in_registers(r, V, 1, off)) { std::printf("%d x %d, K = 0 and %d\n", r, V, k); return 1; }
      }
      if (V <= 64 && sv::rows_in_registers(r, V, 1, off)) { std::printf("%d x %d, a list for one wavefront\n", r, V); return 1; }
      const int deep = 513, list = 512;
      if (V > deep && sv::rows_in_registers(r, V, 1, &deep) != (V <= 65536)) { std::printf("%d x %d, deep\n", r, V); return 1; }
      if (V > list && sv::rows_in_registers(r, V, 1, &list)) { std::printf("%d x %d, list\n", r, V); return 1; }
    }
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no compiler")
def test_a_k_of_the_whole_vocabulary_is_no_k(tmp_path):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2509_24328_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout

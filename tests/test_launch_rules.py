"""The rules for the demapping launches' grids and the second tier's workspace
(csrc/launch_rules.h), checked on the host: a plain C++ program built with g++
calls them.

Launches that write per-block sums stay within the blocks that the workspace
and the reduction are sized for, in every form of a call (the max-log LLR-only
form writes them although nothing reads them), and the size limit of the sweep
without allocation is the same for every set and number of SNR points."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2108_07001_amd", "csrc")

PROG = r"""
#include <cstdio>
#include <initializer_list>
#include "launch_rules.h"
int main() {
  long bad = 0, widest = 0;
  const long sizes[] = {1, 255, 256, 257, 100000, 262144, 262145, 393216, 393217, 1000000, 16000000, 4294967168};
  for (long N : sizes)
    for (int M = 2; M <= 4096; M *= 2)
      for (int S : {1, 2, 5, 41, 64, 200})
        for (int maxlog = 0; maxlog < 2; ++maxlog)
          for (int tx = 0; tx < 2; ++tx) {
            const bool one_kernel = !maxlog && M <= 16;             // what the driver passes
            const int g = air::vec_grid(N, M, S, !one_kernel || tx);
            if (!one_kernel || tx) bad += g > air::kMaxGrid;
            else widest = g > widest ? g : widest;
            bad += g < 1 || air::mfma_grid(N) > air::kMaxGrid || air::t2_grid(air::mfma_grid(N), M) > air::kMaxGrid;
            bad += air::snr_slices(g, S) < 1 || air::snr_slices(g, S) > S;
          }
  std::printf("%ld %ld\n", bad, widest);
  // the largest N of one SNR point in 48 MiB, FP32 sets and matrix cores
  const long bytes = 48l << 20;
  for (int M : {4, 16, 32, 4096})
    for (int S : {1, 2, 64}) {
      long lo = 1, hi = 1l << 31;
      while (hi - lo > 1) {
        const long N = (lo + hi) / 2;
        (air::lists_that_fit(air::list_size(N, air::vec_grid(N, M, S), false), bytes) >= 1 ? lo : hi) = N;
      }
      std::printf("%ld ", lo);
    }
  std::printf("\n");
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_launch_rules(tmp_path):
    src = tmp_path / "rules.cpp"
    src.write_text(PROG)
    exe = tmp_path / "rules"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    first, second = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    assert first.split() == ["0", "2048"]
    assert set(second.split()) == {"11796480"}

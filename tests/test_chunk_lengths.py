"""The chunk lengths that a launch chooses among: the same lengths, in the same order,
as a loop over every number of chunks, in about the square root of its steps."""

import os
import subprocess

from conftest import ROOT

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "chunks.hpp"
int main() {
  for (int planes = 0; planes <= 3000; ++planes)
    for (int least : {1, 2, 4}) {
      std::vector<int> want, got;
      for (int n = 1; n <= planes; ++n) {
        const int t = (planes + n - 1) / n;
        if (t < least) break;
        if (want.empty() || want.back() != t) want.push_back(t);
      }
      aarmr::for_chunk_lengths(planes, least, [&](int t) { got.push_back(t); });
      if (got != want || (long)got.size() * (long)got.size() > 4L * planes) return std::printf("%d %d\n", planes, least), 1;
    }
  return 0;
}
"""


def test_chunk_lengths_match_a_loop_over_every_count(tmp_path):
    src, exe = tmp_path / "chunks.cpp", tmp_path / "chunks"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2205_00385_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout

"""The order in which workgroups take the groups of a tree (csrc/tree_pairs.hpp), on the CPU: every group
of all problems exactly once, and fewer than one round of workgroups without one in the whole launch."""
import os
import shutil
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2212_11744_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "tree_pairs.hpp"
int main() {
  for (int run : {1, 2, 3, 8, 32, 64})
    for (long groups : {1L, 2L, 7L, 8L, 9L, 63L, 64L, 65L, 255L, 256L, 500L, 511L, 512L, 513L, 1024L, 4097L}) {
      const lqt::tile::SpreadGrid g(groups, run);
      std::vector<int> seen(g.grid, 0);
      for (unsigned w = 0; w < g.grid; ++w) {
        const long i = g.run > 1 ? lqt::tile::spread(w, g.run) : (long)w;
        if (i < 0 || i >= (long)g.grid || seen[i]++) return printf("run %d groups %ld w %u\n", run, groups, w), 1;
      }
      const long idle = (long)g.grid - groups;
      if (idle < 0 || idle >= 8L * run || (groups < 8L * run && idle > 0))
        return printf("run %d groups %ld grid %u\n", run, groups, g.grid), 1;
    }
  return 0;
}
"""


def test_every_group_once_and_few_idle_workgroups(tmp_path):
    (tmp_path / "spread.cpp").write_text(PROGRAM)
    subprocess.run([shutil.which("g++"), "-std=c++17", "-I", CSRC, str(tmp_path / "spread.cpp"), "-o",
                    str(tmp_path / "spread")], check=True)
    r = subprocess.run([str(tmp_path / "spread")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout

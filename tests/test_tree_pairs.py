"""The pairing rule of the tree kernels (csrc/tree_pairs.hpp), on the CPU: in every round of every
group size no wave reads a place that another wave writes, the pairs of a round are those of the
reduction, and the places read exist (also by waves without a pair, in the sweep down)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2212_11744_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "tree_pairs.hpp"
int main() {
  for (int nodes : {1, 4})
    for (int waves : {4, 8})
      for (int cnt = 2; cnt <= nodes * waves; ++cnt)
        for (int s = 1; s < cnt; s *= 2)
          for (int w = 0; w < waves; ++w)
            for (int n = 0; n < nodes; ++n) {
              const auto p = lqt::tile::pair_places(w, n, nodes, s, cnt);
              printf("%d %d %d %d %d %d %d %d %d\n", nodes, waves, cnt, s, w, n, p.r, p.any, p.on);
            }
}
"""


@pytest.fixture(scope="module")
def rounds(tmp_path_factory):
    cxx = shutil.which("g++")
    assert cxx, "g++ builds the oracle, too"
    d = tmp_path_factory.mktemp("pairs")
    (d / "pairs.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(d / "pairs.cpp"), "-o", str(d / "pairs")],
                   check=True)
    out = {}
    for line in subprocess.run([str(d / "pairs")], capture_output=True, text=True,
                               check=True).stdout.splitlines():
        nodes, waves, cnt, s, *rest = (int(x) for x in line.split())
        out.setdefault((nodes, waves, cnt, s), []).append(rest)
    return out


def test_no_wave_reads_what_another_writes(rounds):
    for (nodes, waves, cnt, s), lanes in rounds.items():
        writer = {r: w for w, n, r, any_, on in lanes if on}
        for w, n, r, any_, on in lanes:
            if not any_:
                continue  # the wave leaves the round
            for place in (r, r + s):
                assert writer.get(place, w) == w, (nodes, waves, cnt, s, w, n, place)


def test_pairs_of_a_round(rounds):
    for (nodes, waves, cnt, s), lanes in rounds.items():
        want = {r for r in range(0, cnt, 2 * s) if r + s < cnt}
        got = [r for w, n, r, any_, on in lanes if on]
        assert sorted(got) == sorted(want), (nodes, waves, cnt, s)
        for w, n, r, any_, on in lanes:
            assert 0 <= r and r + s < cnt, (nodes, waves, cnt, s, w, n)
            assert any_ == any(o for w2, n2, r2, a2, o in lanes if w2 == w)

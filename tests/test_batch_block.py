"""The blocks that a batch's steps are divided into (csrc/batch_block.hpp, host
arithmetic): whole captured blocks across budget ends where every launch takes
one step, none across them where launches take several."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1404_2363_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "batch_block.hpp"

// argument lines: steps, graph, span, budgets ... -1
int main() {
  long n, graph, span, b;
  while (std::scanf("%ld %ld %ld", &n, &graph, &span) == 3) {
    std::vector<long> ends;
    while (std::scanf("%ld", &b) == 1 && b >= 0) ends.push_back(b);
    for (long t = 0; t < n;) {
      const long blk = (long)lbm::batch_block(n - t, graph, span, [&](int64_t s) {
        int64_t end = INT64_MAX;
        for (long e : ends)
          if (e > t + s && e - t < end) end = e - t;
        return end;
      });
      if (blk < 1) return 1;
      std::printf("%ld ", blk);
      t += blk;
    }
    std::printf("\n");
  }
}
"""


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("batch_block")
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t")],
                   check=True, capture_output=True, text=True)

    def run(n, graph, span, budgets):
        text = " ".join(map(str, [n, graph, span] + list(budgets) + [-1]))
        out = subprocess.run([str(d / "t")], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        return [int(v) for v in out.split()]
    return run


def test_one_step_batches_keep_whole_blocks(blocks):
    assert blocks(100, 32, 0, [7, 11, 40, 41, 99]) == [32, 32, 32, 4]


def test_multi_step_blocks_stop_at_budget_ends(blocks):
    assert blocks(96, 48, 3, []) == [48, 48]
    assert blocks(100, 48, 3, [20]) == [20, 48, 32]
    assert blocks(100, 48, 3, [20, 21, 23, 60]) == [20, 3, 37, 40]      # 20 .. 23 one step at a time, joined
    assert blocks(64, 32, 8, [5, 10, 14, 64]) == [14, 32, 18]
    assert blocks(40, 32, 8, [36]) == [32, 8]                           # too short for the call's last piece


def test_any_budgets(blocks):
    import random
    rng = random.Random(3)
    for _ in range(200):
        n, span = rng.randint(1, 300), rng.choice([0, 3, 8, 10])
        graph = 48 if span == 3 else 32
        budgets = [rng.randint(0, 320) for _ in range(rng.randint(0, 12))]
        got, t = blocks(n, graph, span, budgets), 0
        assert sum(got) == n and max(got) <= graph
        for blk in got:
            inside = [b for b in budgets if t < b < t + blk]
            if inside and span:  # one step at a time: no budget-free stretch long enough is in there
                cuts = [t] + sorted(inside) + [t + blk]
                assert all(b - a < span for a, b in zip(cuts, cuts[1:]))
            t += blk

"""bench.py times and checks whole captured graphs: its block length is a
multiple of every graph length of the library."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_blocks_hold_whole_graphs():
    sys.path.insert(0, ROOT)
    import bench
    src = open(os.path.join(ROOT, "paper_1404_2363_amd", "csrc", "lbm_cde.hip")).read()
    lengths = [int(v) for v in re.findall(r"constexpr int kGraph(?:Steps|Strip) = (\d+);", src)]
    assert len(lengths) == 2
    for n in lengths:
        assert bench.GRAPH_STEPS % n == 0

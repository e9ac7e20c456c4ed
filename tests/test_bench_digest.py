"""The digest that ties the committed HBM counters to the pair kernels covers every source they are built from."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_1707_02423_amd", "csrc")


def test_the_digest_covers_what_the_pair_kernels_include():
    todo, seen = ["pair.hip", "pair_plain_f32.hip", "pair_plain_f64.hip"], set()
    while todo:
        name = todo.pop()
        if name not in seen:
            seen.add(name)
            with open(os.path.join(CSRC, name)) as f:
                todo += [x for x in re.findall(r'#include "([^"]+)"', f.read()) if "/" not in x]
    assert seen == set(bench.PAIR_SOURCES)


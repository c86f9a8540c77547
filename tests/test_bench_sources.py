"""The sources that the stored counter readings depend on."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_2403_06654_amd", "csrc")


def test_the_counter_hash_covers_every_header_of_the_kernels():
    """bench.py uses stored counter readings only while the sources of the 3D
    solves' kernels are unchanged: the passes, the vector kernels and all headers
    of this library that they include."""
    want, todo = set(), ["passes.hip", "vecops.hip"]
    while todo:
        fn = todo.pop()
        if fn in want:
            continue
        want.add(fn)
        text = open(os.path.join(CSRC, fn)).read()
        todo += [h for h in re.findall(r'#include "([^"/]+)"', text) if os.path.exists(os.path.join(CSRC, h))]
    assert want <= set(bench.KERNEL_SOURCES_3D), want - set(bench.KERNEL_SOURCES_3D)

"""The counter summaries that bench.py reports are tied to the kernel's sources:
to the file it is in and every file of the library that one includes."""

import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_2009_12009_amd", "csrc")


def test_hash_covers_every_included_file():
    seen, todo = set(), ["flat_kernels.hip"]
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        todo += re.findall(r'^#include "([^"]+)"', open(os.path.join(CSRC, f)).read(), flags=re.M)
    assert seen == set(bench.KERNEL_SOURCES)

"""The tracked HBM traffic of the attention kernel counts as stale when any source compiled into it has changed: bench.py's list
of those sources holds everything that the attention translation units include."""
import os
import re

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_01204_amd", "csrc")


def test_every_included_source_is_listed():
    seen, todo = set(), ["attn.hip", "attn16.hip"]
    while todo:
        name = todo.pop()
        if name not in seen:
            seen.add(name)
            with open(os.path.join(CSRC, name)) as f:
                todo += re.findall(r'^#include "([^"]+)"', f.read(), re.M)
    assert seen == set(bench.KERNEL_SOURCES)

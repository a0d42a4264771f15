"""The hash beside the recorded HBM traffic covers every source of the kernels
that the record names."""
import os
import re

import bench

PKG = os.path.join(bench.ROOT, "paper_0904_4152_amd")


def test_every_included_header_is_hashed():
    seen, todo = set(), ["csrc/kernels.hip", "csrc/blas1.hip", "csrc/band4.hip"]
    while todo:
        name = todo.pop()
        path = os.path.join(PKG, name)
        if name in seen or not os.path.exists(path):  # the ABI's header lies elsewhere
            continue
        seen.add(name)
        with open(path) as f:
            todo += ["csrc/" + h for h in re.findall(r'#include "([^"]+)"', f.read())]
    assert "csrc/mid_ops.h" in seen
    assert seen <= set(bench.TRAFFIC_SOURCES)

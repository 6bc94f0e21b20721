"""bench.py reports recorded counter traffic only while the sources of the fine-apply kernel are those
the counters were taken with: every header with device code that k_apply.hip includes is among them."""

import os
import re

import bench

# declarations only: launch functions, configuration, kernel arguments
DECLARATIONS = {"internal.h", "agca.h"}


def test_kernel_sources_hold_every_header():
    csrc = os.path.dirname(bench.KERNEL_SOURCES[0])
    seen, todo = set(), ["k_apply.hip"]
    while todo:
        name = todo.pop()
        if name in seen or name in DECLARATIONS:
            continue
        seen.add(name)
        with open(os.path.join(bench.ROOT, csrc, name)) as fh:
            todo += re.findall(r'^\s*#include "([^"]+)"', fh.read(), re.M)
    assert seen == {os.path.basename(p) for p in bench.KERNEL_SOURCES}

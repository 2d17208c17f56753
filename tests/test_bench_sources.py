"""The benchmark's counted traffic is keyed by the kernel's sources: by every header that
holds a part of the row kernel."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_1509_04394_amd", "csrc")


def test_traffic_key_covers_the_kernel_headers():
    todo, seen = ["rowfuse.h"], set()
    while todo:
        f = todo.pop()
        if f not in seen and os.path.exists(os.path.join(CSRC, f)):
            seen.add(f)
            todo += re.findall(r'#include "([\w.]+)"', open(os.path.join(CSRC, f)).read())
    # the operation registry and the launch tables' helpers hold no code of the kernel
    assert seen - {"fz_ops.h"} == set(bench.KERNEL_SOURCES)

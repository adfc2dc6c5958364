"""bench.py reports the real push's counted HBM bytes only while the sources
hash to what they were when the counters were taken: every file the kernel is
compiled from has to be among them."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_2109_10277_amd", "csrc")


def included(name, seen):
    if name in seen:
        return seen
    seen.add(name)
    with open(os.path.join(CSRC, name)) as f:
        for inc in re.findall(r'^#include "([^"/]+)"', f.read(), re.M):
            included(inc, seen)
    return seen


def test_every_source_of_the_real_push_is_hashed():
    needed = included("particles.hip", set()) | {"runtime.cpp"}   # which picks the tiles
    hashed = {os.path.basename(f) for f in bench.PUSH_SOURCES}
    assert needed <= hashed, sorted(needed - hashed)

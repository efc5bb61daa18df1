"""CPU: the bench's list of the dominant kernel's sources holds every header that its translation unit includes
(the hash of these sources tells whether committed counters still belong to the kernel)."""
import os
import re

import bench
from conftest import ROOT


def test_every_included_header_is_listed():
    todo, seen = [os.path.join(ROOT, bench.KERNEL_SOURCES[0])], set()
    while todo:
        f = os.path.normpath(todo.pop())
        if f in seen:
            continue
        seen.add(f)
        todo += [os.path.join(os.path.dirname(f), h) for h in re.findall(r'^#include "([^"]+)"', open(f).read(), re.M)]
    assert {os.path.relpath(f, ROOT) for f in seen} == set(bench.KERNEL_SOURCES)

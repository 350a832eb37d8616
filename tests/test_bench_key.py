"""The key that ties the benchmark's counter records to the kernel they were taken on covers
every file of the kernel's own: the source and, through all of them, the headers it includes."""
import os
import re

import bench


def test_key_covers_the_kernel_sources():
    folder = os.path.dirname(bench.KERNEL_SOURCES[0])
    todo, seen = ["transport.hip"], set()
    while todo:
        name = todo.pop()
        seen.add(name)
        text = open(os.path.join(folder, name)).read()
        todo += [h for h in re.findall(r'#include "([^"]+)"', text) if h not in seen]
    assert sorted(seen) == sorted(os.path.basename(f) for f in bench.KERNEL_SOURCES)

"""The sources that bench.py hashes for each kernel, by which a committed profile
is recognised as one of the current kernel, are the kernel's file and everything
it includes."""
import os
import re

import pytest

bench = pytest.importorskip("bench")
CSRC = os.path.join(bench.ROOT, bench._CSRC)


def included(name, seen):
    seen.add(name)
    with open(os.path.join(CSRC, name)) as f:
        for inc in re.findall(r'^#include "([^"]+)"', f.read(), re.M):
            if inc not in seen and os.path.exists(os.path.join(CSRC, inc)):
                included(inc, seen)
    return seen


@pytest.mark.parametrize("kernel", sorted(bench.KERNEL_SOURCES))
def test_hashed_sources_are_the_include_closure(kernel):
    listed = [os.path.relpath(os.path.join(bench.ROOT, p), CSRC) for p in bench.KERNEL_SOURCES[kernel]]
    assert sorted(listed) == sorted(included(listed[0], set()))

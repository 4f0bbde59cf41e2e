"""The sources whose hash ties a committed counter record to a kernel: the
kernel's own file and every header of the library that it includes, so that a
change of any of them makes the record stale.  Host only."""
import os
import re

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_2511_05222_amd", "csrc")


def headers(name, seen):
    for h in re.findall(r'#include "(vmc_\w+\.hpp)"', open(os.path.join(CSRC, name)).read()):
        if h not in seen:
            seen.add(h)
            headers(h, seen)
    return seen


@pytest.mark.parametrize("kernel", sorted(bench.KERNEL_SRCS))
def test_hash_covers_includes(kernel):
    src = bench.KERNEL_SRCS[kernel]
    need = set()
    for f in src:
        if f.endswith(".hip"):
            headers(f, need)
    assert need <= set(src), sorted(need - set(src))

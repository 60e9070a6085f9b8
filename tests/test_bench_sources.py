"""The device sources whose hash decides whether bench.py takes a committed counter
summary for the code as it is: every file that the profiled kernels include is among
them (but for headers that hold argument layouts only)."""
import os
import re

import pytest

import bench
from test_kernel_isa import CSRC

LAYOUTS = {"kernels.hpp", "coexec.h"}


def included(src, seen=None):
    seen = set() if seen is None else seen
    if src in seen:
        return seen
    seen.add(src)
    with open(os.path.join(CSRC, src)) as f:
        for name in re.findall(r'^#include "(?:\.\./\.\./include/)?([\w.]+)"', f.read(), flags=re.M):
            if name not in LAYOUTS:
                included(name, seen)
    return seen


@pytest.mark.parametrize("kernels,sources", [("kernels.hip", bench.DEVICE_SOURCES),
                                             ("binomial_call.hip", bench.DEVICE_SOURCES),
                                             ("batch_kernels.hip", bench.BATCH_SOURCES)])
def test_counter_summaries_are_bound_to_every_device_source(kernels, sources):
    have = {os.path.basename(s) for s in sources}
    assert included(kernels) <= have, included(kernels) - have
    assert all(os.path.exists(os.path.join(bench.ROOT, s)) for s in sources)

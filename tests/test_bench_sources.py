"""bench.py takes a kernel class's measured traffic from a counter summary only
while the class's sources are those it was taken with: the list of sources has
to name every file that the class's kernels are built from."""
import glob
import os
import re

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_2609_33874_amd", "csrc")
KERNELS = {"gemm": "k_gemm*.hip", "lmhead": "k_gemm.hip", "attn": "k_attn*.hip", "gdn": "k_gdn.hip"}


def includes(name, seen):
    if name in seen:
        return seen
    seen.add(name)
    with open(os.path.join(CSRC, name)) as f:
        for inc in re.findall(r'^#include "([^"]+)"', f.read(), re.M):
            if inc != "kernels.h":  # declarations of the launchers
                includes(inc, seen)
    return seen


@pytest.mark.parametrize("cls", list(KERNELS))
def test_sources_of_a_class_are_complete(cls):
    files = set()
    for f in glob.glob(os.path.join(CSRC, KERNELS[cls])):
        includes(os.path.basename(f), files)
    assert set(bench.KERNEL_SOURCES[cls]) == files

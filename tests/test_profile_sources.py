"""The committed kernel traces of the batched, adjoint and extensions legs were taken
on the committed sources of all kernels, and the cache counters on the step's."""
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def _hash_in(name, key):
    with open(os.path.join(ROOT, "profiles", name)) as f:
        return re.search(rf"^{key}: (\w+)$", f.read(), re.M).group(1)


@pytest.mark.parametrize("name", ["batched_adjoint_legs_kernel_stats.md",
                                  "extensions_c3_1M_kernel_stats.md"])
def test_traces_of_the_legs(name):
    csrc = os.path.join(ROOT, "paper_2008_11578_amd", "csrc")
    files = sorted(f for f in os.listdir(csrc) if f.endswith((".hip", ".h")))
    assert _hash_in(name, "all_kernels_source_hash") == bench.source_hash(files)


def test_cache_counters_of_the_step():
    assert _hash_in("k_step_c3_1M_cache.md", "source_hash") == bench.source_hash()

"""The source lists that decide whether committed counters are those of the current kernels: every list holds what its
files include, and the FFT list every file of the FFT kernels.  No GPU work."""

import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

CSRC = os.path.join(ROOT, "paper_1509_04685_amd", "csrc")
DECLARATIONS = {"cola_internal.h", "lc_internal.h"}


@pytest.mark.parametrize("kind", sorted(bench.KERNEL_SOURCES))
def test_lists_hold_their_includes(kind):
    files = bench.KERNEL_SOURCES[kind]
    assert len(set(files)) == len(files)
    for name in files:
        with open(os.path.join(CSRC, name)) as fh:
            local = set(re.findall(r'#include "([^"]+)"', fh.read()))
        missing = {h for h in local - DECLARATIONS if os.path.exists(os.path.join(CSRC, h))} - set(files)
        assert not missing, (kind, name, missing)


def test_fft_list_holds_every_fft_file():
    there = {f for f in os.listdir(CSRC) if f.startswith("fft")}
    assert there <= set(bench.KERNEL_SOURCES["fft"])


def test_every_kind_with_counters_has_a_list():
    for name in os.listdir(os.path.join(ROOT, "profiles")):
        m = re.match(r"(.+)_\d+_counters\.txt$", name)
        if m:
            assert bench.source_hash(m.group(1)) is not None

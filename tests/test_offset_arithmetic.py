"""Chunk offsets from damaged sizes.  tests/pins/offsets_check.cpp runs the
arithmetic of csrc/offsets.hpp, which the decompression kernels use, over
batches whose size words are damaged: no accepted chunk lies outside its own
payload, and damage in one series changes nothing for the series beside it.
The same with sums that wrap shows that the cases reach both faults."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def counts(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("offsets") / "offsets_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", os.path.join(HERE, "pins", "offsets_check.cpp"), "-o", out],
                   check=True)

    def run(*args):
        f = subprocess.run([out, *args], capture_output=True, text=True, check=True).stdout.split()
        return dict(zip(f[::2], map(int, f[1::2])))
    return run


def test_damaged_sizes_stay_inside_their_series(counts):
    r = counts()
    assert r["chunks"] > 100_000
    assert (r["accepted-outside"], r["wrong-neighbours"], r["missed"]) == (0, 0, 0)


def test_the_cases_reach_the_faults(counts):
    r = counts("wrapping")
    assert r["accepted-outside"] >= 3 and r["wrong-neighbours"] > 0

"""The boxes of test_gpu_sweep_pairs.py are ones whose FP32 sweeps go two in a
launch (otherwise that test compares single sweeps with themselves), and boxes
well inside and outside that rule are on its right side.  Host side, no GPU."""
import ctypes
import os

import pytest

import test_gpu_sweep_pairs as G


@pytest.fixture(scope="module")
def paired():
    from paper_1910_12979_amd import build, macproj
    if not os.path.exists(macproj.LIB_PATH):
        build.build()
    f = macproj.lib()["_ZN2mg12sweep_pairedEiii"]          # bool mg::sweep_paired(int, int, int)
    f.argtypes = [ctypes.c_int] * 3
    f.restype = ctypes.c_bool
    return f


def test_the_gpu_tests_boxes_are_paired(paired):
    marks = [m for m in G.test_pairs_are_two_sweeps.pytestmark if m.name == "parametrize"]
    cases = marks[0].args[1]
    assert len(cases) >= 3
    for n, _, _ in cases:
        assert paired(*n), n


@pytest.mark.parametrize("n,want", [((256, 256, 256), True), ((512, 512, 512), True), ((512, 512, 256), True),
                                    ((288, 288, 288), False), ((128, 128, 128), False), ((64, 64, 64), False),
                                    ((16, 512, 512), False)])
def test_rule(paired, n, want):
    assert paired(*n) == want


def test_forced_tiles_are_not_paired(paired):
    from paper_1910_12979_amd import macproj
    macproj.mg_tune_sweep(9)
    try:
        assert not paired(256, 256, 256)
    finally:
        macproj.mg_tune_sweep(-1)

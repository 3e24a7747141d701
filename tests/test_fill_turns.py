"""Workgroups that clear memory among those that unstuff (pcr_common.h: fill_turn, compiled for the CPU): every share is
taken once, each of the eight dies (workgroup index mod 8) gets the same number of filling ones, and they are spread over the
launch from end to end."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def turns(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("turns") / "libturns.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-o", so, os.path.join(HERE, "host_emul", "fill_turns.cpp")])
    lib = ctypes.CDLL(so)

    def run(others, groups):
        out = np.zeros(others + groups + 8, np.int32)
        return out[:lib.fill_turns(others, groups, out.ctypes.data_as(ctypes.POINTER(ctypes.c_int)))]
    return run


@pytest.mark.parametrize("groups", [0, 1, 7, 8, 9, 500, 1024, 2048])
@pytest.mark.parametrize("others", [0, 1, 5, 8, 17, 250, 1000, 1024, 2047, 2560, 3333, 4096, 5120, 8192, 10240])
def test_shares_dies_and_spread(turns, others, groups):
    out = turns(others, groups)
    fills = np.flatnonzero(out < 0)
    rows = -(-groups // 8)
    assert len(out) == others + 8 * rows and len(fills) == 8 * rows
    assert np.array_equal(np.sort(-1 - out[fills]), np.arange(8 * rows))
    assert np.array_equal(out[out >= 0], np.arange(others))
    assert (np.bincount(fills % 8, minlength=8) == rows).all()
    if rows:                                                  # from one filling row to the next the same distance, and none of that length left at the end
        starts = fills.reshape(rows, 8)[:, 0]
        period = len(out) // 8 // rows
        assert (starts % 8 == 0).all() and (np.diff(starts) == 8 * period).all() and starts[0] == 8 * (period - 1)
        assert len(out) - starts[-1] - 8 < 8 * (rows + 1)

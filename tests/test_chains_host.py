"""Which scans one launch decodes side by side (pcr_chains.h, compiled for the CPU): two scans of a component whose bands
overlap are never decoded at the same time, unless the later one is a refinement scan of the same chain that waits for the
earlier one -- the symbol loops of first scans wait for nothing."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("chains") / "libchains.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-o", so, os.path.join(HERE, "host_emul", "chains.cpp")])
    lib = ctypes.CDLL(so)

    def run(scans, k0=0, k=None):
        a = np.ascontiguousarray(scans, np.int32).reshape(-1, 8)
        out = np.zeros((len(a), 4), np.int32)
        step = lib.chain_plan(a.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), len(a), k0, len(a) if k is None else k, out.ctypes.data_as(ctypes.POINTER(ctypes.c_int)))
        return bool(step), out
    return run


def _scan(comps, Ss, Se, Ah, Al, ri=0, units=1, entries=0):
    return (comps, Ss, Se, Ah, Al, ri, units, entries)


def _check(scans, out, k0, k):
    for g in range(k0, k):
        for q in range(k0, g):
            a, b = scans[q], scans[g]
            if not (a[0] & b[0]) or a[1] > b[2] or b[1] > a[2] or out[g][0] < 0 or out[q][0] < 0:
                continue
            if out[g][0] != out[q][0]:
                assert out[q][0] < out[g][0], ("the later launch has the earlier scan", q, g)
                continue
            assert out[g][0] == 0 and out[g][1] == out[q][1], ("decoded at the same time", q, g)
            assert b[3] > 0 and b[1] > 0, ("a scan that waits for nothing follows another", q, g)
            assert out[q][2] < out[g][2] and out[g][3] >> out[q][2] & 1, ("does not wait", q, g)


DC, LUMA = _scan(1, 0, 0, 0, 0), [_scan(1, 1, 5, 0, 2), _scan(1, 6, 63, 0, 2), _scan(1, 1, 63, 2, 1), _scan(1, 1, 63, 1, 0)]
FILES = {
    "usual": ([DC] + LUMA, True),
    "interleaved": ([_scan(7, 0, 0, 0, 1), _scan(1, 1, 5, 0, 2), _scan(4, 1, 63, 0, 1), _scan(2, 1, 63, 0, 1), _scan(1, 6, 63, 0, 2), _scan(1, 1, 63, 2, 1),
                     _scan(7, 0, 0, 1, 0), _scan(4, 1, 63, 1, 0), _scan(2, 1, 63, 1, 0), _scan(1, 1, 63, 1, 0)], True),
    "ac first twice": ([DC, _scan(1, 1, 63, 0, 1), _scan(1, 1, 63, 0, 0)], False),
    "ac first over a part": ([DC, _scan(1, 1, 20, 0, 1), _scan(1, 10, 63, 0, 1), _scan(1, 1, 63, 1, 0)], False),
    "ac first after a refinement": ([DC, _scan(1, 1, 63, 0, 2), _scan(1, 1, 63, 2, 1), _scan(1, 1, 20, 0, 1)], False),
    "dc first twice": ([_scan(1, 0, 0, 0, 1), _scan(1, 0, 0, 0, 0)] + LUMA, False),
    "dc first of all, then of one": ([_scan(7, 0, 0, 0, 1), _scan(2, 0, 0, 0, 0), _scan(2, 1, 63, 0, 0)], False),
}


@pytest.mark.parametrize("restart", [0, 3])
@pytest.mark.parametrize("name", sorted(FILES))
def test_scans_that_overlap_are_ordered(plan, name, restart):
    scans, step = FILES[name]
    scans = [s[:5] + (restart, 4 if restart else 1, 0) for s in scans]
    assert plan(scans)[0] == step
    for k0 in range(len(scans)):
        for k in range(k0 + 1, len(scans) + 1):
            _check(scans, plan(scans, k0, k)[1], k0, k)


def test_any_sequence_of_scans_is_ordered(plan):
    """Random scans, most of which no encoder would write."""
    rng = random.Random(4)
    for _ in range(3000):
        scans = []
        for _ in range(rng.randint(1, 12)):
            ah = rng.choice([0, 0, 1])
            if rng.random() < 0.3:
                scans.append(_scan(rng.choice([1, 2, 4, 7]), 0, 0, ah, 0))
            else:
                a, b = sorted((rng.randint(1, 63), rng.randint(1, 63)))
                scans.append(_scan(rng.choice([1, 2, 4]), a, b, ah, 0, rng.choice([0, 0, 0, 5]), rng.choice([1, 1, 1, 3]), rng.choice([0, 0, 0, 64])))
        k0 = rng.randrange(len(scans))
        k = rng.randint(k0 + 1, len(scans))
        _check(scans, plan(scans, k0, k)[1], k0, k)

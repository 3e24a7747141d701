"""The walks of scans decoded by many lanes each (pcr_first_split.h, pcr_sequential.h, compiled for the CPU) on look-ups no code has made,
entries of no bits among them: every trip moves on by a bit at least, so that they end whatever the tables hold."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_walks_end_whatever_the_tables_hold(tmp_path):
    exe = str(tmp_path / "walks")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-w", "-o", exe, os.path.join(HERE, "host_emul", "split_walks.cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60, check=True).stdout
    lines = out.splitlines()
    assert lines[-1] == "walks end" and len(lines) == 31
    for line in lines[:-1]:                                   # a symbol takes 46 bits at most (a length of five bits, fifteen more)
        _, _, _, ac, _, dc, _, whole = line.split()
        assert all(0 <= int(v) < 46 for v in (ac, dc, whole)), line

"""Host calls that use several threads, where the system has no more to give: they go on with those there are."""
import os
import resource
import subprocess
import sys

import pytest

import pcrgen

PROGRAM = r"""
import resource, sys
sys.path[:0] = [%(root)r]
import paper_1911_00472_amd as pkg
files = [open(p, "rb").read() for p in sys.argv[1:]]
want = pkg.record_write_indexed(files, None, 16)
size = 4096 * int(open("/proc/self/statm").read().split()[0])
resource.setrlimit(resource.RLIMIT_AS, (size + (24 << 20), size + (24 << 20)))
import threading
try:
    t = threading.Thread(target=int); t.start(); t.join()
    print("a thread could be started")
except RuntimeError:
    print("no more threads")
assert pkg.record_write_indexed(files, None, 16) == want
print("the same record")
"""


def test_record_writer_without_more_threads(tmp_path):
    paths = []
    for i in range(6):
        paths.append(str(tmp_path / ("%d.jpg" % i)))
        open(paths[-1], "wb").write(pcrgen.make_jpeg(i, 1, 90, 60 + i, 3, 6.0, 2, 2, 90))
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", PROGRAM % dict(root=root)] + paths, capture_output=True, text=True, timeout=120,
                       preexec_fn=lambda: resource.setrlimit(resource.RLIMIT_STACK, (64 << 20, 64 << 20)))      # (what a new thread's stack takes)
    if "a thread could be started" in r.stdout:
        pytest.skip("the limit on address space does not keep threads from starting here")
    assert r.returncode == 0 and "the same record" in r.stdout, (r.returncode, r.stdout, r.stderr[-800:])

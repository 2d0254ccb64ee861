"""A C entry whose host memory runs out returns a status: no exception leaves
it (which would end the caller's process)."""
import os
import subprocess
import sys

import pytest

from conftest import ROOT

CHILD = r'''
import ctypes, resource, sys
import numpy as np
from paper_1401_7457_amd import cxbwt
L = cxbwt.lib()
n = 60_000_000  # collections of one read: their boundaries are copied, half a gigabyte
bounds = np.arange(n + 1, dtype=np.uint64)
fake, null = ctypes.c_void_p(0x1000), ctypes.c_void_p(0)
with open("/proc/self/statm") as f:
    now = int(f.read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (now + (64 << 20), now + (64 << 20)))
p = bounds.ctypes.data_as(ctypes.c_void_p)
h = ctypes.c_void_p()
if sys.argv[1] == "batch":
    rc = L.cxbwt_build_batch(fake, fake, n, 0, 10, p, n, fake, fake, fake, 1 << 60, None, null)
elif sys.argv[1] == "start":
    rc = L.cxbwt_build_batch_start(fake, fake, n, 0, 10, p, n, fake, fake, fake, 1 << 60, None, null, ctypes.byref(h))
print("rc", rc, "job", h.value, L.cxbwt_last_error().decode(), flush=True)
'''


@pytest.mark.parametrize("entry", ["batch", "start"])
def test_no_exception_leaves_a_c_entry(entry):
    r = subprocess.run([sys.executable, "-c", CHILD, entry], cwd=ROOT, capture_output=True, text=True, timeout=300,
                       env={**os.environ, "PYTHONPATH": ROOT})
    assert r.returncode == 0, r.stderr[-2000:]
    assert "rc -4 job None out of host memory" in r.stdout, r.stdout

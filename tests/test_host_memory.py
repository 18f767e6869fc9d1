"""Running out of host memory inside a call is a status, not a C++ exception
across the C interface (which would end the process)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import ctypes as C, resource, sys
import numpy as np
sys.path.insert(0, {root!r})
from paper_1705_02028_amd import inputs as I, rd
L = rd.lib()
n = 3000
m = I.split_square(n, periodic=(False, False), bc=("ghost", "ghost"))
nv, nt = C.c_int64(m["nv"]), C.c_int64(m["nt"])
tri = np.ascontiguousarray(m["tri"], np.int32)
x, y = np.ascontiguousarray(m["x"]), np.ascontiguousarray(m["y"])
del m
p = lambda a: a.ctypes.data_as(C.c_void_p)
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (64 << 20), resource.RLIM_INFINITY))
if {call!r} == "flip":
    st = L.rd_delaunay_flip(nv.value, p(x), p(y), 0.0, 0.0, nt.value, p(tri), None, None)
else:
    st = L.rd_delaunay_refine(C.byref(nv), p(x), p(y), nv.value, 0.0, 0.0, C.byref(nt), p(tri), nt.value,
                              0.1, 0.0, None, 0, 0, 1, 0, None, None)
print("status", st, rd.rd_last_error())
assert st == rd.RD_ENOMEM
"""


@pytest.mark.parametrize("call", ["flip", "refine"])
def test_mesh_generation_reports_host_memory(call):
    r = subprocess.run([sys.executable, "-c", PROGRAM.format(root=ROOT, call=call)], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-500:])

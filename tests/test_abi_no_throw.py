"""Nothing throws across the C ABI: where the host's memory runs out, a call
says so.  The planner of a large batch, in a process whose address space is
limited once the library and the description are in it."""
import subprocess
import sys

CODE = r"""
import ctypes as C, resource
import numpy as np
from paper_2505_05940_amd import modal
B = 1 << 20
arr = (modal.modal_instance * B)()
v = [np.full(1, x) for x in (1000.0, 3.0, 1e-3, 1e-3, 1.0, 1.0)]
one = modal.modal_instance(kind=1, n_t=1)
for name, a in zip(("omega", "gamma", "x0", "xm1", "c_out"), v):
    setattr(one, name, a.ctypes.data_as(C.POINTER(C.c_double)))
setattr(one, "lam", v[5].ctypes.data_as(C.POINTER(C.c_double)))
size = C.sizeof(modal.modal_instance)
for i in range(0, B * size, size):
    C.memmove(C.addressof(arr) + i, C.addressof(one), size)
desc = modal.modal_desc(batch=B, scheme=0, inst=arr, fs=44100.0)
out = (C.c_int64 * 4)()
print("plan", modal.lib.modal_plan(C.byref(desc), 64, out), flush=True)
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (4 << 20), resource.getrlimit(resource.RLIMIT_AS)[1]))
code = modal.lib.modal_plan(C.byref(desc), 64, out)
print("limited", modal.STATUS[code], flush=True)
"""


def test_planner_without_memory():
    r = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-2000:])
    assert r.stdout.split("\n")[:2] == ["plan 0", "limited ENOMEM"], r.stdout

"""Planning calls that run out of memory: G10_ENOMEM, and nothing is left behind.  The library's host code runs in a
process of its own against tests/native/no_device.cpp in place of the HIP runtime (no GPU, kernels do not run)."""
import os
import subprocess
import sys

from paper_2310_09443_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes as C, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)                 # before the library: its calls resolve to these
from paper_2310_09443_amd import binding as B
lib = C.CDLL(B.LIB_PATH)
for f in ("test_made", "test_blocks", "test_arrays"):
    getattr(shim, f).restype = C.c_long
K = 600
host = {n: (t * K)(*([1] * K)) for n, t in (("dur", C.c_uint64), ("size", C.c_uint64), ("glob", C.c_uint8))}
a = {n: C.addressof(x) for n, x in host.items()}
trace = B._Trace(K, K, 0, a["dur"], a["size"], a["glob"], None, None, 0)
count = 3
params = (B._Params * count)()
for p in params:
    p.gpu_cap_bytes = 1
    for d in range(2):
        p.bw_out_Bpus[d] = p.bw_in_Bpus[d] = 6000
outs = (B._Result * count)()

def call(n, fail_at):
    # the allocations of one planning call of n plans on a new handle, refused from the `fail_at`-th on: (return code, how many were asked for)
    shim.test_fail_at(C.c_long(-1))
    h = C.c_void_p()
    assert lib.g10_vitality(C.byref(trace), None, C.byref(h)) == B.OK
    arrays = shim.test_arrays()
    shim.test_fail_at(C.c_long(fail_at))
    rc = lib.g10_plan(h, params, outs) if n == 1 else lib.g10_plan_batch(h, params, n, outs)
    made = shim.test_made()
    assert shim.test_arrays() == arrays, (n, fail_at, "an array of the call was not freed")
    lib.g10_plan_free(h)
    lib.g10_trim()
    assert shim.test_blocks() == 0, (n, fail_at, "memory of the handle was not given back")
    return rc, made

for n in (1, count):
    rc, asked = call(n, -1)                                    # (no kernel runs, so the plan never ends: the call gives up)
    assert rc == B.EDEVICE and asked >= 3, (rc, asked)
    for i in range(asked):
        assert call(n, i)[0] == B.ENOMEM, i
print("ok")
"""


def test_every_allocation_refused_in_turn(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    shim = str(tmp_path / "no_device.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", os.path.join(ROOT, "tests", "native", "no_device.cpp"), "-o", shim], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, shim], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stderr[-2000:]

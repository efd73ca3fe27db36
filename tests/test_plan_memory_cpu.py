"""Plans when memory runs out, on the CPU: the library's host code over
tests/fake_hip.cpp, each allocation of a plan's creation refused in turn."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import ctypes, sys
import numpy as np
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
ENOMEM = -3
P = ctypes.c_void_p
lib.pgh_last_error.restype = ctypes.c_char_p
lib.pgh_last_error.argtypes = [P]
ctx = P()
assert lib.pgh_open(ctypes.byref(ctx), 0, None) == 0
table = (ctypes.c_float * 2048)()
assert lib.pgh_set_table(ctx, 4, 6, ctypes.c_float(0.1), table) == 0
lists, n_i, n_j = 50, 40, 300
items = np.array([(n_i * k, n_i, n_j * k, n_j) for k in range(lists)], np.int32)
def create():
    p = P()
    st = lib.pgh_plan_create(ctx, lists, items.ctypes.data_as(P), lists * n_i, lists * n_j,
                             ctypes.byref(p))
    return st, p
a = np.zeros(lists * n_j, np.float32).ctypes.data_as(P)
def force(p):
    n = fake.fake_launches()
    st = lib.pgh_batch_table(ctx, p, a, a, a, a, a, a, a, a, a, a, None)
    assert st == 0, (st, lib.pgh_last_error(ctx))
    assert fake.fake_launches() > n
st, p = create()  # the context's own buffers grow
assert st == 0 and lib.pgh_plan_free(ctx, p) == 0
live = fake.fake_live()
fake.fake_refuse(-1)
st, p = create()
n = fake.fake_count()
assert st == 0 and n >= 2
force(p)
assert lib.pgh_plan_free(ctx, p) == 0 and fake.fake_live() == live
got = []
for k in range(n):
    fake.fake_refuse(k)
    st, p = create()
    assert st in (0, ENOMEM) and bool(p) == (st == 0), (k, st)
    fake.fake_refuse(-1)
    if st == 0:
        # without its second task list the plan serves all the same, and the refusal
        # is not left behind for the next launch to report
        assert fake.fake_last() == 0
        force(p)
        assert lib.pgh_plan_free(ctx, p) == 0
    assert fake.fake_live() == live, k
    got.append(st)
assert got == [ENOMEM] * (n - 1) + [0], got
assert lib.pgh_close(ctx) == 0 and fake.fake_live() == 0
print("plan memory checks passed")
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_each_allocation_of_a_plan_refused(tmp_path):
    fake = str(tmp_path / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC",
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", fake],
                   check=True, capture_output=True, text=True, timeout=120)
    lib = os.environ.get("PGH_LIB", os.path.join(ROOT, "paper_1203_4037_amd", "libpgh.so"))
    r = subprocess.run([sys.executable, "-c", PROGRAM, fake, lib], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0 and "plan memory checks passed" in r.stdout, r.stdout + r.stderr

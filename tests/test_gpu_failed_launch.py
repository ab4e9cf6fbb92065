"""A step call that fails while its launches are recorded (the runtime's
error query reports an error once) leaves the state as it was: the next call
gives the bits of a handle that never failed. The error is injected by a
shared object that answers hipGetLastError before the runtime does; it is
loaded in a process of its own, ahead of the library."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
static int armed;
static int (*real)(void);
void shim_set(int (*f)(void)) { real = f; }
void shim_arm(int n) { armed = n; }
int shim_armed(void) { return armed; }
int hipGetLastError(void) {
  int e = real ? real() : 0;
  if (armed > 0 && --armed == 0) return 999;
  return e;
}
"""

CHILD = """
import ctypes as C, sys
import numpy as np
sys.path.insert(0, sys.argv[2])
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
from paper_2006_13631_amd import hlbm as H
from paper_2006_13631_amd.workloads import random_populations
W9 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
H.load()
with open("/proc/self/maps") as f:
    hip = next(l.split()[-1] for l in f if "libamdhip64" in l)
shim.shim_set(C.cast(C.CDLL(hip).hipGetLastError, C.c_void_p))
large = dict(nx=190, ny=141, nux=97, nuy=46, b=30.0, beta=60.0, kc=0.5, tau=0.7)
small = dict(nx=60, ny=61, nux=32, nuy=20, b=8.0, beta=20.0, kc=0.5, tau=0.7)
lev = dict(boxes=[(12, 12, 48, 44)], nux=40, nuy=24, b=10.0, beta=20.0, kc=0.5, tau=0.7)
makes = [("two steps a launch", lambda: H.Case(max_steps=16, **large), 8),
         ("one step a launch", lambda: H.Case(max_steps=16, **small), 8),
         ("levels", lambda: H.MultiLevel(64, 60, max_steps=64, **lev), 2)]
for name, make, n in makes:
    a, b = make(), make()
    g = random_populations((9, a.nnode), 5, W9, spread=0.01)  # step 0's lattice nodes differ from rest
    a.set_grid(g)
    b.set_grid(g)
    assert a.info().two_step == (name == "two steps a launch")
    shim.shim_arm(1)
    try:
        a.step(n)
    except H.HlbmError as e:
        assert e.code == H.E_HIP, e
    else:
        raise SystemExit(name + ": no error")
    assert shim.shim_armed() == 0
    a.step(n)
    b.step(n)
    for x, y in ((a.grid(), b.grid()), (a.lattice(), b.lattice()), (a.history(), b.history())):
        assert np.array_equal(x, y), name
    print(name, "ok", flush=True)
"""


def test_steps_after_a_failed_call(tmp_path):
    src, so, child = tmp_path / "shim.c", tmp_path / "shim.so", tmp_path / "child.py"
    src.write_text(SHIM)
    child.write_text(CHILD)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True, timeout=60)
    r = subprocess.run([sys.executable, str(child), str(so), ROOT], capture_output=True, text=True, timeout=90)
    print(r.stdout, r.stderr)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.count("ok") == 3

"""Saving and loading a subdomain needs no device memory of its own: both still
work where none can be had.  A subprocess puts a hipMalloc that can be told to
fail in front of the HIP library's."""
import os
import subprocess
import sys
import textwrap

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
typedef int (*fn)(void **, unsigned long);
fn real;
int deny, denied;
int hipMalloc(void **p, unsigned long n) {
  if (!deny) return real(p, n);
  ++denied;
  return 2; /* out of memory */
}
"""

RUN = """
import ctypes, os, sys
import numpy as np
sys.path.insert(0, sys.argv[1])
hip = ctypes.CDLL("/opt/rocm/lib/libamdhip64.so.7")
shim = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
ctypes.c_void_p.in_dll(shim, "real").value = ctypes.cast(hip.hipMalloc, ctypes.c_void_p).value
deny = ctypes.c_int.in_dll(shim, "deny")
import synth
from paper_1906_04722_amd import lbm
few = synth.Problem(nx=40, ny=40, nz=40, bc=(synth.BC_WALLS,) * 3,
                    spheres=np.array([[20.0, 20.0, 20.0, 33.0]]))
for p in (synth.c1_problem(seed=1), few):
    a, b = lbm.Throat(p), lbm.Throat(p)
    a.step(31)
    ref = a.f()
    deny.value = 1
    try:
        lbm.Throat(p)
        raise SystemExit("the allocations were not denied")
    except lbm.LBMError as e:
        assert e.code == lbm.LBM_ENOMEM
    a.save(sys.argv[3])
    b.load(sys.argv[3])
    deny.value = 0
    assert np.array_equal(b.f(), ref)
    a.step(9)
    b.step(9)
    assert np.array_equal(a.f(), b.f())
print("saved and loaded without an allocation")
"""


def test_save_and_load_without_device_memory(tmp_path):
    src, shim, run = (tmp_path / n for n in ("shim.c", "shim.so", "run.py"))
    src.write_text(SHIM)
    run.write_text(textwrap.dedent(RUN))
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-o", str(shim), str(src)])
    out = subprocess.run([sys.executable, str(run), ROOT, str(shim), str(tmp_path / "state.lbm")],
                         capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "without an allocation" in out.stdout

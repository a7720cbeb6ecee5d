"""What a prediction keeps between calls is bounded, also after a call that was
refused.  A subprocess counts the live device memory with a hipMalloc and a
hipFree in front of the HIP library's."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
typedef int (*alloc_fn)(void **, unsigned long);
typedef int (*free_fn)(void *);
alloc_fn real_malloc;
free_fn real_free;
static void *at[4096];
static long size[4096];
long live;
int hipMalloc(void **p, unsigned long n) {
  int i, r = real_malloc(p, n);
  for (i = 0; r == 0 && i < 4096; ++i)
    if (!at[i]) { at[i] = *p; size[i] = (long)n; live += (long)n; break; }
  return r;
}
int hipFree(void *p) {
  int i;
  for (i = 0; p && i < 4096; ++i)
    if (at[i] == p) { at[i] = 0; live -= size[i]; break; }
  return real_free(p);
}
"""

RUN = """
import ctypes, sys
import numpy as np
sys.path.insert(0, sys.argv[1])
hip = ctypes.CDLL("/opt/rocm/lib/libamdhip64.so.7")
shim = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
for ours, theirs in (("real_malloc", hip.hipMalloc), ("real_free", hip.hipFree)):
    ctypes.c_void_p.in_dll(shim, ours).value = ctypes.cast(theirs, ctypes.c_void_p).value
live = ctypes.c_long.in_dll(shim, "live")
from paper_1906_04722_amd import lbm, surrogate
m = surrogate.Surrogate(members=2, seed=1)
m.set_stats(np.zeros(80), np.ones(80), np.zeros(17), np.ones(17))
X = np.random.default_rng(0).normal(size=(200000, 80))
m.predict(X[:100000])
kept = live.value
assert kept > 0
ref = m.predict(X)
assert live.value <= kept, (live.value, kept)
X[150000, 3] = np.nan
try:
    m.predict(X)
    raise SystemExit("a row that is not finite was accepted")
except lbm.LBMError as e:
    assert e.code == lbm.LBM_ENONFINITE
print("live", live.value, "kept", kept)
assert live.value <= kept, (live.value, kept)
again = m.predict(X[:100000])
assert np.array_equal(again[0], ref[0][:100000]) and np.array_equal(again[1], ref[1][:100000])
"""


def test_a_refused_prediction_gives_its_memory_back(tmp_path):
    src, shim, run = (tmp_path / n for n in ("shim.c", "shim.so", "run.py"))
    src.write_text(SHIM)
    run.write_text(RUN)
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-o", str(shim), str(src)])
    out = subprocess.run([sys.executable, str(run), ROOT, str(shim)], capture_output=True, text=True,
                         timeout=100)
    print(out.stdout)
    assert out.returncode == 0, out.stdout + out.stderr

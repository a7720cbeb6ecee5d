"""Runs a piece of code in a process where a hipMalloc and a hipFree of ours
stand in front of the HIP library's, so that a test can count the device memory
that is held, or deny it."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
typedef int (*alloc_fn)(void **, unsigned long);
typedef int (*free_fn)(void *);
alloc_fn real_malloc;
free_fn real_free;
static void *at[4096];
static long size[4096];
long live;
long deny;
int hipMalloc(void **p, unsigned long n) {
  int i, r;
  if (deny && (long)n >= deny) return 2; /* out of memory */
  r = real_malloc(p, n);
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

# live.value: bytes held; deny.value: hipMallocs of that many bytes and more fail
HEAD = """
import ctypes, sys
import numpy as np
sys.path.insert(0, sys.argv[1])
hip = ctypes.CDLL("libamdhip64.so.7")
shim = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
for ours, theirs in (("real_malloc", hip.hipMalloc), ("real_free", hip.hipFree)):
    ctypes.c_void_p.in_dll(shim, ours).value = ctypes.cast(theirs, ctypes.c_void_p).value
live = ctypes.c_long.in_dll(shim, "live")
deny = ctypes.c_long.in_dll(shim, "deny")
"""


def run(tmp_path, code, *args):
    src, lib, main = (tmp_path / n for n in ("shim.c", "shim.so", "main.py"))
    src.write_text(SHIM)
    main.write_text(HEAD + code)
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)])
    out = subprocess.run([sys.executable, str(main), ROOT, str(lib), *args], capture_output=True,
                         text=True, timeout=100)
    print(out.stdout)
    assert out.returncode == 0, out.stdout + out.stderr

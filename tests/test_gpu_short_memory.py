"""Allocations that fail.  A child process puts its own hipMalloc and hipHostMalloc
before the runtime's, which refuse what is larger than a limit with
hipErrorOutOfMemory and pass the rest on: a context whose neighbour slots do not fit
takes the compacted cache, one that fits nothing reports RWPT_ENOMEM and goes on,
and queries without page-locked memory return the same values."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <dlfcn.h>
#include <stddef.h>
size_t device_limit = (size_t)-1, host_limit = (size_t)-1;
int refused = 0;
static void *real(const char *name) {
  void *lib = dlopen("libamdhip64.so", RTLD_LAZY);
  if (!lib) lib = dlopen("/opt/rocm/lib/libamdhip64.so", RTLD_LAZY);
  return dlsym(lib, name);
}
int hipMalloc(void **p, size_t n) {
  if (n > device_limit) { ++refused; return 2; }
  return ((int (*)(void **, size_t))real("hipMalloc"))(p, n);
}
int hipHostMalloc(void **p, size_t n, unsigned flags) {
  if (n > host_limit) { ++refused; return 2; }
  return ((int (*)(void **, size_t, unsigned))real("hipHostMalloc"))(p, n, flags);
}
"""

HEAD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_1811_05474_amd import rwpt, workloads as W
limit, refused = ctypes.c_size_t.in_dll(shim, "device_limit"), ctypes.c_int.in_dll(shim, "refused")
"""

SLOTS = r"""
n, nb, dt = 60000, 10.0, 0.1
D = (nb / (n * 4.18879)) ** (2.0 / 3.0) / 7.2
x, M = W.positions(n, 3, 1), W.masses(n, 2, 1)
out = []
# 938 tiles of 64 particles with 32 slots: 15.4 MB of weights and 7.7 MB of indices; all else is below 2 MB
for cap in (2**62, 10_000_000, 5_000_000):
    limit.value, refused.value = cap, 0
    e = rwpt.Ensemble(dim=3, n_species=2, react=(0, 1), rw_ratio=1.0, precision=rwpt.RWPT_FP64, seed=3)
    e.init([n], x, M)
    e.step(dt, D, 3)
    out.append(e.masses())
    assert (refused.value > 0) == (cap < 2**62), (cap, refused.value)
    e.close()
assert all(np.abs(o - out[0]).max() <= 1e-11 * np.abs(out[0]).max() for o in out[1:])
limit.value = 1 << 18
e = rwpt.Ensemble(dim=3, n_species=2, react=(0, 1), rw_ratio=1.0, precision=rwpt.RWPT_FP64, seed=3)
try:
    e.init([n], x, M)
    raise SystemExit("no error")
except rwpt.RwptError as err:
    assert err.status == rwpt.RWPT_ENOMEM, err
limit.value = 2**62
e.init([n], x, M)
e.step(dt, D, 3)
assert np.array_equal(e.masses(), out[0])
print("CHILD OK")
"""

QUERIES = r"""
limit = ctypes.c_size_t.in_dll(shim, "host_limit")
for prec in (rwpt.RWPT_FP32, rwpt.RWPT_FP64):
    for n in (1000, 700001):  # one chunk of the read-back and several
        out = []
        for cap in (2**62, 1000, 0):
            limit.value, refused.value = cap, 0
            e = rwpt.Ensemble(dim=2, n_species=2, react=(0, 1), rw_ratio=1.0, precision=prec, seed=3)
            e.init([n], W.positions(n, 2, 1), W.masses(n, 2, 1))
            e.step(0.1, 0.5 / n, 2)
            out.append((e.masses(), e.positions()))
            assert (refused.value > 0) == (cap < 2**62)
            e.close()
        for o in out[1:]:
            assert all(np.array_equal(a, b) for a, b in zip(out[0], o))
print("CHILD OK")
"""


@pytest.mark.parametrize("child", [SLOTS, QUERIES], ids=["slots", "queries"])
def test_without_memory(child, tmp_path):
    src, lib = tmp_path / "shim.c", tmp_path / "libshim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", str(lib), str(src), "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-c", HEAD + child, str(lib), ROOT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "CHILD OK" in r.stdout, r.stdout + r.stderr

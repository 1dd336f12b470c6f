"""Creation of a graph when a device allocation fails: each one in turn is made
to fail (in a process of its own, where hipMalloc is counted on its way to the
runtime).  A graph whose triangle layout cannot be had keeps the edge list, with
the same results; only what every graph needs makes creation fail, and nothing
stays allocated."""
import pytest

from hip_shim import run_child

pytestmark = pytest.mark.gpu

SHIM = r"""
#include <cstddef>
static int (*real_malloc)(void**, size_t);
static int (*real_free)(void*);
static int calls, fail_at, held;
extern "C" {
void shim_real(void* m, void* f) {
  real_malloc = (int (*)(void**, size_t))m;
  real_free = (int (*)(void*))f;
}
void shim_reset(int at) { calls = 0; fail_at = at; }
int shim_calls() { return calls; }
int shim_held() { return held; }
int hipMalloc(void** p, size_t n) {
  if (++calls == fail_at) { *p = nullptr; return 2; }  // hipErrorOutOfMemory
  const int e = real_malloc(p, n);
  if (e == 0) ++held;
  return e;
}
int hipFree(void* p) {
  const int e = real_free(p);
  if (e == 0 && p) --held;
  return e;
}
}
"""

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before the library, which then binds to it
import numpy as np
import graphgen as gg, oracle
import paper_2311_12281_amd as S
hip = S.lib()
shim.shim_real(ctypes.cast(hip.hipMalloc, ctypes.c_void_p), ctypes.cast(hip.hipFree, ctypes.c_void_p))
g = gg.rmat(12, 16, seed=8)
counts = oracle.counts(g)
expect = oracle.cluster(g, counts, 1, 5, 3)
def check(G):
    labels, roles = G.run(1, 5, 3)
    assert np.array_equal(labels, expect[0]) and np.array_equal(roles, expect[1])
    assert np.array_equal(G.similarity(), counts)
shim.shim_reset(0)
G = S.Graph.from_csr(g)
total, whole = shim.shim_calls(), G.device_bytes()
check(G)
G.close()
assert total > 3 and shim.shim_held() == 0, (total, shim.shim_held())
refused, kept = [], []
for k in range(1, total + 1):
    print("allocation", k, "of", total, flush=True)
    shim.shim_reset(k)
    try:
        G = S.Graph.from_csr(g)
    except S.ScanError as e:
        assert e.code == S.SCAN_E_NOMEM, e
        refused.append(k)
    else:
        shim.shim_reset(0)
        kept.append(G.device_bytes())
        check(G)
        G.close()
    assert shim.shim_held() == 0, k
# offsets, ids and the flags of their check
assert refused == [1, 2, 3], refused
assert all(b < whole for b in kept), (kept, whole)
print("OK")
"""


def test_each_allocation_fails_once(tmp_path):
    run_child(tmp_path, SHIM, CHILD)

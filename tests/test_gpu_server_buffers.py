"""The server's pinned result buffers when a graph is added: those that are large
enough stay, and while larger ones are allocated the graphs already there are
served.  (In a process of its own, where hipHostMalloc is counted and can be held
up on its way to the runtime.)"""
import pytest

from hip_shim import run_child

pytestmark = pytest.mark.gpu

SHIM = r"""
#include <atomic>
#include <chrono>
#include <cstddef>
#include <thread>
static int (*real)(void**, size_t, unsigned);
static std::atomic<int> calls{0}, hold{0}, held{0};
extern "C" {
void shim_real(void* f) { real = (int (*)(void**, size_t, unsigned))f; }
int shim_calls() { return calls; }
void shim_hold(int on) { hold = on; }  // the next call waits until this is taken back (10 s at most)
int shim_held() { return held; }
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  ++calls;
  int one = 1;
  if (hold.compare_exchange_strong(one, 2)) {
    held = 1;
    for (int k = 0; k < 10000 && hold == 2; ++k) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    held = 0;
  }
  return real(p, n, flags);
}
}
"""

CHILD = r"""
import ctypes, sys, threading, time
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before the library, which then binds to it
import numpy as np
import graphgen as gg, oracle
import paper_2311_12281_amd as S
shim.shim_real(ctypes.cast(S.lib().hipHostMalloc, ctypes.c_void_p))
small, dense, large = gg.planted(3000, 30, 0.2, 0.001, 1), gg.planted(3000, 5, 0.6, 0.01, 2), gg.rmat(13, 16, seed=3)
expect = oracle.scan(small, 1, 5, 4)
def ask(srv, gid):
    labels, roles, _ = srv.wait(srv.submit(gid, 1, 5, 4), gid)
    assert np.array_equal(labels, expect[0]) and np.array_equal(roles, expect[1])
with S.Server(num_slots=6) as srv:
    a = srv.add(small)
    ask(srv, a)
    pinned = shim.shim_calls()
    assert pinned >= 12  # labels and roles of six
    srv.add(dense)  # as many vertices, longer rows: larger slots, the same results
    assert shim.shim_calls() == pinned, (shim.shim_calls(), pinned)
    ask(srv, a)
    shim.shim_hold(1)
    adding = threading.Thread(target=srv.add, args=(large,))
    adding.start()
    while not shim.shim_held():
        time.sleep(0.001)
    ask(srv, a)
    still = shim.shim_held()
    shim.shim_hold(0)
    adding.join()
    assert still == 1, "the query waited for the buffers"
    ask(srv, a)
print("OK")
"""


def test_buffers_when_a_graph_is_added(tmp_path):
    run_child(tmp_path, SHIM, CHILD)

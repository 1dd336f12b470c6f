"""Overlapping calls on one graph whose callers bring streams: one handle that
is another stream in every thread (hipStreamPerThread), and streams destroyed
as soon as the call on them has returned.  Every result against the oracle."""
import ctypes
import threading

import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2311_12281_amd as S
from gpu_helpers import assert_same, note

pytestmark = pytest.mark.gpu

PER_THREAD = 2  # hipStreamPerThread
PARAMS = [((1, 5), 5), ((1, 2), 3), ((3, 10), 4), ((1, 10), 6)]


@pytest.mark.parametrize("streams", ["per-thread", "own", "mixed"])
def test_callers_streams(streams):
    g = gg.rmat(14, 16, seed=41)
    oc = oracle.counts(g, threads=oracle.max_threads())
    expect = {pm: oracle.cluster(g, oc, *pm[0], pm[1]) for pm in PARAMS}
    hip = S.lib()  # the HIP runtime's own entry points come with the library
    nt, calls = 5, 6
    note("streams", streams, f"{nt} threads x {calls} calls")
    out, errs = {}, []
    start = threading.Barrier(nt)

    def work(t):
        dl, dr = S.scan_device_alloc(4 * g.n), S.scan_device_alloc(g.n)
        try:
            start.wait()
            for k in range(calls):
                (p, q), mu = pm = PARAMS[(t + k) % len(PARAMS)]
                if streams == "per-thread" or (streams == "mixed" and t % 2):
                    G.run_device(p, q, mu, dl, dr, PER_THREAD)
                else:
                    s = ctypes.c_void_p()
                    assert hip.hipStreamCreate(ctypes.byref(s)) == 0
                    G.run_device(p, q, mu, dl, dr, s.value)
                    assert hip.hipStreamDestroy(s) == 0
                lab, rol = np.empty(g.n, np.int32), np.empty(g.n, np.uint8)
                S.scan_memcpy_d2h(lab, dl, 4 * g.n)
                S.scan_memcpy_d2h(rol, dr, g.n)
                out[(t, k)] = (pm, lab, rol)
        except BaseException as e:  # noqa: BLE001 - raised below
            errs.append(e)
        finally:
            S.scan_device_free(dl)
            S.scan_device_free(dr)

    with S.Graph.from_csr(g) as G:
        ts = [threading.Thread(target=work, args=(t,)) for t in range(nt)]
        for x in ts:
            x.start()
        for x in ts:
            x.join()
    if errs:
        raise errs[0]
    for (t, k), (pm, lab, rol) in sorted(out.items()):
        assert_same(lab, rol, *expect[pm], f"thread {t} call {k} eps={pm[0]} mu={pm[1]}")

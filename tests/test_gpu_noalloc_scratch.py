"""scan_run_device_noalloc on the triangle path: its scratch lies in the static
array where that holds it, and a graph then has one scratch of its own, not two.
Calls on graphs of both kinds follow each other on the one array."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2311_12281_amd as S
from gpu_helpers import assert_same, note
from test_zz_no_alloc import _device_result

pytestmark = pytest.mark.gpu


def _clique(n):
    i, j = np.triu_indices(n, 1)
    return gg.from_pairs(n, i.astype(np.int32), j.astype(np.int32))


def test_one_scratch():
    g = _clique(1000)
    bits = 4 * sum(-(-d // 32) * min(d, 32) + sum(-(-d // 32) - (c >> 5) for c in range(32, d)) for d in range(1000))
    assert 20e6 < bits < 25e6
    with S.Graph.from_csr(g) as G:
        held = G.device_bytes()
        note("clique of 1,000", f"bits {bits}, held {held}")
        G.run(1, 2, 5)
    # rows, ids and records: 3 records of 16 bytes an edge, and 30 bytes
    assert held < 80 * g.m + 1.5 * bits


@pytest.mark.parametrize("hub_outlier", [False, True])
def test_both_kinds_in_turn(hub_outlier):
    graphs = [gg.rmat(14, 16, seed=51), gg.chung_lu(300000, 30.0, 2.1, 5000.0, seed=52), _clique(300),
              gg.planted(9001, 45, 0.15, 0.0005, 53)]
    params = [(1, 5, 3), (2, 5, 2), (1, 2, 5), (1, 5, 4)]
    handles = [S.Graph.from_csr(g, hub_outlier=hub_outlier) for g in graphs]
    expect = []
    for g, pm in zip(graphs, params):
        ol, orr = oracle.scan(g, *pm, threads=oracle.max_threads())
        expect.append((ol, oracle.hub_outlier(g, ol, orr) if hub_outlier else orr))
    for k in (0, 1, 2, 3, 1, 0, 3, 2, 0):
        note("noalloc in turn", k, hub_outlier)
        nl, nr = _device_result(handles[k], graphs[k].n, handles[k].run_device_noalloc, *params[k])
        assert_same(nl, nr, *expect[k], f"graph {k}")
        G = handles[(k + 1) % 4]  # a call on its own scratch in between
        assert_same(*G.run(*params[(k + 1) % 4]), *expect[(k + 1) % 4], f"graph {(k + 1) % 4} by scan_run")
    for G in handles:
        G.close()

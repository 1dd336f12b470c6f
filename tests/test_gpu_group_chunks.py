"""Group kernels on buckets of few edges, where a wave takes fewer than 64 at a
time and all buckets share a launch (partitioned graphs), against the oracle:
rings whose vertices all have one degree, so that one bucket holds every edge,
with edge counts around the chunk sizes, and one graph with every bucket."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2311_12281_amd as S
from gpu_helpers import assert_same, note

pytestmark = pytest.mark.gpu


def _ring(n, k):
    return [(i, (i + d) % n) for i in range(n) for d in range(1, k + 1)]


def _check(g, name):
    budget = 8 * (g.n + 1) + 22 * g.n + (1 << 20) + (1 << 16) + max(4096, 6 * g.nnz)
    note("group chunks", name, f"m={g.m} budget={budget}")
    oc = oracle.counts(g, threads=oracle.max_threads())
    for pruning in (True, False):
        with S.Graph.from_csr(g, budget=budget, pruning=pruning) as P:
            assert np.array_equal(P.similarity(), oc)
            for (p, q), mu in [((1, 2), 2), ((3, 5), 3), ((1, 10), 6)]:
                gl, gr = P.run(p, q, mu)
                ol, orr = oracle.cluster(g, oc, p, q, mu)
                assert_same(gl, gr, ol, orr, f"{name} pruning={pruning} eps={p}/{q} mu={mu}")


@pytest.mark.parametrize("n,k", [(5, 1), (64, 1), (65, 2), (4097, 4), (33, 8), (8193, 8), (41, 16), (700, 32),
                                 (8192, 33), (300, 100)])
def test_one_bucket(n, k):
    _check(gg.from_edges(n, _ring(n, k)), f"ring {n} {k}")


def test_every_bucket():
    rng = np.random.default_rng(5)
    edges, at = [], 0
    for k, n in [(1, 50), (3, 60), (6, 70), (12, 90), (25, 120), (60, 200)]:
        edges += [(at + a, at + b) for a, b in _ring(n, k)]
        at += n
    edges += [(at, int(v)) for v in rng.choice(at, 580, replace=False)]  # a row above 512
    edges += [(at + 1, int(v)) for v in rng.choice(at, 560, replace=False)]
    _check(gg.from_edges(at + 2, edges), "every bucket")

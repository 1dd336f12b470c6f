"""The edge-list kernels of a graph that is resident: a device budget that the
graph fits keeps it off the triangle path.  Against the oracle, counts and
clusterings."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2311_12281_amd as S
from gpu_helpers import assert_groups_whole, assert_same, note
from test_gpu_group_chunks import _ring

pytestmark = pytest.mark.gpu


def check_resident(g, params, name, **opts):
    """On the pruned edge-list path unless opts say otherwise."""
    budget = S.scan_graph_footprint(g.n, g.nnz, S.make_opts(**opts))
    note("edge list", name, f"n={g.n} m={g.m}", opts)
    oc = oracle.counts(g, threads=oracle.max_threads())
    with S.Graph.from_csr(g, budget=budget, **opts) as G:
        assert 0 < G.device_bytes() <= budget
        gc = G.similarity()
        assert np.array_equal(gc, oc), f"{name}: counts differ at {np.count_nonzero(gc != oc)} arcs"
        assert_groups_whole(G, name)
        for (p, q), mu in params:
            gl, gr = G.run(p, q, mu)
            assert G.stats()["h2d_bytes"] == 0  # resident
            assert_groups_whole(G, f"{name} eps={p}/{q} mu={mu}")
            ol, orr = oracle.cluster(g, oc, p, q, mu)
            assert_same(gl, gr, ol, orr, f"{name} eps={p}/{q} mu={mu}")


@pytest.mark.parametrize("n,k", [(5, 1), (65, 2), (16385, 2), (1025, 4), (8193, 8), (2049, 16), (700, 32), (1024, 33),
                                 (300, 100)])
def test_one_bucket(n, k):
    """Rings whose vertices all have one degree: edge counts around the sizes at which a wave's chunk
    halves (2048 waves of 64 edges and fewer)."""
    check_resident(gg.from_edges(n, _ring(n, k)), [((1, 2), 2), ((3, 5), 3), ((1, 10), 6)], f"ring {n} {k}")

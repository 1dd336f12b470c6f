"""The triangle path at the edges of its pieces, against the oracle: row lengths
around a line (32 entries), a wave's step (64) and the wave kernel's limit
(128); the three lookup tables of the block kernel (chosen by the vertex's
place in the degree order, 16384 and 65534); rows above 4096 entries, which
the edge-list kernels take instead."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2311_12281_amd as S
from gpu_helpers import assert_same, note

pytestmark = pytest.mark.gpu


def _check(g, name, params):
    oc = oracle.counts(g, threads=oracle.max_threads())
    note(name, f"n={g.n} m={g.m}")
    with S.Graph.from_csr(g) as G:
        gc = G.similarity()
        assert np.array_equal(gc, oc), f"{name}: counts differ at {np.count_nonzero(gc != oc)} arcs"
        for (p, q), mu in params:
            gl, gr = G.run(p, q, mu)
            ol, orr = oracle.cluster(g, oc, p, q, mu)
            assert_same(gl, gr, ol, orr, f"{name} eps={p}/{q} mu={mu}")


@pytest.mark.parametrize("k", [2, 3, 32, 33, 34, 64, 65, 66, 96, 97, 128, 129, 130, 131, 257, 300])
def test_row_lengths(k):
    """A clique of k with some edges missing and a pendant vertex per member:
    rows of every length up to k."""
    rng = np.random.default_rng(k)
    edges = [(i, j) for i in range(k) for j in range(i + 1, k) if rng.random() < 0.9]
    edges += [(i, k + i) for i in range(k)]
    perm = rng.permutation(2 * k)
    _check(gg.from_edges(2 * k, [(int(perm[a]), int(perm[b])) for a, b in edges]), f"clique {k}",
           [((1, 2), 2), ((4, 5), 3), ((1, 10), 5)])


def test_lookup_tables():
    """70,000 vertices of about equal degree (270): rows above the wave
    kernel's limit on both sides of both table limits."""
    g, _ = gg.permute(gg.planted(70000, 175, 0.6, 0.0004, 3), 4)
    deg = np.sort(g.degrees())[::-1]
    assert g.n > 65534 and deg[-1] > 200
    _check(g, "tables", [((1, 2), 5), ((2, 5), 100)])


def test_rows_above_the_limit():
    """A clique of 4,200 with a few edges missing has rows above 4,096 entries."""
    n = 4200
    i, j = np.triu_indices(n, 1)
    keep = np.random.default_rng(7).random(i.size) < 0.995
    g = gg.from_pairs(n, i[keep].astype(np.int32), j[keep].astype(np.int32))
    _check(g, "long rows", [((99, 100), 4000), ((1, 2), 5)])


@pytest.mark.parametrize("k", [513, 895, 896, 897, 1008, 1345, 1793])
def test_in_edge_batches(k):
    """k vertices joined to the same four: in-edge records of the block kernel
    around a wave's batch (56) and a job (896), some of several lines."""
    rng = np.random.default_rng(k)
    edges = [(a, b) for a in range(4) for b in range(a)]
    edges += [(a, 4 + i) for i in range(k) for a in range(4)]
    edges += [(4 + a, 4 + b) for a in range(90) for b in range(a) if rng.random() < 0.9]
    perm = rng.permutation(4 + k)
    _check(gg.from_edges(4 + k, [(int(perm[a]), int(perm[b])) for a, b in edges]), f"in-edges {k}",
           [((1, 2), 2), ((1, 10), 5)])


@pytest.mark.parametrize("k", [31, 32, 33, 63, 64, 65, 66, 97, 129, 257, 500])
def test_wave_parts(k):
    """k vertices joined to the same three: the in-edges of a wave's row around
    the parts that waves take (32 records)."""
    rng = np.random.default_rng(k)
    edges = [(1, 0), (2, 0), (2, 1)] + [(a, 3 + i) for i in range(k) for a in range(3)]
    perm = rng.permutation(3 + k)
    _check(gg.from_edges(3 + k, [(int(perm[a]), int(perm[b])) for a, b in edges]), f"parts {k}",
           [((1, 2), 2), ((1, 10), 5)])

"""Sizes around the limits of the triangle layout: beyond them a graph keeps the
edge list, with the same results."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2311_12281_amd as S
from gpu_helpers import assert_same, note
from test_zz_no_alloc import _device_result

pytestmark = pytest.mark.gpu


def _spread(n):
    """Few edges over n vertices: a small graph whose vertices are moved, in order, to ids from one end
    to the other.  The graph, the ids and the small graph."""
    small = gg.planted(400, 8, 0.5, 0.01, 5)
    ids = np.linspace(0, n - 1, small.n).astype(np.int64)
    row_ptr = np.zeros(n + 1, np.int64)
    row_ptr[ids + 1] = small.degrees()
    np.cumsum(row_ptr, out=row_ptr)
    return gg.CSR(n, row_ptr, ids[small.col_idx].astype(np.int32)), ids, small


def _check(labels, roles, ids, small, p, q, mu, ctx):
    ol, orr = oracle.scan(small, p, q, mu)
    assert_same(labels[ids], roles[ids], np.where(ol < 0, -1, ids[ol]).astype(np.int32), orr, ctx)
    assert np.count_nonzero(roles) == np.count_nonzero(orr) and np.count_nonzero(labels >= 0) == np.count_nonzero(ol >= 0)


@pytest.mark.parametrize("n", [67_108_860, 67_108_861])
def test_vertex_limit(n):
    """A wave per vertex is 2^32 threads from 67,108,861 vertices on, more than a launch takes."""
    g, ids, small = _spread(n)
    note("vertices", n)
    with S.Graph.from_csr(g) as G:
        assert np.array_equal(G.similarity(), oracle.counts(small))
        for (p, q), mu in [((1, 2), 3), ((1, 5), 5)]:
            _check(*G.run(p, q, mu), ids, small, p, q, mu, f"n={n} eps={p}/{q}")


def test_vertex_limit_in_a_batch_and_a_server():
    g, ids, small = _spread(67_108_700)
    note("batch of", g.n + small.n, "vertices")
    with S.Batch([g, small], [(1, 2), (1, 5)], [3, 5]) as B:
        labels, roles = B.run()
        (l0, l1), (r0, r1) = B.split(labels), B.split(roles)
        _check(l0, r0, ids, small, 1, 2, 3, "batch, first")
        assert_same(l1, r1, *oracle.scan(small, 1, 5, 5), "batch, second")
    g, ids, small = _spread(67_108_861)
    note("server", g.n)
    with S.Server(num_slots=1) as srv:
        gid = srv.add(g)
        _check(*srv.wait(srv.submit(gid, 1, 2, 3), gid)[:2], ids, small, 1, 2, 3, "server")


@pytest.mark.parametrize("n,hub", [(63, 40), (4_095, 251), (4_096, 252), (4_097, 253), (8_193, 2_044), (8_192, 2_045),
                                   (262_147, 65_531), (262_144, 65_532), (300_001, 70_000)])
def test_renaming(n, hub):
    """The sort by degree: vertices around its tiles of 4,096, largest degrees around one, two and three
    passes of 8 bits; and around 2,048 neighbours, above which a row is laid out in chunks."""
    rng = np.random.default_rng(n + hub)
    src = [np.arange(n - 2), np.arange(n - 2), np.zeros(hub, np.int64) + 17]
    dst = [np.arange(1, n - 1), np.arange(2, n), rng.choice(np.setdiff1d(np.arange(n), np.arange(15, 20)), hub, replace=False)]
    g = gg.from_pairs(n, np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32))
    assert g.degrees().max() == hub + 4
    oc = oracle.counts(g, threads=oracle.max_threads())
    note("renaming", n, hub)
    with S.Graph.from_csr(g) as G:
        assert np.array_equal(G.similarity(), oc)
        for (p, q), mu in [((3, 5), 3), ((1, 4), 4)]:
            assert_same(*G.run(p, q, mu), *oracle.cluster(g, oc, p, q, mu), f"n={n} hub={hub} eps={p}/{q}")


def test_renaming_of_a_large_batch():
    graphs = [gg.rmat(9 + k % 6, 8, seed=80 + k) for k in range(90)] + [gg.from_edges(0, []), gg.from_edges(3, [(0, 2)])]
    assert sum(g.n for g in graphs) > 1 << 18
    eps, mus = [(1 + k % 5, 8) for k in range(len(graphs))], [2 + k % 4 for k in range(len(graphs))]
    note("renaming of a batch")
    with S.Batch(graphs, eps, mus) as B:
        labels, roles = B.run()
        for k, (g, (p, q), mu, l, r) in enumerate(zip(graphs, eps, mus, B.split(labels), B.split(roles))):
            assert_same(l, r, *oracle.scan(g, p, q, mu), f"graph {k} eps={p}/{q} mu={mu}")


def _rings(parts, seed=None):
    """Disjoint rings (vertices, neighbours on each side), ids shuffled if a seed is given."""
    src, dst, at = [], [], 0
    for n, k in parts:
        i = np.arange(n)
        for d in range(1, k + 1):
            src.append(at + i)
            dst.append(at + (i + d) % n)
        at += n
    p = np.arange(at) if seed is None else np.random.default_rng(seed).permutation(at)
    return gg.from_pairs(at, p[np.concatenate(src)].astype(np.int32), p[np.concatenate(dst)].astype(np.int32))


@pytest.mark.parametrize("parts", [
    [(65_535, 4)], [(65_536, 4)], [(65_537, 4), (100, 5)], [(1_001, 40), (65_600, 3)], [(70_001, 1), (33, 2)],
    [(30_000, 2), (30_000, 4), (6_007, 1), (5_000, 5)], [(400, 150), (70_001, 4)], [(3_000, 300), (66_001, 2)]], ids=str)
@pytest.mark.parametrize("seed", [None, 5])
def test_vertices_of_few_neighbours(parts, seed):
    """From 65,536 vertices of at most 8 neighbours on, eight of them share a wave while the rows are laid
    out, and k_tri_few counts for them unless the others have more records."""
    g = _rings(parts, seed)
    oc = oracle.counts(g, threads=oracle.max_threads())
    note("few neighbours", parts, seed)
    with S.Graph.from_csr(g) as G:
        assert np.array_equal(G.similarity(), oc)
        for (p, q), mu in [((1, 2), 3), ((7, 10), 2), ((4, 5), 5)]:
            assert_same(*G.run(p, q, mu), *oracle.cluster(g, oc, p, q, mu), f"{parts} eps={p}/{q}")


def test_few_neighbours_served_and_without_allocations():
    g = _rings([(500, 60), (66_000, 4), (300, 2)], 9)
    p, q, mu = 3, 5, 4
    ol, orr = oracle.scan(g, p, q, mu, threads=oracle.max_threads())
    note("few neighbours, no-alloc and served")
    with S.Graph.from_csr(g) as G:
        for _ in range(2):
            assert_same(*_device_result(G, g.n, G.run_device_noalloc, p, q, mu), ol, orr, "no-alloc")
    with S.Server(num_slots=2) as srv:
        gid = srv.add(g)
        assert_same(*srv.wait(srv.submit(gid, p, q, mu), gid)[:2], ol, orr, "served")


def test_a_missing_reverse_arc_among_them():
    g = _rings([(70_000, 2)])
    ci = g.col_idx.copy()
    u = 43_210  # its last neighbour becomes one that does not name it back
    assert ci[g.row_ptr[u + 1] - 1] == u + 2
    ci[g.row_ptr[u + 1] - 1] = u + 3
    note("missing reverse arc")
    with pytest.raises(S.ScanError) as ei:
        S.scan_graph_create(g.n, g.nnz, g.row_ptr, ci)
    assert ei.value.code == S.SCAN_E_GRAPH

"""The edge-list kernels of a graph that is resident (a device budget that the
graph fits keeps it off the triangle path), and the queue kernel of a batch.
Against the oracle, counts and clusterings: on graphs of their own and in the
tests of resident graphs and batches, which otherwise run on the triangle path."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2311_12281_amd as S
import test_gpu_batched as batched
import test_gpu_concurrent as concurrent
import test_gpu_hub_outlier as hubs
import test_gpu_parity as parity
import test_zz_no_alloc as noalloc
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


@pytest.fixture
def edge_list(monkeypatch):
    """Graphs without a budget get one of twice their footprint: the edge list, with room for the buffer
    sets of overlapping calls."""
    real = S.Graph.from_csr.__func__

    def from_csr(cls, g, **opts):
        fits = S.scan_graph_footprint(g.n, g.nnz, S.make_opts(**opts))
        if not opts.get("budget"):
            opts["budget"] = 2 * fits + (8 << 20)
        return real(cls, g, **opts)

    monkeypatch.setattr(S.Graph, "from_csr", classmethod(from_csr))


@pytest.mark.parametrize("case", [
    parity.test_paper_example, parity.test_closed_forms, parity.test_small_graphs_against_oracle,
    parity.test_planted_config_A, parity.test_planted_pruning_off_is_identical, parity.test_rmat_relabelled,
    parity.test_chung_lu, parity.test_repeated_runs_identical, parity.test_edge_cases,
    parity.test_device_entry_points, parity.test_stats_are_consistent, parity.test_windowed_hub,
    parity.test_full_survivor_batch, parity.test_crowded_hash_bucket, hubs.test_paper_example_hubs_and_outliers,
    hubs.test_hub_outlier_off_keeps_three_roles, concurrent.test_overlapping_host_calls,
    concurrent.test_overlapping_device_calls, concurrent.test_similarity_and_runs_overlap,
    noalloc.test_noalloc_refuses_oversize_run], ids=lambda f: f.__name__[5:])
def test_tests_of_resident_graphs(edge_list, case):
    case()


@pytest.mark.parametrize("scale", [14, 16, 18])
def test_rmat(edge_list, scale):
    parity.test_rmat(scale)


@pytest.mark.parametrize("ranked", [False, True])
@pytest.mark.parametrize("case", [parity.test_rmat20_permuted, parity.test_bitmap_window_edges,
                                  parity.test_bitmap_and_hash_windows], ids=lambda f: f.__name__[5:])
def test_ranked_rows(edge_list, case, ranked):
    case(ranked)


@pytest.mark.parametrize("name,gen", [("rmat16", lambda: gg.rmat(16, 16, seed=2)),
                                      ("spread-hub", parity.spread_hub_graph), ("windowed-hub", parity.windowed_hub_graph)])
def test_strategies_identical(edge_list, name, gen):
    parity.test_strategies_identical(name, gen)


@pytest.mark.parametrize("hub_outlier", [False, True])
def test_noalloc(edge_list, hub_outlier):
    noalloc.test_noalloc_matches_scan_run_device(hub_outlier)


def test_hub_outlier(edge_list):
    g = gg.planted(20000, 100, 0.2, 0.002, 11)
    for (p, q), mu in [((1, 5), 5), ((1, 3), 4)]:
        hubs._check(g, p, q, mu)


@pytest.mark.parametrize("case", [
    batched.test_batch_matches_oracle_per_graph, batched.test_batch_of_skewed_graphs,
    batched.test_batch_replays_match_eager, batched.test_batch_equals_scan_run_and_autotune,
    batched.test_batch_new_params_without_recapture, batched.test_batch_hub_outlier_roles],
    ids=lambda f: f.__name__[5:])
def test_tests_of_batches(monkeypatch, case):
    """On the queue kernel, which a stated wait for its items selects (20 s, as without one)."""
    monkeypatch.setenv("SCAN_BATCH_WATCHDOG_US", "20000000")
    case()


def test_batch_without_pruning():
    graphs = [gg.rmat(10 + k % 4, 8 + k, seed=60 + k) for k in range(12)] + [gg.planted(2000, 20, 0.3, 0.002, 7)]
    eps, mus = [(1 + k % 4, 5) for k in range(13)], [2 + k % 5 for k in range(13)]
    note("batch, pruning off")
    with S.Batch(graphs, eps, mus, pruning=False) as B:
        labels, roles = B.run()
        for k, (g, (p, q), mu, l, r) in enumerate(zip(graphs, eps, mus, B.split(labels), B.split(roles))):
            assert_same(l, r, *oracle.scan(g, p, q, mu), f"graph {k} eps={p}/{q} mu={mu}")

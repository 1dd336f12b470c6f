"""Device memory of graphs created without a budget: within five times
scan_graph_footprint plus 512 MiB, as scan.h states, with every buffer that its
calls take, whatever the shape of the graph; results against the oracle."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2311_12281_amd as S
from gpu_helpers import assert_same, note

pytestmark = pytest.mark.gpu


def _dense(n, p):
    i, j = np.triu_indices(n, 1)
    keep = np.random.default_rng(3).random(i.size) < p
    return gg.from_pairs(n, i[keep].astype(np.int32), j[keep].astype(np.int32))


def _grid(w, diagonals):
    v = np.arange(w * w, dtype=np.int32).reshape(w, w)
    a, b = [v[:, :-1], v[:-1]], [v[:, 1:], v[1:]]
    if diagonals:
        a.append(v[:-1, :-1])
        b.append(v[1:, 1:])
    return gg.from_pairs(w * w, np.concatenate([x.ravel() for x in a]), np.concatenate([x.ravel() for x in b]))


GRAPHS = {
    "dense rows of 3,600": lambda: _dense(4000, 0.9),
    "dense rows of 1,200": lambda: _dense(4000, 0.3),
    "path": lambda: gg.from_pairs(3_000_000, np.arange(2_999_999, dtype=np.int32), np.arange(1, 3_000_000, dtype=np.int32)),
    "grid": lambda: _grid(1500, False),
    "triangulated grid": lambda: _grid(1500, True),
    "rmat": lambda: gg.rmat(17, 16, seed=6),
    "star": lambda: gg.from_pairs(200_001, np.zeros(200_000, np.int32), np.arange(1, 200_001, dtype=np.int32)),
}


@pytest.mark.parametrize("name", GRAPHS)
def test_within_the_stated_bound(name):
    g = GRAPHS[name]()
    most = 5 * S.scan_graph_footprint(g.n, g.nnz) + (512 << 20)
    oc = oracle.counts(g, threads=oracle.max_threads())
    note("memory", name, f"n={g.n} m={g.m}")
    with S.Graph.from_csr(g) as G:
        for (p, q), mu in [((1, 5), 3), ((3, 5), 4)]:
            assert_same(*G.run(p, q, mu), *oracle.cluster(g, oc, p, q, mu), f"{name} eps={p}/{q} mu={mu}")
        assert np.array_equal(G.similarity(), oc)
        held = G.device_bytes()
        note(f"{held / 1e6:.0f} MB of {most / 1e6:.0f}")
        assert held <= most


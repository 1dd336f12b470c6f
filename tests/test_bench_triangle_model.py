"""The bench's byte model of a triangle-path solve, which reports look-ups in all
and none per degree bucket."""
import bench
import graphgen as gg


def test_per_eps_bytes_of_the_triangle_path():
    # a triangle 0-1-2 with a pendant 3 on vertex 2
    g = gg.from_edges(4, [(0, 1), (1, 2), (2, 0), (2, 3)])
    fixed = 4 * 8 + 8 * 5 + 17 * 4  # rows, offsets, per-vertex state
    st = {"cores_bucket_probes": [0] * 7, "cores_bucket_evaluated": [4, 0, 0, 0, 0, 0, 0], "probes": {"cores": 96}}
    assert bench.triangle_bytes(st, g.m) == 2 * 96 + 28 * 4
    assert bench.solve_byte_models(g, [st])["per_eps_probe_model_bytes"] == [2 * 96 + 28 * 4 + fixed]

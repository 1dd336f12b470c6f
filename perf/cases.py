"""Timed cases of the library: what its users have it do, through its public calls.

Each case is a dict of plain values.  ``kind`` names the call:

* ``run``         ``Graph.run``: cluster a resident graph, labels and roles to host arrays
* ``device``      ``Graph.run_device``: the same with the outputs left in device memory, one
                  call per (eps, mu) of ``params``
* ``noalloc``     ``Graph.run_device_noalloc``: the entry point of loops that may not allocate
* ``similarity``  ``Graph.similarity``: the closed count of every arc, to a host array
* ``oneshot``     a host CSR to labels and roles: create, run, destroy
* ``batch``       ``Batch.run``: many small graphs in one captured replay
* ``serve``       ``Server``: a burst of queries on resident graphs, submitted and awaited
* ``partitioned`` ``Graph.run`` on a graph larger than its device budget

Graphs come from the seeded generators (``graphgen``): planted partitions
(communities of about equal degree), R-MAT (skewed, with hubs) and Chung-Lu
(power law).  ``params`` is "p/q,mu" items separated by ";".
"""
import math

import numpy as np
import torch

import graphgen as gg
import paper_2311_12281_amd as S


def listed():
    return [
        # the smallest call a user makes (a few thousand vertices): launches and copies count
        {"name": "run_planted2k", "kind": "run", "graph": "planted", "n": 2000, "blocks": 10, "deg": 43.0,
         "params": "1/5,5"},
        # the plain SCAN workload of the paper's small graphs: 10,000 vertices in 50 blocks
        {"name": "run_planted10k", "kind": "run", "graph": "planted", "n": 10000, "blocks": 50, "deg": 34.7,
         "params": "1/5,5"},
        # a community graph of odd size, many clusters and borders, with hub and outlier roles
        {"name": "run_planted150k_roles", "kind": "run", "graph": "planted", "n": 150001, "blocks": 3000, "deg": 31.0,
         "params": "2/5,4", "hub_outlier": True},
        # a mid-size skewed graph
        {"name": "run_rmat17", "kind": "run", "graph": "rmat", "scale": 17, "ef": 16, "params": "3/10,3"},
        # a power-law graph (social network), low threshold: most edges have to be intersected
        {"name": "run_chunglu500k", "kind": "run", "graph": "chunglu", "n": 500009, "deg": 30.0, "maxdeg": 9000.0,
         "params": "1/5,4"},
        # the headline workload: R-MAT scale 22 at three thresholds, outputs left in device memory
        {"name": "device_rmat22", "kind": "device", "graph": "rmat", "scale": 22, "ef": 16,
         "params": "1/5,5;1/2,5;4/5,5"},
        # a tight loop that may not allocate, on a small skewed graph
        {"name": "noalloc_rmat14", "kind": "noalloc", "graph": "rmat", "scale": 14, "ef": 16, "params": "3/10,4"},
        # exact counts of every arc, for a caller that thresholds by itself; ids without order
        {"name": "similarity_rmat19", "kind": "similarity", "graph": "rmat", "scale": 19, "ef": 12, "params": ""},
        # a new graph every time: upload, validation, layout and one solve
        {"name": "oneshot_rmat18", "kind": "oneshot", "graph": "rmat", "scale": 18, "ef": 16, "params": "1/5,3"},
        # hundreds of small graphs with parameters of their own in one replay
        {"name": "batch_300", "kind": "batch", "count": 300, "n_hi": 20000},
        # a burst of queries on a few resident graphs
        {"name": "serve_24q", "kind": "serve", "graphs": 3, "scale_lo": 16, "scale_hi": 18, "queries": 24, "slots": 4},
        # a graph streamed through a device budget it does not fit
        {"name": "partitioned_chunglu200k", "kind": "partitioned", "graph": "chunglu", "n": 200000, "deg": 30.0,
         "maxdeg": 4000.0, "frac": 0.2, "params": "1/5,4"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_params(rng, case, count=1):
    """Thresholds of use, up to where a graph of this kind has no similar edge."""
    out = []
    for _ in range(count):
        if case["graph"] == "planted":
            # the similarity inside a block is about 0.74 deg / (vertices of a block)
            top = max(2, int(6 * case["deg"] * case["blocks"] / case["n"]))
            p = rng.randint((top + 1) // 2, top)
            mu = rng.randint(2, 6)
        else:
            p = rng.randint(1, 5)
            mu = rng.randint(2, 5) if p <= 3 else 2
        out.append("%d/10,%d" % (p, mu))
    return ";".join(out)


def _draw_graph(rng, big):
    """One graph of the listed range; big: the upper end of its edge count."""
    g = rng.choice(["planted", "rmat", "chunglu"])
    if g == "planted":
        n = _log_int(rng, 500, max(2000, big // 20))
        deg = rng.uniform(8, 64)
        return {"graph": g, "n": n, "blocks": max(2, int(n / (deg * rng.uniform(1.1, 2.5)))), "deg": deg}
    if g == "rmat":
        top = max(12, int(math.log2(big / 16)))
        return {"graph": g, "scale": rng.randint(11, top), "ef": rng.randint(8, 24), "permute": rng.random() < 0.3}
    n = _log_int(rng, 3000, max(6000, big // 16))
    return {"graph": g, "n": n, "deg": rng.uniform(6, 40), "maxdeg": float(max(100, n // rng.randint(20, 100)))}


def draw(rng):
    kind = rng.choice(["run", "run", "run", "device", "noalloc", "similarity", "oneshot", "batch", "serve",
                       "partitioned"])
    if kind == "batch":
        return {"kind": kind, "count": _log_int(rng, 20, 400), "n_hi": _log_int(rng, 1000, 20000)}
    if kind == "serve":
        lo = rng.randint(14, 16)
        return {"kind": kind, "graphs": rng.randint(1, 4), "scale_lo": lo, "scale_hi": lo + rng.randint(0, 2),
                "queries": rng.randint(4, 30), "slots": rng.randint(1, 6)}
    if kind == "partitioned":
        n = _log_int(rng, 100000, 300000)
        return {"kind": kind, "graph": "chunglu", "n": n, "deg": 30.0, "maxdeg": n / 50.0,
                "frac": rng.uniform(0.15, 0.5), "params": _draw_params(rng, {"graph": "chunglu"})}
    big = {"run": 1 << 24, "device": 1 << 24, "noalloc": 1 << 20, "similarity": 1 << 22, "oneshot": 1 << 22}[kind]
    case = {"kind": kind, **_draw_graph(rng, big)}
    solves = rng.randint(1, 3) if kind == "device" else 1
    case["params"] = "" if kind == "similarity" else _draw_params(rng, case, solves)
    if kind == "run" and rng.random() < 0.25:
        case["hub_outlier"] = True
    return case


def _graph(case, seed):
    """The case's graph as a host CSR.  The arcs of a counted graph are the
    same for every seed but for their ids, so that its counts are as many."""
    if case["kind"] == "similarity":
        return gg.permute(_generate(case, 2), seed)[0]
    g = _generate(case, seed)
    # the generator numbers communities one after the other, which no real graph does
    return gg.permute(g, seed + 1)[0] if case.get("permute") or case["graph"] == "planted" else g


def _generate(case, seed):
    if case["graph"] == "planted":
        # 86 % of the mean degree inside a vertex's block, as in the batched workload
        n, B, D = case["n"], min(case["blocks"], case["n"] // 2), case["deg"]
        s = n / B
        p_in = min(1.0, 0.86 * D / max(1.0, s - 1))
        p_out = min(1.0, max(0.0, (D - p_in * (s - 1)) / max(1.0, n - s)))
        return gg.planted(n, B, p_in, p_out, seed)
    if case["graph"] == "rmat":
        return gg.rmat(case["scale"], case["ef"], seed=seed)
    return gg.chung_lu(case["n"], case["deg"], 2.1, case["maxdeg"], seed=seed)


def _params(case):
    out = []
    for item in case["params"].split(";"):
        eps, mu = item.split(",")
        p, q = eps.split("/")
        out.append((int(p), int(q), int(mu)))
    return out


def _budget(g, frac):
    """Device bytes that hold the per-vertex state, but only part of the graph."""
    resident = 8 * (g.n + 1) + 22 * g.n + (1 << 20)
    layout = 8 * (g.n + 1) + 4 * g.nnz + 13 * (g.nnz // 2) + 22 * g.n + (1 << 20)
    return int(resident + frac * (layout - resident))


def _batch(case, seed):
    specs = gg.planted_batch_specs(case["count"], seed=4, n_hi=case["n_hi"])
    graphs = [gg.planted(s.n, s.blocks, s.p_in, s.p_out, s.seed + seed) for s in specs]
    return graphs, [s.eps for s in specs], [s.mu for s in specs]


def _served(case, seed):
    """The resident graphs and the burst of queries."""
    specs, _ = gg.serving_specs(case["graphs"], 0, seed=5, scale_lo=case["scale_lo"], scale_hi=case["scale_hi"],
                                ef_lo=8, ef_hi=24)
    graphs = [gg.rmat(s.scale, s.edge_factor, seed=seed + k) for k, s in enumerate(specs)]
    return graphs, gg.serving_queries(case["queries"], case["graphs"], seed=6)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return {"kind": kind, "batch": S.Batch(*_batch(case, seed))}
    if kind == "serve":
        graphs, queries = _served(case, seed)
        srv = S.Server(num_slots=case["slots"])
        gids = [srv.add(g) for g in graphs]
        # a client reuses its result arrays
        out = [(np.empty(graphs[k].n, np.int32), np.empty(graphs[k].n, np.uint8)) for k, _, _, _ in queries]
        return {"kind": kind, "server": srv, "queries": [(gids[k], p, q, mu) for k, p, q, mu in queries], "out": out}
    g = _graph(case, seed)
    if kind == "oneshot":
        return {"kind": kind, "csr": g, "params": _params(case)}
    opts = {"hub_outlier": bool(case.get("hub_outlier"))}
    if kind == "partitioned":
        opts["budget"] = _budget(g, case["frac"])
    st = {"kind": kind, "graph": S.Graph.from_csr(g, **opts)}
    if kind != "similarity":
        st["params"] = _params(case)
    if kind in ("device", "noalloc"):
        st["out"] = [(torch.empty(g.n, dtype=torch.int32, device="cuda"),
                      torch.empty(g.n, dtype=torch.uint8, device="cuda")) for _ in st["params"]]
    return st


def run(st):
    kind = st["kind"]
    if kind == "batch":
        return st["batch"].run()
    if kind == "serve":
        srv = st["server"]
        reqs = [(srv.submit(gid, p, q, mu), gid) for gid, p, q, mu in st["queries"]]
        return [srv.wait(r, gid, lab, rol)[:2] for (r, gid), (lab, rol) in zip(reqs, st["out"])]
    if kind == "oneshot":
        with S.Graph.from_csr(st["csr"]) as G:
            return [G.run(*pm) for pm in st["params"]]
    G = st["graph"]
    if kind == "similarity":
        return G.similarity()
    if kind in ("device", "noalloc"):
        call = G.run_device if kind == "device" else G.run_device_noalloc
        for pm, (lab, rol) in zip(st["params"], st["out"]):
            call(*pm, lab.data_ptr(), rol.data_ptr())
        return st["out"]
    return [G.run(*pm) for pm in st["params"]]


def work(case):
    """Each graph read once per solve, each result written once (no floating point on the path)."""
    kind = case["kind"]
    if kind == "batch":
        graphs = _batch(case, 1)[0]
        return {"bytes": sum(8 * (g.n + 1) + 4 * g.nnz + 5 * g.n for g in graphs), "flops": 0}
    if kind == "serve":
        graphs, queries = _served(case, 1)
        # a query reads an edge's endpoints and its count
        return {"bytes": sum(12 * graphs[k].m + 8 * (graphs[k].n + 1) + 5 * graphs[k].n for k, _, _, _ in queries),
                "flops": 0}
    g = _graph(case, 1)
    read = 8 * (g.n + 1) + 4 * g.nnz
    if kind == "similarity":
        return {"bytes": read + 4 * g.nnz, "flops": 0}
    return {"bytes": len(_params(case)) * (read + 5 * g.n), "flops": 0}


def _exact_one(g, p, q, mu, split):
    """SCAN from its definitions on a dense adjacency matrix: (labels, roles)."""
    A = torch.zeros((g.n, g.n), dtype=torch.float64)
    src = torch.from_numpy(np.repeat(np.arange(g.n), np.diff(g.row_ptr)))
    dst = torch.from_numpy(g.col_idx.astype(np.int64))
    A[src, dst] = 1
    closed = A + torch.eye(g.n, dtype=torch.float64)
    common = (closed.cuda() @ closed.cuda()).cpu()[src, dst].to(torch.int64)
    size = torch.from_numpy(np.diff(g.row_ptr) + 1)
    sim = (common * q) ** 2 >= p * p * size[src] * size[dst]
    near = torch.ones(g.n, dtype=torch.int64).index_add_(0, src[sim], torch.ones(int(sim.sum()), dtype=torch.int64))
    core = near >= mu
    none = g.n
    label = torch.where(core, torch.arange(g.n), none)
    both = sim & core[src] & core[dst]
    while True:  # smallest core id of the connected similar cores
        new = label.scatter_reduce(0, dst[both], label[src[both]], "amin")
        if torch.equal(new, label):
            break
        label = new
    one = sim & core[src] & ~core[dst]
    label = label.scatter_reduce(0, dst[one], label[src[one]], "amin")
    role = torch.where(core, 1, torch.where(label < none, 2, 0))
    if split:
        out = role == 0
        seen = out[src] & (label[dst] < none)
        lo = torch.full((g.n,), none).scatter_reduce(0, src[seen], label[dst[seen]], "amin")
        hi = torch.full((g.n,), -1).scatter_reduce(0, src[seen], label[dst[seen]], "amax")
        role = torch.where(out, torch.where(hi > lo, 3, 4), role)
    return torch.where(label < none, label, -1).to(torch.int32), role.to(torch.uint8)


def exact(case, seed):
    """Whole numbers from the definitions, for single graphs small enough for a dense matrix."""
    if case["kind"] not in ("run", "device", "noalloc", "oneshot") or case.get("n", 1 << case.get("scale", 31)) > 12000:
        return None
    g = _graph(case, seed)
    return [_exact_one(g, p, q, mu, bool(case.get("hub_outlier"))) for p, q, mu in _params(case)]

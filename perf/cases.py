"""Work that programs built on this library have it do, as cases that can be
timed and compared.

Every case goes through the Python binding's public calls (`Graph`, `Batch`,
`Server` and their methods).  The inputs are the repository's own synthetic
families: R-MAT (skewed social, web and Kronecker graphs), Erdos-Renyi
(unclustered) and random geometric graphs (clustered, short rows), at the
sizes of its workloads and tests and at odd sizes between them.

    op        one pass                                        what is kept between passes
    tc        build, partition and count                      the edge list (device)
    stream    the same, blocks streamed under a device cap    the edge list (device)
    count     count of a partitioned graph                    the graph
    batch     counts of many small graphs, one launch         the batch, launch shape tuned
    serve     a burst of requests submitted and drained       the server, the edge lists (host)
    support   triangles on every edge                         the graph, the output tensor
    vertex    triangles at every vertex                       the graph, the output tensor
    ktruss    edges of the k-truss                            the graph
    cliques   4-cliques, per block 4-list                     the partitioned graph
    components / pagerank  over the blocks                    the partitioned graph
"""
from __future__ import annotations

import math
import os
import tempfile

import numpy as np
import torch

# Launch shapes that the library's autotuner finds go to a file of this
# process, so that the passes of one program do not depend on another's.
os.environ.setdefault("PGABB_TUNE_CACHE", os.path.join(tempfile.mkdtemp(prefix="pgabb_cases_"), "tune.txt"))

import paper_2209_04541_amd as P
from paper_2209_04541_amd import gen

# Seeds of these inputs: gen.seed(_CONFIG, ...), a stream apart from the
# workloads' own.
_CONFIG = 77


def listed():
    return [
        # the plain workload: a small unclustered graph counted whole, where
        # launches and round trips are the time
        {"name": "tc_er4096", "op": "tc", "family": "er", "n": 4096, "pairs": 32768, "p": 1},
        # the block workload: a skewed graph built, cut into 8 x 8 blocks and counted
        {"name": "tc_rmat20_p8", "op": "tc", "family": "rmat", "scale": 20, "ef": 16, "p": 8},
        # a graph held on the device in blocks and counted again (shards,
        # repeated counts, served requests at their largest scale)
        {"name": "count_rmat22_p8", "op": "count", "family": "rmat", "scale": 22, "ef": 16, "p": 8},
        # a graph whose blocks do not fit the device budget given to it
        {"name": "stream_rmat21_p16", "op": "stream", "family": "rmat", "scale": 21, "ef": 16, "p": 16,
         "cap_mib": 160},
        # the batch workload's mix of small graphs, an odd number of them
        {"name": "batch_777", "op": "batch", "graphs": 777},
        # a burst of requests of the served workload's kind, from host memory
        {"name": "serve_16", "op": "serve", "requests": 16, "scale_lo": 10, "scale_hi": 16},
        # clustering coefficients of edges on the block workload's graph
        {"name": "support_rmat20", "op": "support", "family": "rmat", "scale": 20, "ef": 16},
        # local clustering coefficients of a spatial graph, odd size
        {"name": "vertex_rgg", "op": "vertex", "family": "rgg", "n": 200003, "degree": 24},
        {"name": "ktruss_rmat18", "op": "ktruss", "family": "rmat", "scale": 18, "ef": 16, "k": 8},
        {"name": "cliques_rmat18_p4", "op": "cliques", "family": "rmat", "scale": 18, "ef": 16, "p": 4},
        {"name": "components_rmat20_p8", "op": "components", "family": "rmat", "scale": 20, "ef": 16, "p": 8},
        {"name": "pagerank_rmat20_p8", "op": "pagerank", "family": "rmat", "scale": 20, "ef": 16, "p": 8},
    ]


# Largest number of input pairs a drawn case of each operation takes.
_MOST_PAIRS = {"tc": 1 << 24, "count": 1 << 25, "stream": 1 << 25, "support": 1 << 24, "vertex": 1 << 24,
               "ktruss": 1 << 22, "cliques": 1 << 22, "components": 1 << 24, "pagerank": 1 << 24}


def _draw_graph(rng, lo, hi):
    """A family and its sizes, between lo and hi input pairs."""
    pairs = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    family = rng.choice(("rmat", "rmat", "er", "rgg"))
    if family == "rmat":
        ef = rng.randint(8, 32)
        scale = max(10, int(math.log2(pairs / ef)))
        return {"family": "rmat", "scale": scale, "ef": ef}
    degree = rng.randint(8, 64)
    n = max(65, int(2 * pairs / degree)) | 1
    if family == "er":
        return {"family": "er", "n": n, "pairs": n * degree // 2}
    return {"family": "rgg", "n": min(n, 400001), "degree": degree}


def draw(rng):
    op = rng.choice(("tc", "tc", "count", "count", "stream", "batch", "serve", "support", "vertex", "ktruss",
                     "cliques", "components", "pagerank"))
    if op == "batch":
        return {"op": op, "graphs": rng.randint(50, 777)}
    if op == "serve":
        lo = rng.randint(10, 13)
        return {"op": op, "requests": rng.randint(3, 24), "scale_lo": lo, "scale_hi": rng.randint(lo, 16)}
    low = 1 << (20 if op == "stream" else 13)
    case = {"op": op, **_draw_graph(rng, low, _MOST_PAIRS[op])}
    if op == "stream":
        case["p"] = rng.randint(9, 24)
        # from about a third of the block store (some 24 bytes per pair) up
        case["cap_mib"] = max(16, int(_pairs(case) * 24 * rng.uniform(0.3, 1.2)) >> 20)
    elif op in ("support", "vertex", "ktruss"):
        if op == "ktruss":
            case["k"] = rng.randint(3, 12)
    else:
        case["p"] = rng.choice((1, 2, 3, 4, 5, 8, 8, 11, 16))
        if op == "cliques":
            case["p"] = min(case["p"], 8)
    return case


def _graph_pairs(case, seed):
    """(n, src, dst) of the case's graph on the host."""
    sv = gen.seed(_CONFIG, int(seed) & 0x7FFFFFFF)
    if case["family"] == "rmat":
        return gen.rmat(case["scale"], case["ef"], sv)
    if case["family"] == "er":
        return gen.er(case["n"], case["pairs"], sv)
    return gen.rgg(case["n"], case["degree"], sv)


def _device_pairs(case, seed):
    n, s, d = _graph_pairs(case, seed)
    return n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda()


def _request(case, seed, r):
    """Request r of a served burst: an R-MAT graph of a scale in the burst's range."""
    sv = gen.seed(_CONFIG + 1, (int(seed) * 1009 + r) & 0x7FFFFFFF)
    scale = case["scale_lo"] + r % (case["scale_hi"] - case["scale_lo"] + 1)
    return gen.rmat(scale, gen.uniform_int(sv, 1, 8, 32), sv)


def _batch_graphs(case, seed):
    """Graphs of the batch workload's recipe: random geometric and Erdos-Renyi
    in turn, 64 to 8192 vertices, average degree 8 to 64."""
    out = []
    for g in range(case["graphs"]):
        sv = gen.seed(_CONFIG + 2, (int(seed) * 100003 + g) & 0x7FFFFFFF)
        n = gen.uniform_int(sv, 1, 64, 8192)
        d = gen.uniform_int(sv, 2, 8, 64)
        out.append(gen.rgg(n, d, sv) if g % 2 == 0 else gen.er(n, min(n * d // 2, n * (n - 1) // 2), sv))
    return out


def prepare(case, seed):
    op = case["op"]
    st = {"op": op, "case": dict(case)}
    if op == "batch":
        st["batch"] = P.Batch(_batch_graphs(case, seed))
        st["batch"].count()  # tunes the launch shape and captures the launch
        return st
    if op == "serve":
        st["graphs"] = [_request(case, seed, r) for r in range(case["requests"])]
        st["server"] = P.Server(8 << 30)
        return st
    n, src, dst = _device_pairs(case, seed)
    if op in ("tc", "stream"):
        st["edges"] = (n, src, dst)
        return st
    g = P.Graph(n, src, dst)
    if "p" in case:
        g.partition(case["p"])
    st["graph"] = g
    # the number of distinct edges differs from seed to seed: edge results go
    # to the front of a buffer of the number of pairs
    if op == "support":
        st["whole"] = torch.zeros(_most_edges(case), dtype=torch.int32, device="cuda")
        st["out"] = st["whole"][:g.info()["m"]]
    elif op == "ktruss":
        st["whole"] = np.zeros(_most_edges(case), np.uint8)
    elif op == "vertex":
        st["out"] = torch.empty(n, dtype=torch.int64, device="cuda")
    return st


def run(st):
    op, case = st["op"], st["case"]
    if op == "tc":
        with P.Graph(*st["edges"]) as g:
            g.partition(case["p"])
            return {"triangles": g.count(), "tasks": g.task_counts()[1].astype(np.int64)}
    if op == "stream":
        with P.Graph(*st["edges"]) as g:
            g.partition(case["p"])
            return {"triangles": g.count(device_cap_bytes=case["cap_mib"] << 20, stream_blocks=True),
                    "tasks": g.task_counts()[1].astype(np.int64)}
    if op == "batch":
        return {"triangles": st["batch"].count().astype(np.int64)}
    if op == "serve":
        srv = st["server"]
        tickets = [srv.submit(*g) for g in st["graphs"]]
        srv.drain()
        return {"triangles": [srv.poll(t)[1] for t in tickets]}
    g = st["graph"]
    if op == "count":
        return {"triangles": g.count(), "tasks": g.task_counts()[1].astype(np.int64)}
    if op == "support":
        return {"triangles": g.edge_support(st["out"])[1], "counts": st["whole"]}
    if op == "vertex":
        return {"triangles": g.vertex_counts(st["out"])[1], "counts": st["out"]}
    if op == "ktruss":
        keep, edges, rounds = g.ktruss(case["k"])
        st["whole"][:len(keep)] = keep
        return {"keep": st["whole"], "edges": edges, "rounds": rounds}
    if op == "cliques":
        return {"cliques": g.four_cliques(), "lists": g.four_clique_lists()[1].astype(np.int64)}
    if op == "components":
        label, count, _ = g.components()
        return {"label": label, "components": count}
    ranks, iterations, _ = g.pagerank()
    return {"ranks": ranks, "iterations": iterations}


def _pairs(case):
    if case["family"] == "rmat":
        return case["ef"] << case["scale"]
    if case["family"] == "er":
        return case["pairs"]
    return case["n"] * case["degree"] // 2


def _most_edges(case):
    """A bound of the distinct edges, the same for every seed (a random
    geometric graph's pairs vary around their mean)."""
    return 2 * _pairs(case) if case["family"] == "rgg" else _pairs(case)


def _vertices(case):
    return 1 << case["scale"] if case["family"] == "rmat" else case["n"]


def work(case):
    """Each input read once and each output written once: 8 bytes per input
    pair where the pass starts from pairs, else 4 bytes per distinct edge
    (taken as the pairs) and 8 per vertex of the graph held; 4 bytes per
    distinct edge over the host link and back where the blocks are streamed.
    PageRank's operations are one addition per edge end and five per vertex
    and iteration, for the eight iterations that these graphs take."""
    op = case["op"]
    if op == "batch":
        m = case["graphs"] * 65000
        return {"bytes": 4 * m + 8 * case["graphs"] * 4100 + 8 * case["graphs"], "flops": 0}
    if op == "serve":
        scales = [case["scale_lo"] + r % (case["scale_hi"] - case["scale_lo"] + 1) for r in range(case["requests"])]
        return {"bytes": sum(8 * (20 << s) for s in scales), "flops": 0}
    m, n = _pairs(case), _vertices(case)
    if op == "tc":
        return {"bytes": 8 * m, "flops": 0}
    if op == "stream":
        return {"bytes": 16 * m, "flops": 0}
    held = 4 * m + 8 * n
    if op == "support":
        return {"bytes": held + 4 * m, "flops": 0}
    if op == "vertex":
        return {"bytes": held + 8 * n, "flops": 0}
    if op == "ktruss":
        return {"bytes": held + m, "flops": 0}
    if op == "components":
        return {"bytes": held + 4 * n, "flops": 0}
    if op == "pagerank":
        return {"bytes": 8 * (held + 16 * n), "flops": 8 * (2 * m + 5 * n)}
    return {"bytes": held, "flops": 0}


def _exact_pagerank(case, seed):
    n, s, d = _device_pairs(case, seed)
    lo, hi = torch.minimum(s, d).long(), torch.maximum(s, d).long()
    key = torch.unique((lo * n + hi)[lo != hi])
    a, b = torch.cat((key // n, key % n)), torch.cat((key % n, key // n))
    deg = torch.bincount(a, minlength=n).double()
    r = torch.full((n,), 1.0 / n, dtype=torch.float64, device=a.device)
    iterations = 0
    while iterations < 20:
        share = torch.where(deg > 0, r / deg.clamp(min=1), 0.0)
        new = (1.0 - 0.85) / n + 0.85 * torch.zeros_like(r).index_add_(0, b, share[a])
        change = float((new - r).abs().sum())
        r = new
        iterations += 1
        if change < 1e-4:
            break
    return {"ranks": r, "iterations": None}


def exact(case, seed):
    """PageRank's iteration in plain float64 operations, and the count of a
    small graph by dense products; the other results are whole numbers."""
    if case["op"] == "pagerank":
        return _exact_pagerank(case, seed)
    if case["op"] == "tc" and _vertices(case) <= 8192:
        n, s, d = _device_pairs(case, seed)
        a = torch.zeros((n, n), dtype=torch.float64, device=s.device)
        a[s.long(), d.long()] = 1.0
        a = torch.maximum(a, a.T.clone())
        a.fill_diagonal_(0.0)
        return {"triangles": int(round(float((a * (a @ a)).sum()) / 6)), "tasks": None}
    return None

"""Performance cases: graph queries as a user's program issues them through
paper_1911_09135_amd.alb, from a thousand vertices to 8.4 million.

Graph families (the generators' of this repository, drawn here with torch on
the GPU so that a case is ready in a second): RMAT with the Graph500 corner
probabilities, whose hub is vertex 0; capped-Zipf out-degrees (exponent 1.9,
cap n / 4) with uniform targets, the extreme out-degree skew; an undirected
grid, the low-degree, high-diameter class of road networks.  Weights are
uniform in [1, 100].  Self-loops and duplicate edges are dropped.
"""
import math

import numpy as np
import torch

from paper_1911_09135_amd import alb

DAMPING = 0.85


def listed():
    return [
        # the smallest call: a query on a graph of a thousand vertices, launch and barrier latency only
        {"name": "bfs-rmat10", "algo": "bfs", "family": "rmat", "scale": 10, "ef": 16, "source": "random",
         "host": False},
        # a small interactive query whose levels the program reads on the host (the call's default output)
        {"name": "bfs-rmat14-host", "algo": "bfs", "family": "rmat", "scale": 14, "ef": 16, "source": "hub",
         "host": True},
        # the largest breadth-first search: out-degree skew, label array beyond the L2s, odd vertex count
        {"name": "bfs-zipf-8.4M", "algo": "bfs", "family": "zipf", "n": 8400001, "source": "hub", "host": False},
        # an ordinary shortest-path query
        {"name": "sssp-rmat17", "algo": "sssp", "family": "rmat", "scale": 17, "ef": 15, "source": "random",
         "host": False},
        # the benchmark's headline query
        {"name": "sssp-rmat22", "algo": "sssp", "family": "rmat", "scale": 22, "ef": 16, "source": "hub",
         "host": False},
        # a road-like graph: thousands of rounds with short worklists
        {"name": "sssp-grid-1001x777", "algo": "sssp", "family": "grid", "rows": 1001, "cols": 777,
         "source": "random", "host": False},
        # components of a social-network-like graph
        {"name": "cc-rmat20", "algo": "cc", "family": "rmat", "scale": 20, "ef": 16, "host": False},
        # core of a skewed graph: decrements that pile onto hubs
        {"name": "kcore-zipf-1M", "algo": "kcore", "family": "zipf", "n": 1000003, "k": 16, "host": False},
        # push PageRank, the iteration count of the benchmark
        {"name": "pagerank-zipf-1M", "algo": "pagerank", "family": "zipf", "n": 1048576, "iterations": 50,
         "host": False},
        # pull PageRank on in-degree skew
        {"name": "pagerank-pull-rmat20", "algo": "pagerank_pull", "family": "rmat", "scale": 20, "ef": 16,
         "iterations": 20, "host": False},
        # many queries on graphs of different sizes in one call
        {"name": "batch-sssp-64", "algo": "sssp_batch", "family": "set", "graphs": 16, "lo": 12, "hi": 18, "ef": 16,
         "queries": 64, "plan": False},
        # a burst of mixed requests to the server, results in pinned host memory
        {"name": "serve-burst-48", "algo": "serve", "family": "set", "graphs": 8, "lo": 12, "hi": 17, "ef": 16,
         "queries": 48},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    algo = rng.choice(["bfs", "bfs", "sssp", "sssp", "cc", "kcore", "pagerank", "pagerank_pull", "bfs_batch",
                       "sssp_batch", "serve"])
    if algo in ("bfs_batch", "sssp_batch", "serve"):
        lo = rng.randint(9, 13)
        c = {"algo": algo, "family": "set", "graphs": rng.randint(2, 16), "lo": lo, "hi": lo + rng.randint(1, 4),
             "ef": rng.randint(6, 16), "queries": _log(rng, 3, 64)}
        if algo != "serve":
            c["plan"] = rng.random() < 0.4
        return c
    family = rng.choice(["rmat", "zipf", "grid"] if algo in ("bfs", "sssp", "cc") else ["rmat", "zipf"])
    c = {"algo": algo, "family": family}
    top = 22 if algo in ("bfs", "sssp") else 20
    if family == "rmat":
        c.update(scale=rng.randint(10, top), ef=rng.randint(6, 16))
    elif family == "zipf":
        c.update(n=_log(rng, 1000, 1 << top) | 1)
    else:
        c.update(rows=_log(rng, 30, 900), cols=_log(rng, 30, 800))
    if algo in ("bfs", "sssp"):
        c["source"] = rng.choice(["hub", "random"])
    if algo == "kcore":
        c["k"] = rng.randint(3, 32)
    if algo in ("pagerank", "pagerank_pull"):
        c["iterations"] = rng.choice([5, 10, 20, 50])
    c["host"] = rng.random() < 0.25
    return c


# --------------------------------------------------------------------------
# Graphs, drawn on the GPU from the seed alone
# --------------------------------------------------------------------------

def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return gen


def _rmat(scale, ef, gen):
    n, m = 1 << scale, ef << scale
    src = torch.zeros(m, dtype=torch.int64, device="cuda")
    dst = torch.zeros(m, dtype=torch.int64, device="cuda")
    for _ in range(scale):  # quadrant probabilities 0.57, 0.19, 0.19, 0.05
        u = torch.rand(m, device="cuda", generator=gen)
        src = src * 2 + (u >= 0.76)
        dst = dst * 2 + (((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    return n, src, dst


def _zipf(n, gen):
    cap = max(n // 4, 1)
    cdf = torch.arange(1, cap + 1, dtype=torch.float64, device="cuda").pow_(-1.9).cumsum(0)
    cdf /= cdf[-1].clone()
    u = torch.rand(n, dtype=torch.float64, device="cuda", generator=gen)
    deg = torch.searchsorted(cdf, u).clamp_(max=cap - 1) + 1
    src = torch.repeat_interleave(torch.arange(n, device="cuda"), deg)
    dst = torch.randint(0, n, (src.numel(),), device="cuda", generator=gen)
    return n, src, dst


def _grid(rows, cols):
    ids = torch.arange(rows * cols, device="cuda").view(rows, cols)
    src = torch.cat([ids[:, :-1].flatten(), ids[:-1].flatten()])
    dst = torch.cat([ids[:, 1:].flatten(), ids[1:].flatten()])
    return rows * cols, torch.cat([src, dst]), torch.cat([dst, src])


class Csr:
    """Host CSR arrays of one graph, as a program has them before it creates a handle."""

    def __init__(self, n, src, dst, gen, weighted, symmetric=False):
        key = src * n + dst
        if symmetric:
            key = torch.cat([key, dst * n + src])
        key = key[src.repeat(2) != dst.repeat(2)] if symmetric else key[src != dst]
        key = torch.unique_consecutive(key.sort().values)
        row, col = key // n, key % n
        off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        off[1:] = torch.bincount(row, minlength=n).cumsum(0)
        self.n = n
        self.off = off.to(torch.int32).cpu().numpy()
        self.col = col.to(torch.int32).cpu().numpy()
        self.w = None
        if weighted:
            w = torch.randint(1, 101, (col.numel(),), device="cuda", generator=gen, dtype=torch.int32)
            self.w = w.cpu().numpy()

    def source(self, rule, gen):
        deg = np.diff(self.off)
        if rule == "hub":
            return int(np.argmax(deg))
        some = np.flatnonzero(deg >= max(1, int(deg.mean())))  # at least the mean out-degree
        return int(some[int(torch.randint(0, some.size, (1,), device="cuda", generator=gen))])


def _csr(case, gen):
    if case["family"] == "rmat":
        n, src, dst = _rmat(case["scale"], case["ef"], gen)
    elif case["family"] == "zipf":
        n, src, dst = _zipf(case["n"], gen)
    else:
        n, src, dst = _grid(case["rows"], case["cols"])
    both = case["algo"] in ("cc", "kcore") and case["family"] != "grid"
    return Csr(n, src, dst, gen, case["algo"] == "sssp", both)


def _members(case, gen, weighted):
    span = case["hi"] - case["lo"] + 1
    return [Csr(*_rmat(case["lo"] + i % span, case["ef"], gen), gen, weighted) for i in range(case["graphs"])]


# --------------------------------------------------------------------------
# The program: handles and outputs it keeps, and one pass
# --------------------------------------------------------------------------

def prepare(case, seed):
    gen = _generator(seed)
    algo = case["algo"]
    if case["family"] == "set":
        graphs = _members(case, gen, algo != "bfs_batch")
        members = [i % len(graphs) for i in range(case["queries"])]
        sources = [graphs[i].source("random", gen) for i in members]
        state = {"case": case, "set": alb.GraphSet(graphs), "members": members, "sources": sources}
        if algo == "serve":
            state["server"] = alb.Server(state["set"])
            state["kinds"] = ["bfs" if i % 2 else "sssp" for i in range(case["queries"])]
            state["outs"] = [torch.empty(graphs[i].n, dtype=torch.int32, pin_memory=True).numpy() for i in members]
        else:
            state["outs"] = [torch.empty(graphs[i].n, dtype=torch.int32, device="cuda") for i in members]
            if case["plan"]:
                state["plan"] = alb.BatchPlan(state["set"], algo[:-len("_batch")], members, sources,
                                              outs=state["outs"])
        return state
    csr = _csr(case, gen)
    state = {"case": case}
    if algo in ("bfs", "sssp"):
        state["source"] = csr.source(case["source"], gen)
    state["graph"] = alb.Graph(csr.off, csr.col, csr.w, symmetric=algo in ("cc", "kcore"),
                               build_transpose=algo == "pagerank_pull")
    dtype = torch.float32 if algo.startswith("pagerank") else torch.int32
    state["out"] = None if case["host"] else torch.empty(csr.n, dtype=dtype, device="cuda")
    return state


def run(state):
    case = state["case"]
    algo = case["algo"]
    if algo == "serve":
        server = state["server"]
        tickets = [server.submit(kind, member, source, out=out) for kind, member, source, out
                   in zip(state["kinds"], state["members"], state["sources"], state["outs"])]
        return [server.wait(t)[0] for t in tickets]
    if algo == "bfs_batch" or algo == "sssp_batch":
        if case["plan"]:
            return state["plan"].run()[0]
        batch = alb.bfs_batch if algo == "bfs_batch" else alb.sssp_batch
        return batch(state["set"], state["members"], state["sources"], outs=state["outs"])[0]
    g, out = state["graph"], state["out"]
    if algo == "bfs":
        return alb.bfs(g, state["source"], out=out)[0]
    if algo == "sssp":
        return alb.sssp(g, state["source"], out=out)[0]
    if algo == "cc":
        return alb.cc(g, out=out)[0]
    if algo == "kcore":
        return alb.kcore(g, case["k"], out=out)[0]
    if algo == "pagerank":
        return alb.pagerank(g, DAMPING, case["iterations"], out=out)[0]
    return alb.pagerank_pull(g, DAMPING, case["iterations"], out=out)[0]


# --------------------------------------------------------------------------
# What a pass cannot do without, and its result in 64 bits
# --------------------------------------------------------------------------

def _size(case):
    """Vertices and (expected) edges."""
    if case["family"] == "rmat":
        n, m = 1 << case["scale"], case["ef"] << case["scale"]
    elif case["family"] == "zipf":
        n = case["n"]
        k = np.arange(1, max(n // 4, 1) + 1, dtype=np.float64)
        m = int(n * np.sum(k ** -0.9) / np.sum(k ** -1.9))
    else:
        rows, cols = case["rows"], case["cols"]
        return rows * cols, 2 * (rows * (cols - 1) + cols * (rows - 1))
    return n, 2 * m if case["algo"] in ("cc", "kcore") else m


def work(case):
    """CSR read once (once per PageRank iteration, whose result the next one needs), weights where the query has
    them, one 4-byte result per vertex; one operation per edge (two with weights)."""
    if case["family"] == "set":
        span = case["hi"] - case["lo"] + 1
        total, ops = 0, 0
        for i in range(case["queries"]):
            scale = case["lo"] + (i % case["graphs"]) % span
            n, m = 1 << scale, case["ef"] << scale
            weighted = case["algo"] == "sssp_batch" or (case["algo"] == "serve" and i % 2 == 0)
            total += 4 * (2 * n + m * (2 if weighted else 1))
            ops += m * (2 if weighted else 1)
        return {"bytes": total, "flops": ops}
    n, m = _size(case)
    if case["algo"].startswith("pagerank"):
        return {"bytes": case["iterations"] * 4 * (2 * n + m) + 4 * n, "flops": case["iterations"] * (2 * n + m)}
    per_edge = 2 if case["algo"] == "sssp" else 1
    return {"bytes": 4 * (2 * n + per_edge * m), "flops": per_edge * m}


def exact(case, seed):
    """PageRank in 64 bits; levels, distances, components and cores are whole numbers."""
    if not case["algo"].startswith("pagerank"):
        return None
    csr = _csr(case, _generator(seed))
    n = csr.n
    off = torch.from_numpy(csr.off).cuda().to(torch.int64)
    deg = off[1:] - off[:-1]
    src = torch.repeat_interleave(torch.arange(n, device="cuda"), deg)
    dst = torch.from_numpy(csr.col).cuda().to(torch.int64)
    rank = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    damping = float(np.float32(DAMPING))  # the call takes its damping as 32 bits
    for _ in range(case["iterations"]):
        share = torch.where(deg > 0, rank / deg.clamp(min=1), torch.zeros_like(rank))
        into = torch.zeros_like(rank).index_add_(0, dst, share[src])
        rank = (1 - damping) / n + damping * (into + rank[deg == 0].sum() / n)
    return rank.cpu().numpy() if case["host"] else rank

"""The work that programs give this library, as cases that can be timed.

A case is a dict of plain values: which entry point (``op``), the graph (``graph``:
size, mean degree, shape) and the call's options.  ``listed()`` names twelve of
them, ``draw(rng)`` makes others of the same ranges, ``prepare`` builds what a
program holds before the call (graphs and workspaces on the GPU), ``run`` makes one
pass through the public entry points, ``work`` states the bytes and operations a
pass cannot do without, and ``exact`` computes the results by plain NumPy where
that takes seconds.

Graphs are drawn on the GPU from the seed, with a fixed number of edges: power-law
graphs by sampling both ends of every edge in proportion to the expected degrees
(repeats and loops dropped), dense-core graphs by adding planted communities to such a
background, Erdos-Renyi graphs by uniform ends.  Sizes are those of the benchmark and the tests: G(2000, 0.01), the
power-law graph of one million vertices and mean degree 32, the dense-core graph
of half a million vertices with 50 communities of 60 to 80, the batch of 10,000 graphs
of 50 to 5,000 vertices.
"""
import math

import numpy as np
import torch

import paper_2104_13209_amd as kc

ORDERS = {"degree": kc.ORDER_DEGREE, "degeneracy": kc.ORDER_DEGENERACY,
          "approx": kc.ORDER_APPROX_DEGENERACY, "color": kc.ORDER_COLOR}
SCHEMES = {"auto": kc.SCHEME_AUTO, "vertex": kc.SCHEME_VC, "edge": kc.SCHEME_EC}
DEV = "cuda:0"
CAP = 1.45         # largest expected degree of a power-law graph, in units of sqrt(n * mean degree)
SIZES = 128        # clique sizes reported by a count of every size


# ------------------------------------------------------------------- cases

def _case(op, shape, n, mean, **more):
    c = {"op": op, "shape": shape, "n": n, "mean": mean, "gamma": 2.1, "cap": 0.0, "communities": 0,
         "cmin": 0, "cmax": 0, "density": 0.9, "order": "degree", "k": 4, "scheme": "auto", "pivot": False}
    c.update(more)
    return c


def listed():
    cases = [
        # a small graph as tests and notebooks use them: every call is launches and latency
        _case("orient", "uniform", 2000, 20.0, name="small_orient"),
        _case("count", "uniform", 2000, 20.0, k=3, name="small_count_k3"),
        # loading a large graph: the default criterion, and the degeneracy order that
        # deep counts want (both with the input check that is on by default)
        _case("orient", "powerlaw", 1_000_000, 32.0, name="orient_degree_1m"),
        _case("orient", "powerlaw", 1_000_000, 32.0, order="degeneracy", name="orient_degeneracy_1m"),
        # counting on that graph at a small, a middle and a large clique size
        _case("count", "powerlaw", 1_000_000, 32.0, order="degeneracy", k=4, name="count_k4_1m"),
        _case("count", "powerlaw", 1_000_000, 32.0, order="degeneracy", k=7, scheme="edge", name="count_k7_1m"),
        _case("count", "powerlaw", 1_000_000, 32.0, order="degeneracy", k=10, scheme="edge", name="count_k10_1m"),
        # the pivoting traversal at one size, on an odd-sized middle graph
        _case("count", "powerlaw", 74_003, 32.0, k=9, pivot=True, name="pivot_k9_74k"),
        # every clique size at once: communities far denser than what is around them
        _case("count_all", "densecore", 500_000, 40.0, cap=1000.0, communities=50, cmin=60, cmax=80,
              order="degeneracy", name="count_all_densecore"),
        # per-vertex counts (features of a graph's vertices)
        _case("local", "powerlaw", 200_003, 24.0, k=5, name="local_k5_200k"),
        # many independent graphs in one call
        _case("batch", "batch", 10_000, 36.0, gamma=2.3, k=5, name="batch_10k_k5"),
        # a burst of mixed queries to the server over resident graphs
        _case("serve", "powerlaw", 30_011, 24.0, graphs=8, queries=48, name="serve_burst"),
    ]
    return cases


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _kmax(n, mean):
    """A clique size that a power-law graph of this size still has."""
    m = n * mean / 2
    return 4 if m < 50_000 else 6 if m < 400_000 else 8 if m < 2_000_000 else 10


def draw(rng):
    op = rng.choice(["orient", "orient", "count", "count", "count", "pivot", "count_all", "local", "batch", "serve"])
    mean = round(rng.uniform(8.0, 32.0), 2)
    if op == "orient":
        return _case("orient", rng.choice(["uniform", "powerlaw", "powerlaw"]), _log_int(rng, 1000, 1_000_000), mean,
                     order=rng.choice(["degree", "degeneracy", "degeneracy", "approx", "color"]))
    if op == "count":
        n = _log_int(rng, 1000, 1_000_000)
        shape = rng.choice(["uniform", "powerlaw", "powerlaw"])
        return _case("count", shape, n, mean, order=rng.choice(["degree", "degeneracy"]),
                     k=3 if shape == "uniform" else rng.randint(3, _kmax(n, mean)),
                     scheme=rng.choice(["auto", "auto", "edge"]))
    if op == "pivot":
        n = _log_int(rng, 1000, 100_000)
        return _case("count", "powerlaw", n, mean, order=rng.choice(["degree", "degeneracy"]),
                     k=rng.randint(3, _kmax(n, mean)), scheme=rng.choice(["auto", "vertex", "edge"]), pivot=True)
    if op == "count_all":
        n = _log_int(rng, 5000, 300_000)
        lo = rng.randint(20, 60)
        return _case("count_all", "densecore", n, mean, cap=round(min(500.0, math.sqrt(n * mean) / 2), 1),
                     communities=rng.randint(4, 40), cmin=lo, cmax=lo + rng.randint(1, 14),
                     order=rng.choice(["degree", "degeneracy"]), scheme=rng.choice(["auto", "edge"]))
    if op == "local":
        return _case("local", "powerlaw", _log_int(rng, 1000, 200_000), min(mean, 24.0), k=rng.randint(3, 6),
                     pivot=rng.random() < 0.25)
    if op == "batch":
        return _case("batch", "batch", _log_int(rng, 100, 6000), 36.0, gamma=2.3, k=rng.randint(3, 7))
    return _case("serve", "powerlaw", _log_int(rng, 10_000, 40_000), min(mean, 24.0), graphs=rng.randint(2, 8),
                 queries=rng.randint(8, 48))


# ------------------------------------------------------------------ graphs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFF)
    return g


def _xmin(gamma, mean, xmax):
    """x_min of a power law x^-gamma on [x_min, xmax] with this mean."""
    lo, hi = 1e-6, mean
    for _ in range(100):
        mid = 0.5 * (lo + hi)
        a, b = 1.0 - gamma, 2.0 - gamma
        m = ((xmax ** b - mid ** b) / b) / ((xmax ** a - mid ** a) / a)
        lo, hi = (mid, hi) if m < mean else (lo, mid)
    return 0.5 * (lo + hi)


def _keys(n, pairs):
    """The distinct undirected edges among these pairs, as ascending keys u * n + v, u < v."""
    u, v = torch.minimum(pairs[0], pairs[1]), torch.maximum(pairs[0], pairs[1])
    return torch.unique((u * n + v)[u != v])


def _csr(n, key):
    """(row_ptr, col) int32 of the simple symmetric graph with these edges, rows ascending."""
    u, v = key // n, key % n
    key = torch.sort(torch.cat([u * n + v, v * n + u])).values
    rows = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rows[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return rows.to(torch.int32), (key % n).to(torch.int32)


def _edges(case, seed):
    """Exactly n * mean / 2 edges (and those of the planted communities), as keys."""
    n, mean, gamma = case["n"], case["mean"], case["gamma"]
    g = _gen(seed)
    m = int(n * mean / 2)
    if case["shape"] != "uniform":
        wmax = case["cap"] or CAP * math.sqrt(n * mean)
        xmin = _xmin(gamma, mean, wmax)
        a = 1.0 - gamma
        u = np.random.default_rng(seed).random(n)
        w = (xmin ** a + u * (wmax ** a - xmin ** a)) ** (1.0 / a)
        cum = torch.from_numpy(np.cumsum(w)).to(DEV)
    keys, more = torch.empty(0, dtype=torch.int64, device=DEV), 1.15
    while keys.numel() < m:
        if case["shape"] == "uniform":
            pairs = torch.randint(0, n, (2, int(more * m)), generator=g, device=DEV)
        else:
            r = torch.rand((2, int(more * m)), generator=g, device=DEV, dtype=torch.float64) * float(w.sum())
            pairs = torch.searchsorted(cum, r).clamp_(max=n - 1)
        keys = _keys(n, pairs)
        more *= 1.2
    keys = keys[torch.randperm(keys.numel(), generator=g, device=DEV)[:m]]
    if case["shape"] == "densecore":
        # community sizes run through [cmin, cmax]; every community keeps the same share of its pairs
        rng = np.random.default_rng(seed + 1)
        ids = rng.permutation(n)
        at, extra = 0, []
        for c in range(case["communities"]):
            s = case["cmin"] + c % (case["cmax"] - case["cmin"] + 1)
            i, j = np.triu_indices(s, 1)
            keep = rng.permutation(i.size)[:int(case["density"] * i.size)]
            extra.append(np.stack([ids[at + i[keep]], ids[at + j[keep]]]))
            at += s
        extra = torch.from_numpy(np.concatenate(extra, axis=1)).to(DEV)
        keys = torch.cat([keys, _keys(n, extra)])
    return torch.unique(keys)


def _graph(case, seed):
    rp, col = _csr(case["n"], _edges(case, seed))
    return kc.Csr(case["n"], rp, col)


def _batch(case, seed):
    """case["n"] graphs packed into one CSR: 50 to 5,000 vertices (log-uniform), mean degree
    8 to 64, half with uniform and half with power-law ends."""
    rng = np.random.default_rng(seed)
    ng = case["n"]
    size = np.exp(rng.uniform(math.log(50), math.log(5000), ng)).astype(np.int64)
    mean = np.minimum(rng.uniform(8.0, 64.0, ng), size - 1)
    voff = np.concatenate([[0], np.cumsum(size)])
    edges = (size * mean / 2).astype(np.int64)
    n = int(voff[-1])
    g = _gen(seed)
    gid = torch.repeat_interleave(torch.arange(ng, device=DEV), torch.from_numpy(edges).to(DEV))
    sz = torch.from_numpy(size).to(DEV)[gid]
    off = torch.from_numpy(voff[:-1]).to(DEV)[gid]
    plain = torch.from_numpy(rng.random(ng) < 0.5).to(DEV)[gid]
    q = 1.0 - 1.0 / (case["gamma"] - 1.0)
    szf = sz.to(torch.float64)
    # vertices are numbered at random inside their graph
    mix = torch.argsort(torch.rand(n, generator=g, device=DEV, dtype=torch.float64) +
                        torch.repeat_interleave(torch.arange(ng, device=DEV), torch.from_numpy(size).to(DEV)))
    ends = []
    for _ in range(2):
        u = torch.rand(gid.numel(), generator=g, device=DEV, dtype=torch.float64)
        heavy = (u * ((szf + 2.0) ** q - 2.0 ** q) + 2.0 ** q) ** (1.0 / q) - 2.0
        i = torch.where(plain, u * szf, heavy).to(torch.int64)
        ends.append(mix[off + torch.minimum(i.clamp_(min=0), sz - 1)])
    rp, col = _csr(n, _keys(n, torch.stack(ends)))
    deg = rp[1:] - rp[:-1]
    vo = torch.from_numpy(voff).to(DEV)
    at = rp.to(torch.int64)[vo]
    return kc.BatchDev(ng, n, int(deg.max()), rp, col, vo.to(torch.int32), int((at[1:] - at[:-1]).max()) // 2)


# ------------------------------------------------------------ prepare, run

def prepare(case, seed):
    op = case["op"]
    if op == "orient":
        return {"case": case, "graph": _graph(case, seed)}
    if op == "batch":
        b = _batch(case, seed)
        return {"case": case, "batch": b,
                "ws": torch.empty(kc.batch_workspace_bytes(b, case["k"]), dtype=torch.uint8, device=DEV),
                "out": torch.empty(2 * b.ngraphs, dtype=torch.int64, device=DEV)}
    if op == "serve":
        rng = np.random.default_rng(seed)
        dags = [kc.orient(_graph(case, seed + 17 * i), kc.ORDER_DEGENERACY) for i in range(case["graphs"])]
        queries = [(int(rng.integers(0, len(dags))), int(rng.integers(3, 11)), bool(rng.random() < 0.3))
                   for _ in range(case["queries"])]
        return {"case": case, "server": kc.Server(dags, slots=4, mem_budget=4 << 30), "queries": queries}
    dag = kc.orient(_graph(case, seed), ORDERS[case["order"]])
    need = kc.count_workspace_bytes(dag, case["k"], case["pivot"] or op == "count_all")
    return {"case": case, "dag": dag, "ws": torch.empty(need, dtype=torch.uint8, device=DEV)}


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "orient":
        d = kc.orient(state["graph"], ORDERS[case["order"]])
        return [d.row_ptr, d.col, d.src, d.perm, d.d_max, d.degeneracy]
    if op == "count":
        return kc.count(state["dag"], case["k"], pivot=case["pivot"], scheme=SCHEMES[case["scheme"]], ws=state["ws"])
    if op == "count_all":
        counts, omega = kc.count_all(state["dag"], cap=SIZES, scheme=SCHEMES[case["scheme"]], ws=state["ws"])
        # exact 128-bit integers, as two 64-bit halves
        return [np.array([[c & (2 ** 64 - 1), c >> 64] for c in counts], dtype=np.uint64), omega]
    if op == "local":
        return kc.count_local(state["dag"], case["k"], pivot=case["pivot"], scheme=SCHEMES[case["scheme"]], ws=state["ws"])
    if op == "batch":
        kc.batch_count_async(state["batch"], case["k"], state["out"], state["ws"])
        return state["out"]
    server = state["server"]
    tickets = [server.submit(g, k, pivot) for g, k, pivot in state["queries"]]
    return np.array([server.wait(t).value for t in tickets], dtype=np.uint64)


def work(case):
    """Input read once and output written once; operations are not stated (the size of a
    search tree is not known beforehand)."""
    op = case["op"]
    if op == "batch":
        n = case["n"] * (5000 - 50) / math.log(100.0)
        return {"bytes": 4.0 * n + 4.0 * n * case["mean"] + 16.0 * case["n"], "flops": 0.0}
    n, m = case["n"], case["n"] * case["mean"] / 2
    if op == "orient":
        return {"bytes": 4.0 * (n + 2 * m) + 4.0 * (2 * n + 2 * m), "flops": 0.0}
    dag = 4.0 * (n + m)
    if op == "serve":
        return {"bytes": case["queries"] * dag, "flops": 0.0}
    return {"bytes": dag + (8.0 * n if op == "local" else 0.0), "flops": 0.0}


# ------------------------------------------------------------------- exact

def _exact_orient_by_degree(rp, col):
    n = rp.size - 1
    deg = np.diff(rp.astype(np.int64))
    perm = np.lexsort((np.arange(n), deg))
    rank = np.empty(n, np.int64)
    rank[perm] = np.arange(n)
    a, b = rank[np.repeat(np.arange(n), deg)], rank[col]
    key = np.sort((a * n + b)[a < b])
    out = np.bincount(key // n, minlength=n)
    ptr = np.concatenate([[0], np.cumsum(out)])
    return [ptr.astype(np.int32), (key % n).astype(np.int32), (key // n).astype(np.int32), perm.astype(np.int32),
            int(out.max()) if n else 0, -1]


def _exact_counts(rp, col, k):
    """(k-cliques, per-vertex counts) by plain depth-first search over sorted neighbour sets."""
    n = rp.size - 1
    later = [set(x for x in col[rp[v]:rp[v + 1]].tolist() if x > v) for v in range(n)]
    per = np.zeros(n, np.int64)
    total = 0
    stack = [((v,), later[v]) for v in range(n)]
    while stack:
        path, cand = stack.pop()
        if len(path) + 1 == k:
            total += len(cand)
            per[list(path)] += len(cand)
            per[list(cand)] += 1
            continue
        for x in cand:
            rest = cand & later[x]
            if len(rest) >= k - len(path) - 1 - 1 and rest:
                stack.append((path + (x,), rest))
    return total, per


def exact(case, seed):
    op = case["op"]
    if op == "orient" and case["order"] == "degree" and case["n"] <= 1_000_000:
        rp, col = _csr(case["n"], _edges(case, seed))
        return _exact_orient_by_degree(rp.cpu().numpy(), col.cpu().numpy())
    if op in ("count", "local") and case["n"] <= 4000 and case["k"] <= 5 and case["shape"] == "uniform":
        rp, col = _csr(case["n"], _edges(case, seed))
        total, per = _exact_counts(rp.cpu().numpy(), col.cpu().numpy(), case["k"])
        return total if op == "count" else per
    return None

"""What this library is used for, as cases that can be timed and checked.

Each case is one call sequence a program makes through the package's public
class ``BC``: all-source or sampled betweenness by every form, per-source
readouts, edge betweenness, Algorithm 2 over all pairs, Algorithm 1's sampled
distances, and many small graphs in one launch.  Graph families and sizes are
those of the benchmark workloads and the tests (``graphgen``), plus the smaller,
larger and ragged sizes around them.
"""
import functools
import math

import numpy as np
import torch

import graphgen as gg
import paper_0809_1906_amd as bcgpu

DEV = "cuda:0"


def listed():
    return [
        # The smallest call: one source's distances, counts and dependencies on
        # a graph of a few hundred vertices, with every option at its default.
        # Nothing but launches and host steps.
        {"name": "sssp1_er300", "kind": "sssp", "family": "er+tree", "n": 300, "degree": 6.0, "count": 1, "form": "auto"},
        # A small all-source run in FP64, the benchmark's er1024 workload: the
        # accurate form, one workgroup per source.
        {"name": "plain_er1024", "kind": "bc", "family": "er+tree", "n": 1024, "degree": 8.0, "form": "plain"},
        # FP64 on a skewed graph with hubs, a sample of its sources: the
        # baseline the benchmark compares the batched forms with.
        {"name": "plain_rmat15_s2048", "kind": "bc", "family": "rmat", "scale": 15, "form": "plain", "sources": 2048},
        # A large-diameter graph (a ring lattice with few shortcuts, tens of
        # levels of a few hundred vertices each), as road and grid-like graphs
        # are: many short launches per batch.
        {"name": "sparse_ring6001", "kind": "bc", "family": "ws", "n": 6001, "p": 0.005, "form": "sparse", "batch": 256},
        # The headline: every source of RMAT-16, batches of 256.
        {"name": "hybrid_rmat16", "kind": "bc", "family": "rmat", "scale": 16, "form": "hybrid", "batch": 256},
        # Edge betweenness beside the vertex scores, batched, on a mid-sized
        # skewed graph.
        {"name": "edges_rmat13", "kind": "bc", "family": "rmat", "scale": 13, "form": "sparse", "batch": 256, "edges": True},
        # The dense graph of the algebraic method, all sources, batches of 512.
        {"name": "algebraic_er16384", "kind": "bc", "family": "er", "n": 16384, "degree": 256.0, "form": "algebraic",
         "batch": 512},
        # Small integer weights by products, one 0/1 matrix per weight, at a
        # size that is no multiple of a tile.
        {"name": "algebraic_er5003w4", "kind": "bc", "family": "er", "n": 5003, "degree": 128.0, "form": "algebraic",
         "batch": 512, "wmax": 4},
        # Weights 1..255 on a skewed graph, a sample of its sources: the
        # bucketed shortest-path sweep.
        {"name": "weighted_rmat16_s1024", "kind": "bc", "family": "rmat", "scale": 16, "form": "auto", "wmax": 255,
         "sources": 1024},
        # Many uneven small-world graphs in one launch, the benchmark's ws4096
        # recipe (n uniform in 64..4096) with fewer graphs.
        {"name": "many_ws_256", "kind": "many", "count": 256, "nmin": 64, "nmax": 4096},
        # Very many tiny graphs (molecule-sized): a launch whose units are a
        # few wavefronts' work each.
        {"name": "many_small_3000", "kind": "many", "count": 3000, "nmin": 16, "nmax": 128},
        # Algorithm 2 over all ordered pairs, FP64, from the batched forward's
        # distances and counts.
        {"name": "allpairs_er6001", "kind": "allpairs", "family": "er", "n": 6001, "degree": 64.0, "form": "algebraic",
         "batch": 512},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sssp", "plain", "ring", "hybrid", "edges", "algebraic", "algebraic-w", "weighted", "many",
                       "many-small", "allpairs", "sampled"])
    if kind == "sssp":
        n = _log_int(rng, 40, 20000)
        return {"kind": "sssp", "family": "er+tree", "n": n, "degree": rng.uniform(2.0, 24.0),
                "count": min(n, _log_int(rng, 1, 64)), "form": rng.choice(["auto", "plain"])}
    if kind == "plain":
        if rng.random() < 0.5:
            return {"kind": "bc", "family": "er+tree", "n": _log_int(rng, 100, 4000), "degree": rng.uniform(2.0, 24.0),
                    "form": "plain"}
        return {"kind": "bc", "family": "rmat", "scale": rng.randint(10, 15), "form": "plain",
                "sources": _log_int(rng, 16, 2048)}
    if kind == "ring":
        return {"kind": "bc", "family": "ws", "n": _log_int(rng, 500, 6001), "p": math.exp(rng.uniform(math.log(0.004), math.log(0.1))),
                "form": "sparse", "batch": rng.choice([128, 256, 512])}
    if kind == "hybrid":
        return {"kind": "bc", "family": "rmat", "scale": rng.randint(11, 16), "form": rng.choice(["hybrid", "sparse"]),
                "batch": rng.choice([256, 512])}
    if kind == "edges":
        return {"kind": "bc", "family": "rmat", "scale": rng.randint(10, 14), "form": rng.choice(["hybrid", "sparse"]),
                "batch": 256, "edges": True}
    if kind == "algebraic":
        n = _log_int(rng, 1000, 16384)
        return {"kind": "bc", "family": "er", "n": n, "degree": rng.uniform(0.004, 0.016) * n + 8.0,
                "form": rng.choice(["algebraic", "hybrid"]), "batch": rng.choice([256, 512])}
    if kind == "algebraic-w":
        n = _log_int(rng, 1000, 7000)
        return {"kind": "bc", "family": "er", "n": n, "degree": rng.uniform(0.01, 0.03) * n + 8.0, "form": "algebraic",
                "batch": rng.choice([256, 512]), "wmax": rng.randint(2, 8)}
    if kind == "weighted":
        return {"kind": "bc", "family": "rmat", "scale": rng.randint(10, 16), "form": "auto",
                "wmax": rng.choice([10, 100, 255]), "sources": _log_int(rng, 16, 1024)}
    if kind == "many":
        return {"kind": "many", "count": _log_int(rng, 16, 256), "nmin": 64, "nmax": rng.choice([1500, 4096])}
    if kind == "many-small":
        lo = rng.randint(8, 40)
        return {"kind": "many", "count": _log_int(rng, 200, 3000), "nmin": lo, "nmax": lo + rng.randint(10, 200)}
    if kind == "allpairs":
        n = _log_int(rng, 500, 6001)
        return {"kind": "allpairs", "family": "er", "n": n, "degree": rng.uniform(8.0, 64.0),
                "form": rng.choice(["algebraic", "sparse", "plain"]), "batch": rng.choice([256, 512])}
    return {"kind": "sampled", "family": "rmat", "scale": rng.randint(11, 16), "form": "auto",
            "count": _log_int(rng, 1, 1024)}


# ---- inputs --------------------------------------------------------------------------

@functools.lru_cache(maxsize=2)
def _rmat(scale):
    return gg.rmat(scale, 16, gg.workload_seed(1))


def _graph(case, seed):
    fam = case["family"]
    if fam == "er":
        g = gg.erdos_renyi(case["n"], case["degree"], seed, lcc=False)
    elif fam == "er+tree":
        g = gg.er_plus_tree(case["n"], case["degree"], seed)
    elif fam == "ws":
        g = gg.watts_strogatz(case["n"], 6, case["p"], seed)
    else:
        # one R-MAT draw per scale (its largest component's size depends on the
        # draw), renumbered at random
        g = _rmat(case["scale"])
        g = g.relabel(np.random.RandomState(seed % (1 << 32)).permutation(g.n))
    if case.get("wmax"):
        g = gg.with_uniform_weights(g, seed, 1, case["wmax"])
    return g


def _many(case, seed):
    sizes = np.random.RandomState(case["count"]).randint(case["nmin"], case["nmax"] + 1, case["count"])
    return [gg.watts_strogatz(int(n), 6, 0.1, seed * 100003 + i) for i, n in enumerate(sizes)]


def _sources(case, seed, n):
    """The sampled sources, or None for every vertex."""
    k = case.get("sources") or case.get("count")
    return gg.sample_sources(n, min(k, n), seed + 1) if k else None


def prepare(case, seed):
    """The graph's context (and the source and sample lists) a program keeps."""
    if case["kind"] == "many":
        return {"case": case, "ctx": bcgpu.BC(_many(case, seed))}
    g = _graph(case, seed)
    batch = 0 if case["form"] in ("auto", "plain") else case.get("batch", 0)
    ctx = bcgpu.BC(g, form=case["form"], batch=batch, edges=bool(case.get("edges")))
    state = {"case": case, "ctx": ctx, "sources": _sources(case, seed, g.n)}
    if case["kind"] == "sampled":
        # the section's sample size, ceil(sqrt(n) ln n)
        state["sample"] = gg.sample_sources(g.n, min(g.n, math.ceil(math.sqrt(g.n) * math.log(g.n))), seed + 2)
        state["out"] = torch.empty((state["sources"].size, g.n), dtype=torch.int32, device=DEV)
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "sssp":
        return list(ctx.sssp(state["sources"]))
    if kind == "allpairs":
        return ctx.all_pairs()
    if kind == "sampled":
        return ctx.sampled_distances(state["sources"], state["sample"], out=state["out"])
    ctx.reset()
    ctx.run(state.get("sources"))
    if case.get("edges"):
        return [ctx.read(), ctx.read_edges()]
    return ctx.read()


# ---- what a pass cannot do without -----------------------------------------------------

def _shape(case):
    """(vertices, arcs, sources) a case is expected to have."""
    if case["kind"] == "many":
        lo, hi = case["nmin"], case["nmax"]
        mean = (lo + hi) / 2.0
        square = mean * mean + (hi - lo) * (hi - lo) / 12.0
        # sources x arcs summed over the graphs is count * 6 * E[n^2]
        return case["count"] * mean, 6.0 * case["count"] * mean, square / mean
    if case["family"] == "rmat":
        n = 0.72 * (1 << case["scale"])
        arcs = 28.0 * (1 << case["scale"])
    else:
        n = float(case["n"])
        arcs = n * (6.0 if case["family"] == "ws" else case["degree"])
    k = case.get("sources") or case.get("count")
    return n, arcs, float(min(k, n)) if k else n


def work(case):
    """The graph read once, the results written once; one multiply-add per
    (source, arc) in each sweep direction the call has."""
    n, arcs, s = _shape(case)
    graph = 4.0 * (n + 1.0) + arcs * (5.0 if case.get("wmax") else 4.0)
    kind = case["kind"]
    if kind == "sssp":
        return {"bytes": graph + 20.0 * s * n, "flops": 4.0 * s * arcs}
    if kind == "sampled":
        return {"bytes": graph + 4.0 * s * n, "flops": 2.0 * s * arcs}
    out = 8.0 * n + (8.0 * arcs if case.get("edges") else 0.0)
    return {"bytes": graph + out, "flops": (6.0 if case.get("edges") else 4.0) * s * arcs}


# ---- the same results in 64 bits by plain torch -----------------------------------------

def _level_sweeps(mats, src, with_edges=False):
    """Brandes's two sweeps for the columns `src`, levels by products in FP64.

    mats[c - 1] is the 0/1 matrix of the edges of weight c (dense or sparse
    CSR); distances are levels.  Returns distances, counts, dependencies (each
    [n, S]) and, for unit weights, the n x n sums of the per-arc terms.
    """
    M, n, S = len(mats), mats[0].shape[0], src.numel()
    f8 = dict(dtype=torch.float64, device=DEV)
    cols = torch.arange(S, device=DEV)
    sigma = torch.zeros((n, S), **f8)
    sigma[src, cols] = 1.0
    dist = torch.full((n, S), -1, dtype=torch.int32, device=DEV)
    dist[src, cols] = 0
    level, empty = 0, 0
    while empty < M:
        level += 1
        x = torch.zeros((n, S), **f8)
        for c in range(1, min(M, level) + 1):
            x += mats[c - 1] @ torch.where(dist == level - c, sigma, 0.0)
        new = (x > 0) & (dist < 0)
        empty = 0 if bool(new.any()) else empty + 1
        dist[new] = level
        sigma[new] = x[new]
    top = int(dist.max())
    delta = torch.zeros((n, S), **f8)
    coef = torch.zeros((n, S), **f8)  # (1 + delta) / sigma of the levels done
    terms = torch.zeros((n, n), **f8) if with_edges else None
    for l in range(top, -1, -1):
        at = dist == l
        y = torch.zeros((n, S), **f8)
        for c in range(1, min(M, top - l) + 1):
            y += mats[c - 1] @ torch.where(dist == l + c, coef, 0.0)
        delta = torch.where(at, sigma * y, delta)
        coef = torch.where(at, (1.0 + delta) / torch.where(at, sigma, 1.0), coef)
        if with_edges and l < top:
            terms += torch.where(at, sigma, 0.0) @ torch.where(dist == l + 1, coef, 0.0).T.contiguous()
    return dist, sigma, delta, terms


def _relaxed_sweeps(g, src):
    """The sweeps by arc relaxation to a fixed point, for many weights."""
    n, S = g.n, src.numel()
    u = torch.from_numpy(np.repeat(np.arange(n), np.diff(g.row_ptr))).to(DEV)
    v = torch.from_numpy(g.col.astype(np.int64)).to(DEV)
    w = torch.from_numpy(g.weight.astype(np.int32)).to(DEV)[:, None]
    cols = torch.arange(S, device=DEV)
    inf = 1 << 29
    dist = torch.full((n, S), inf, dtype=torch.int32, device=DEV)
    dist[src, cols] = 0
    while True:
        nxt = dist.clone().index_reduce_(0, v, dist[u] + w, "amin")
        if torch.equal(nxt, dist):
            break
        dist = nxt
    dag = (dist[u] + w == dist[v]) & (dist[u] < inf)
    start = torch.zeros((n, S), dtype=torch.float64, device=DEV)
    start[src, cols] = 1.0
    sigma = start
    while True:
        nxt = start.clone().index_add_(0, v, torch.where(dag, sigma[u], 0.0))
        if torch.equal(nxt, sigma):
            break
        sigma = nxt
    ratio = torch.where(dag, sigma[u] / sigma[v].clamp(min=1.0), 0.0)
    delta = torch.zeros((n, S), dtype=torch.float64, device=DEV)
    while True:
        nxt = torch.zeros_like(delta).index_add_(0, u, ratio * (1.0 + delta[v]))
        if bool(((nxt - delta).abs() <= 1e-15 * nxt).all()):
            return nxt
        delta = nxt


def _matrices(g):
    """One 0/1 matrix per weight, dense where that fits easily."""
    rp = torch.from_numpy(g.row_ptr.astype(np.int64)).to(DEV)
    col = torch.from_numpy(g.col.astype(np.int64)).to(DEV)
    weight = torch.ones(col.numel(), dtype=torch.int64, device=DEV) if g.weight is None \
        else torch.from_numpy(g.weight.astype(np.int64)).to(DEV)
    if g.weight is None and g.n > 20000:
        return [torch.sparse_csr_tensor(rp, col, torch.ones(col.numel(), dtype=torch.float64, device=DEV), (g.n, g.n))]
    row = torch.repeat_interleave(torch.arange(g.n, device=DEV), rp[1:] - rp[:-1])
    out = []
    for c in range(1, int(weight.max()) + 1):
        a = torch.zeros((g.n, g.n), dtype=torch.float64, device=DEV)
        a[row[weight == c], col[weight == c]] = 1.0
        out.append(a)
    return out


def _score(delta, src):
    cols = torch.arange(src.numel(), device=DEV)
    delta = delta.clone()
    delta[src, cols] = 0.0
    return delta.sum(1)


def _many_scores(graphs):
    """All-source scores of small graphs, padded and taken in groups of one size."""
    out = [None] * len(graphs)
    order = sorted(range(len(graphs)), key=lambda i: graphs[i].n)
    at = 0
    while at < len(order):
        size = graphs[order[min(len(order), at + 64) - 1]].n
        take = max(1, min(256, int(2.0e8 / (size * size))))
        ids = order[at:at + take]
        at += len(ids)
        N = max(graphs[i].n for i in ids)
        A = torch.zeros((len(ids), N, N), dtype=torch.float64, device=DEV)
        sigma = torch.zeros_like(A)
        dist = torch.full(A.shape, -1, dtype=torch.int32, device=DEV)
        for k, i in enumerate(ids):
            g = graphs[i]
            row = torch.from_numpy(np.repeat(np.arange(g.n), np.diff(g.row_ptr))).to(DEV)
            A[k, row, torch.from_numpy(g.col.astype(np.int64)).to(DEV)] = 1.0
            own = torch.arange(g.n, device=DEV)
            sigma[k, own, own] = 1.0
            dist[k, own, own] = 0
        level = 0
        while True:
            x = torch.bmm(A, torch.where(dist == level, sigma, 0.0))
            new = (x > 0) & (dist < 0)
            if not bool(new.any()):
                break
            level += 1
            dist[new] = level
            sigma[new] = x[new]
        delta = torch.zeros_like(A)
        for l in range(level - 1, 0, -1):
            up = dist == l + 1
            y = torch.bmm(A, torch.where(up, (1.0 + delta) / torch.where(up, sigma, 1.0), 0.0))
            delta = torch.where(dist == l, sigma * y, delta)
        score = delta.sum(2)
        for k, i in enumerate(ids):
            out[i] = score[k, :graphs[i].n].cpu().numpy()
    return np.concatenate(out)


def exact(case, seed):
    """The case's outputs in 64 bits; None where they are whole numbers that
    depend on the drawn sample, or would take too long."""
    kind = case["kind"]
    if kind == "sampled":
        return None
    if kind == "many":
        return _many_scores(_many(case, seed))
    g = _graph(case, seed)
    sources = _sources(case, seed, g.n)
    every = torch.arange(g.n, device=DEV) if sources is None else torch.from_numpy(sources.astype(np.int64)).to(DEV)
    if case.get("wmax") and case["form"] == "auto":
        step = max(1, int(1.5e8 / max(g.nnz, 1)))
        return sum(_score(_relaxed_sweeps(g, every[i:i + step]), every[i:i + step])
                   for i in range(0, every.numel(), step)).cpu().numpy()
    mats = _matrices(g)
    if kind == "sssp":
        dist, sigma, delta, _ = _level_sweeps(mats, every)
        rows = [t.T.contiguous().cpu().numpy() for t in (dist, sigma, delta)]
        return [rows[0], rows[1].astype(np.uint64), rows[2]]
    step = max(256, min(4096, int(6.0e7 / g.n)))
    score = torch.zeros(g.n, dtype=torch.float64, device=DEV)
    terms = 0.0
    for i in range(0, every.numel(), step):
        part = every[i:i + step]
        _, _, delta, t = _level_sweeps(mats, part, bool(case.get("edges")))
        score += _score(delta, part)
        if case.get("edges"):
            terms = terms + t
    if not case.get("edges"):
        return score.cpu().numpy()
    row = torch.from_numpy(np.repeat(np.arange(g.n), np.diff(g.row_ptr))).to(DEV)
    col = torch.from_numpy(g.col.astype(np.int64)).to(DEV)
    return [score.cpu().numpy(), (terms[row, col] + terms[col, row]).cpu().numpy()]

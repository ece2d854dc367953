"""How the per-source sweeps deal a chunk's arcs to waves: chunk totals around
a thread's one arc and a full round, rows of one arc and of thousands, and the
sizes where the LDS routes end."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def spider(legs, length):
    """Legs of `length` vertices around a centre: levels of rows of two arcs."""
    v = 1 + np.arange(legs * length)
    return gg.from_edges(1 + legs * length, np.where((v - 1) % length == 0, 0, v - 1), v)


GRAPHS = {f"star{d}": (lambda d=d: gg.star(d + 1)) for d in (511, 512, 513, 1024, 1025, 2048, 4095, 4096, 4097, 8193)}
GRAPHS |= {
    "spider": lambda: spider(2500, 4),
    "tree": lambda: gg.random_tree(15000, 3),
    "bipartite": lambda: gg.complete_bipartite(700, 40),
    "mixed": lambda: gg.disjoint_union(gg.star(5000), spider(700, 3), gg.complete(150), gg.path(1)),
    "plain-two-per-unit": lambda: gg.er_plus_tree(71068, 2.0, 2),
    "plain-last": lambda: gg.er_plus_tree(142204, 2.0, 4),
    "weighted-two-per-unit": lambda: gg.er_plus_tree(37704, 2.0, 2),
    "weighted-last": lambda: gg.er_plus_tree(75448, 2.0, 4),
}


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0)))


@pytest.mark.parametrize("grid", [0, 64])  # 64: the sweeps with their state in memory
@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_arcs_dealt(gpu_lib, name, weights, grid):
    g = GRAPHS[name]()
    if weights:
        g = gg.with_uniform_weights(g, 5, 1, 3)
    print(f"arc_deal {name} n={g.n} weights={weights} grid={grid}", flush=True)
    src = np.concatenate([[0, g.n - 1], gg.sample_sources(g.n, 20, 7)]).astype(np.int32)
    want = oracle.edge_bc(g, sources=src, threads=8)
    with gpu_lib.BC(g, form="plain", edges=True, grid=grid) as ctx:
        ctx.run(src)
        assert rel_err(ctx.read(), want[0]) <= 1e-12  # FP64 throughout
        assert rel_err(ctx.read_edges(), want[1]) <= 1e-12
        dist, sigma, _ = ctx.sssp(src[:2])
    for i in range(2):
        d, sg, _ = oracle.sssp_u64(g, int(src[i]))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)

"""Runs over every vertex whose leaves are folded into their neighbours'
sweeps: the same scores and the same depth as the same sources given as a list,
with few and many leaves per neighbour, batches handed back for their depth or
their counts, and components that are single edges or vertices."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def pendants(g, at):
    """g with one new leaf per entry of at, joined to that vertex."""
    row = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    keep = row < g.col
    leaves = g.n + np.arange(len(at))
    return gg.from_edges(g.n + len(at), np.concatenate([row[keep], at]), np.concatenate([g.col[keep], leaves]))


GRAPHS = {
    "hubs": lambda: gg.rmat(13, 16, 1),
    "star": lambda: gg.star(9000),
    "tree": lambda: gg.random_tree(9000, 3),
    "edges-and-points": lambda: gg.disjoint_union(*[gg.path(2)] * 2000, *[gg.path(3)] * 1500, *[gg.path(1)] * 99),
    # one leaf on most vertices, one of them the far end of a long path
    "deep": lambda: gg.disjoint_union(pendants(gg.er_plus_tree(6000, 4.0, 5), np.arange(0, 6000, 2)), gg.path(150)),
    # C(58, 29) = 3e16 paths: 64-bit counts
    "wide": lambda: gg.disjoint_union(pendants(gg.grid(30, 30), np.arange(900)), gg.star(7000)),
}


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0)))


@pytest.mark.parametrize("form,batch", [("sparse", 64), ("sparse", 256), ("algebraic", 256)])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_leaf_sources(gpu_lib, name, form, batch):
    g = GRAPHS[name]()
    print(f"leaf_sources {name} n={g.n} batch={batch} form={form}", flush=True)
    every = np.arange(g.n, dtype=np.int32)
    with gpu_lib.BC(g, form=form, batch=batch) as ctx:
        ctx.run(every)
        want, levels = ctx.read(), ctx.info().max_levels
    with gpu_lib.BC(g, form=form, batch=batch) as ctx:
        for _ in range(2):
            ctx.reset()
            ctx.run()
            # a count's c is rounded to FP32: one unit apart where the FP64
            # sums before it differ in their last bits
            assert rel_err(ctx.read(), want) <= 2.0**-23
            assert ctx.info().max_levels == levels
        ctx.run(every[:batch + 3])  # a list again: every weight is 1
        assert rel_err(ctx.read(), oracle.bc(g) + oracle.bc(g, sources=every[:batch + 3])) <= 1e-5


def test_lists_with_repeats(gpu_lib):
    g = GRAPHS["hubs"]()
    src = np.concatenate([gg.sample_sources(g.n, 700, 3), gg.sample_sources(g.n, 90, 4), np.full(50, 5)]).astype(np.int32)
    want = oracle.edge_bc(g, sources=src, threads=8)
    for edges in (False, True):
        with gpu_lib.BC(g, form="sparse", batch=256, edges=edges) as ctx:
            ctx.run(src)
            assert rel_err(ctx.read(), want[0]) <= 1e-5
            if edges:
                assert rel_err(ctx.read_edges(), want[1]) <= 1e-5


def test_leaf_sources_host_driven(gpu_lib):
    g = gg.rmat(13, 16, 2)
    want = oracle.bc(g)
    for kw in (dict(host_driven=True), dict(timing=True), dict(vertex_order="input")):
        with gpu_lib.BC(g, form="sparse", batch=256, **kw) as ctx:
            ctx.run()
            assert rel_err(ctx.read(), want) <= 1e-5

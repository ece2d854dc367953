"""The weighted sweep with its distances in LDS: the sizes where the workgroups
per compute unit and the route change, distances and counts at the limits where
a source is handed to the other sweep, DAG arcs past their room, hubs and edge
terms."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def tree(n, seed):
    return gg.with_uniform_weights(gg.er_plus_tree(n, 2.0, seed), seed, 1, 255)


def union(weight, *parts):
    return gg.with_constant_weight(gg.disjoint_union(*parts), weight)


GRAPHS = {
    "hubs": lambda: gg.with_uniform_weights(gg.rmat(13, 16, 1), 1, 1, 255),
    "few-weights": lambda: gg.with_uniform_weights(gg.rmat(13, 16, 2), 2, 1, 3),
    "two-per-unit": lambda: tree(37832, 3),
    "one-per-unit": lambda: tree(37833, 4),
    "last": lambda: tree(75704, 5),
    "past": lambda: tree(75705, 6),  # distances in memory
    "wide": lambda: union(7, gg.star(7200), gg.path(1), gg.grid(34, 34)),  # C(66,33) < 2^63
    "wide-1024": lambda: union(255, gg.star(40000), gg.path(3)),
    "far": lambda: union(255, gg.path(257), gg.path(258), gg.path(259)),  # ends 65280, 65535, 65790 apart
    "farthest": lambda: union(2, gg.path(32768), gg.path(2)),  # ends 65534 apart
    "mostly-far": lambda: union(255, gg.path(1500), gg.star(300)),
    "dense": lambda: union(9, gg.complete_bipartite(400, 400)),  # more DAG arcs than room
    "counts": lambda: union(3, gg.grid(34, 35), gg.star(30)),  # C(67,33) between 2^63 and 2^64
}


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0)))


@pytest.mark.parametrize("edges", [False, True])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_weighted_lds(gpu_lib, name, edges):
    g = GRAPHS[name]()
    print(f"weighted_lds {name} n={g.n} edges={edges}", flush=True)
    ends = np.array([0, g.n - 1], np.int32)  # ends of paths, corners of grids
    src = np.concatenate([ends, gg.sample_sources(g.n, 1700 if name == "mostly-far" else 60, 7)]).astype(np.int32)
    want = oracle.edge_bc(g, sources=src, threads=8)
    with gpu_lib.BC(g, edges=edges) as ctx:
        for turn in range(2):  # the second turn knows what the first handed back
            ctx.reset()
            ctx.run(src)
            assert rel_err(ctx.read(), want[0]) <= 1e-12  # FP64 throughout
            if edges:
                assert rel_err(ctx.read_edges(), want[1]) <= 1e-12
        dist, sigma, delta = ctx.sssp(src[:3])
    for i in range(3):
        d, sg, dl = oracle.sssp_u64(g, int(src[i]))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)
        assert rel_err(delta[i], dl) <= 1e-12


def test_weighted_lds_overflow(gpu_lib):
    g = union(5, gg.star(300), gg.grid(35, 35))  # C(68,34) > 2^64 - 1
    with gpu_lib.BC(g) as ctx:
        ctx.run(np.array([g.n - 1], np.int32))
        with pytest.raises(gpu_lib.BCError) as ei:
            ctx.read()
        assert ei.value.status == gpu_lib.BC_ERR_OVERFLOW
        ctx.reset()
        ctx.run(np.array([5], np.int32))
        assert rel_err(ctx.read(), oracle.bc(g, sources=np.array([5], np.int32))) <= 1e-12


def test_a_few_far_sources_decide_nothing(gpu_lib):
    """A far source takes a launch of either sweep, until most of at least 256
    sources were far; a near one takes one launch."""
    g = union(255, gg.path(600), gg.star(300))  # a path's vertices are up to 152745 apart
    far, near = np.arange(100, dtype=np.int32), np.arange(600, 650, dtype=np.int32)
    sums, launches = np.zeros(g.n), 0
    with gpu_lib.BC(g, timing=1) as ctx:
        # by the last far hundred 202 of 302 sources have been far
        for src, new in ((far[:1], 2), (far[:1], 2), (near, 1), (far, 2), (near, 1), (far, 2), (far[:1], 1),
                         (near, 1), (far, 1)):
            print(f"weighted_lds far={src.size and src[0] < 600} count={src.size}", flush=True)
            ctx.run(src)
            launches += new
            assert ctx.timing("weighted_sweep")[1] == launches
            sums += oracle.bc(g, sources=src)
        assert rel_err(ctx.read(), sums) <= 1e-12

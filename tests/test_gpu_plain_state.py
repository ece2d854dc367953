"""The plain form's sweep with its states in LDS: the sizes where the
workgroups per compute unit and the route change, few and many sources, hubs,
edge terms, the readout and the count limits."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

GRAPHS = {
    "hubs": lambda: gg.rmat(14, 16, 1),
    "parts": lambda: gg.disjoint_union(gg.star(7200), gg.path(900), gg.path(1), gg.grid(34, 34)),  # C(66,33) = 7.2e18
    "two-per-unit": lambda: gg.er_plus_tree(71580, 2.0, 2),
    "one-per-unit": lambda: gg.er_plus_tree(71581, 2.0, 3),
    "last": lambda: gg.er_plus_tree(143228, 2.0, 4),
    "past": lambda: gg.er_plus_tree(143229, 2.0, 5),  # states in memory
}


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0)))


@pytest.mark.parametrize("edges", [False, True])
@pytest.mark.parametrize("count", [3, 300])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_plain_states(gpu_lib, name, count, edges):
    g = GRAPHS[name]()
    print(f"plain_state {name} n={g.n} count={count} edges={edges}", flush=True)
    src = gg.sample_sources(g.n, count, 7)
    if name == "parts":
        src[0], src[1] = 8101, g.n - 1  # the single vertex, a corner of the grid
    want = oracle.edge_bc(g, sources=src, threads=8)
    with gpu_lib.BC(g, form="plain", edges=edges) as ctx:
        ctx.run(src)
        assert rel_err(ctx.read(), want[0]) <= 1e-12  # FP64 throughout
        if edges:
            assert rel_err(ctx.read_edges(), want[1]) <= 1e-12
        dist, sigma, delta = ctx.sssp(src[:3])
    for i in range(3):
        d, sg, dl = oracle.sssp_u64(g, int(src[i]))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)
        assert rel_err(delta[i], dl) <= 1e-12


def test_plain_states_overflow(gpu_lib):
    g = gg.disjoint_union(gg.star(7200), gg.grid(35, 35))  # C(68,34) > 2^64 - 1
    with gpu_lib.BC(g, form="plain") as ctx:
        ctx.run(np.array([g.n - 1], np.int32))
        with pytest.raises(gpu_lib.BCError) as ei:
            ctx.read()
        assert ei.value.status == gpu_lib.BC_ERR_OVERFLOW
        ctx.reset()
        ctx.run(np.array([5], np.int32))
        assert rel_err(ctx.read(), oracle.bc(g, sources=np.array([5], np.int32))) <= 1e-12

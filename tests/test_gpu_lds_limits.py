"""The per-source sweeps at the sizes where their LDS routes change, derived
from the LDS the kernels hold besides a vertex's state, and the plain sweep with
its state in memory on rows of every kind, in graphs past the last of those
sizes."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from test_gpu_arc_deal import spider

pytestmark = pytest.mark.gpu

LDS = 160 << 10


def fixed(threads, arcs, sums):
    """A chunk of `threads` vertices, the waves' arc bits, the chunk's sums, the rest."""
    waves = threads // 64
    return 4 * (3 * threads + 1 + waves) + waves * 2 * arcs * 4 + sums * threads + 64


# a byte of state a vertex, in words; a 16-bit distance, eight at a time
PLAIN_TWO = (LDS - 2 * fixed(512, 8, 8)) // 2 // 4 * 4
PLAIN_LAST = (LDS - fixed(1024, 8, 8)) // 4 * 4
WEIGHTED_TWO = (LDS - 2 * fixed(512, 4, 0)) // 2 // 16 * 8
WEIGHTED_LAST = (LDS - fixed(1024, 4, 0)) // 16 * 8


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0)))


@pytest.mark.parametrize("count", [3, 300])
@pytest.mark.parametrize("n", [PLAIN_TWO, PLAIN_TWO + 1, PLAIN_LAST, PLAIN_LAST + 1])
def test_plain_limits(gpu_lib, n, count):
    import torch
    g = gg.er_plus_tree(n, 2.0, 2)
    print(f"lds_limits plain n={n} count={count}", flush=True)
    src = gg.sample_sources(n, count, 7)
    bc, eb = oracle.edge_bc(g, sources=src, threads=8)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    groups, each = (2048, 28) if n > PLAIN_LAST else (2 * cus if n <= PLAIN_TWO else cus, 16)
    with gpu_lib.BC(g, form="plain", edges=True) as ctx:
        rest = ctx.info().device_bytes - groups * each * n  # the graph and the edge terms
        assert 0 < rest < 1000 * n, "workspaces of another route"
        ctx.run(src)
        assert rel_err(ctx.read(), bc) <= 1e-12  # FP64 throughout
        assert rel_err(ctx.read_edges(), eb) <= 1e-12
        dist, sigma, delta = ctx.sssp(src[:2])
    for i in range(2):
        d, sg, dl = oracle.sssp_u64(g, int(src[i]))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)
        assert rel_err(delta[i], dl) <= 1e-12


@pytest.mark.parametrize("n", [WEIGHTED_TWO, WEIGHTED_TWO + 1, WEIGHTED_LAST, WEIGHTED_LAST + 1])
def test_weighted_limits(gpu_lib, n):
    far = 300  # a path's ends are 76245 apart, past 16 bits
    parts = gg.disjoint_union(gg.path(far), gg.er_plus_tree(n - far, 2.0, 3))
    weights = np.full(parts.col.size, 255, np.uint32)
    weights[parts.row_ptr[far]:] = gg.with_uniform_weights(parts, 4, 1, 255).weight[parts.row_ptr[far]:]
    g = gg.Graph(parts.n, parts.row_ptr, parts.col, weights, "path and tree")
    print(f"lds_limits weighted n={n}", flush=True)
    src = np.concatenate([[0], far + gg.sample_sources(n - far, 300, 7)]).astype(np.int32)
    want = oracle.bc(g, sources=src, threads=8)
    with gpu_lib.BC(g, timing=1) as ctx:
        ctx.run(src)
        # the far source goes on to the other sweep, where that is not the first
        assert ctx.timing("weighted_sweep")[1] == (1 if n > WEIGHTED_LAST else 2)
        assert rel_err(ctx.read(), want) <= 1e-12  # FP64 throughout
        dist, sigma, _ = ctx.sssp(src[:2])
    for i in range(2):
        d, sg, _ = oracle.sssp_u64(g, int(src[i]))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)


SHAPES = {f"star{d}": (lambda d=d: gg.star(d + 1)) for d in (1, 255, 256, 257, 2047, 2048, 2049, 8193)}
SHAPES |= {
    "spider": lambda: spider(2500, 4),
    "bipartite": lambda: gg.complete_bipartite(700, 40),
    "hubs": lambda: gg.rmat(12, 16, 3),
    "mixed": lambda: gg.disjoint_union(gg.star(5000), spider(700, 3), gg.complete(150), gg.path(300)),
}


@pytest.mark.parametrize("grid", [0, 64])
@pytest.mark.parametrize("name", list(SHAPES))
def test_plain_states_in_memory(gpu_lib, name, grid):
    """Vertices without edges take the graph past the LDS, whatever its shape."""
    shape = SHAPES[name]()
    n = PLAIN_LAST + 1
    row_ptr = np.concatenate([shape.row_ptr, np.full(n - shape.n, shape.row_ptr[-1])]).astype(np.int32)
    g = gg.Graph(n, row_ptr, shape.col, None, name)
    print(f"lds_limits memory {name} grid={grid}", flush=True)
    src = np.concatenate([[0, shape.n - 1, n - 1], gg.sample_sources(shape.n, min(shape.n, 20), 7)]).astype(np.int32)
    want = oracle.edge_bc(g, sources=src, threads=8)
    with gpu_lib.BC(g, form="plain", edges=True, grid=grid) as ctx:
        ctx.run(src)
        assert rel_err(ctx.read(), want[0]) <= 1e-12  # FP64 throughout
        assert rel_err(ctx.read_edges(), want[1]) <= 1e-12
        dist, sigma, _ = ctx.sssp(src[:3])
    for i in range(3):
        d, sg, _ = oracle.sssp_u64(g, int(src[i]))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)

"""Products over few tiles (forward tiles shared by two blocks, backward
blocks of 64 rows) and just past the rules: fewer non-empty stages than blocks, counts of several limbs,
weight classes; forms agree with the oracle and batches replayed with
batches driven from the host."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

CASES = {
    "short-k": (lambda: gg.erdos_renyi(3800, 12.0, 1, lcc=False), 256),  # K = 3840: one block
    "k4096": (lambda: gg.erdos_renyi(3900, 12.0, 1, lcc=False), 256),
    # up to nine limbs, two or three non-empty stages a level
    "limbs": (lambda: gg.disjoint_union(gg.grid(31, 31), gg.star(3200)), 256),
    "tiles160": (lambda: gg.erdos_renyi(5003, 20.0, 2, lcc=False), 512),
    "tiles256": (lambda: gg.erdos_renyi(8190, 16.0, 3, lcc=False), 512),
    "tiles264": (lambda: gg.erdos_renyi(8200, 16.0, 4, lcc=False), 512),  # one block
    "classes": (lambda: gg.with_uniform_weights(gg.erdos_renyi(1500, 30.0, 5, lcc=False), 6, 1, 4), 512),
    "sparse-classes": (lambda: gg.with_uniform_weights(gg.path(300), 7, 1, 8), 256),
}


@pytest.mark.parametrize("name", list(CASES))
def test_split_products(gpu_lib, name):
    make, batch = CASES[name]
    g = make()
    print(f"split_products {name} n={g.n}", flush=True)
    src = gg.sample_sources(g.n, min(g.n, 2 * batch + 77), 8)  # three batches, the last ragged
    want = oracle.bc(g, sources=src, threads=8)
    for host in (False, True):
        with gpu_lib.BC(g, form="algebraic", batch=batch, host_driven=host) as ctx:
            for times in (1, 2):
                ctx.run(src)
                got = ctx.read()
                err = np.max(np.abs(got - times * want) / np.maximum(times * want, 1.0))
                assert err <= 1e-5  # FP32 c(v)
            dist, sigma, _ = ctx.sssp(src[:3])
    for i in range(3):
        d, sg, _ = oracle.sssp_u64(g, int(src[i]))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)

"""The many-graph group sweep at the sizes where its layout changes: class
edges, ragged groups and bursts, sums at the edge of 32 bits, dense graphs on
both sides of the burst limit."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0))) if y.size else 0.0


CASES = {
    # one vertex, one edge, and both sides of the small-graph class
    "class-edges": lambda: [gg.path(1), gg.path(2)] + [gg.watts_strogatz(n, 6, 0.1, n) for n in (255, 256, 257)],
    # degrees 7, 8 and 9: one burst short, full, and one column over
    "burst-edges": lambda: [gg.complete(8), gg.complete(9), gg.complete(10), gg.star(9), gg.star(10), gg.star(3000)],
    # rows of more than eight bursts beside short ones in a wave
    "hubs": lambda: [gg.rmat(12, 16, 7), gg.rmat(8, 16, 8)],
    # unreached vertices, isolated ones among them
    "disconnected": lambda: [gg.disjoint_union(gg.path(300), gg.cycle(7), gg.path(1)), gg.disjoint_union(gg.path(1), gg.star(5))],
    # C(34,17) = 2.3e9: no 32-bit sum wraps, but a neighbour's count times the
    # degree could; C(36,18) = 9.1e9 wraps and goes to the full sweep
    "counts": lambda: [gg.grid(18, 18), gg.grid(19, 19)],
    # 61600 bursts (group sweep) and 80000 (full sweep)
    "dense": lambda: [gg.complete(700), gg.complete(800)],
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("unit", [0, 64])
def test_group_sweep_edges(gpu_lib, name, unit):
    gs = CASES[name]()
    print(f"many_groups {name} unit={unit}", flush=True)
    want = np.concatenate([oracle.bc(g, threads=8) for g in gs])
    with gpu_lib.BC(gs, batch=unit) as ctx:
        for times in (1, 2):  # the second run is a replay
            ctx.run()
            # c(v) is FP32: the batched forms' tolerance
            assert rel_err(ctx.read(), times * want) <= 1e-5

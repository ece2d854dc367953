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


def fans(*widths, then=0):
    """A chain of fans: the count multiplies by each width; `then` more edges."""
    edges, at, new = [], 0, 1
    for w in widths:
        mids = list(range(new, new + w))
        new += w + 1
        edges += [(at, x) for x in mids] + [(x, new - 1) for x in mids]
        at = new - 1
    for _ in range(then):
        edges.append((at, new))
        at, new = new, new + 1
    return edges, at, new


def wrapping_sum(more=0):
    """From vertex 0 a vertex has predecessors with 255 * 2^24 and 2^25
    shortest paths (times 2^more): either is below 2^32, their sum is not, and
    the smaller one is below 2^32 over the largest degree."""
    a, ea, na = fans(15, 17, *[2] * (24 + more))
    b, eb, nb = fans(*[2] * (25 + more), then=2)
    move = lambda x: 0 if x == 0 else x + na - 1  # noqa: E731
    e = a + [(move(x), move(y)) for x, y in b]
    n = na + nb - 1
    e += [(ea, n), (move(eb), n), (n, n + 1)]
    u, v = np.array(e).T
    return gg.from_edges(n + 2, u, v, name="wrapping-sum")


CASES = {
    "wrapping-sum": lambda: [wrapping_sum()] * 40,
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

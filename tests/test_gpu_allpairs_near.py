"""Algorithm 2's near triples (an end next to the vertex) and its choice of
matrices: distances up to and past the byte matrix's, with and without far
triples, column tiles at their edges, hubs, unreachable parts."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

GRAPHS = {
    "diameter1": lambda: gg.complete(65),
    "diameter2": lambda: gg.star(700),
    "diameter3": lambda: gg.er_plus_tree(255, 40.0, 2),
    "tile": lambda: gg.er_plus_tree(256, 6.0, 3),
    "tile-over": lambda: gg.er_plus_tree(257, 6.0, 4),
    "bytes-last": lambda: gg.cycle(500),  # distances up to 250
    "bytes-past": lambda: gg.path(300),
    "parts": lambda: gg.disjoint_union(gg.path(1), gg.cycle(9), gg.star(40), gg.grid(5, 6)),
    "hubs": lambda: gg.rmat(11, 16, 5),
}


@pytest.mark.parametrize("form", ["plain", "sparse", "algebraic"])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_near_and_far(gpu_lib, name, form):
    g = GRAPHS[name]()
    print(f"allpairs {form} {name} n={g.n}", flush=True)
    want = oracle.bc(g, threads=8)
    with gpu_lib.BC(g, form=form) as ctx:
        got = ctx.all_pairs()
    # FP64 sums of FP64 terms, as Algorithm 2's other tests
    assert float(np.max(np.abs(got - want) / np.maximum(np.abs(want), 1.0))) <= 1e-12

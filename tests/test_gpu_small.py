"""Sweeps of small graphs with their state in LDS: sizes at the edges of the
route and of a group, hubs, depth up to n, counts near the limits, and the
readout, against the oracle."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

GRAPHS = {
    "one": lambda: gg.path(1),
    "two": lambda: gg.path(2),
    "isolated": lambda: gg.disjoint_union(gg.path(1), gg.cycle(9), gg.path(1), gg.path(70)),
    "deep": lambda: gg.path(2100),
    "hubs": lambda: gg.rmat(12, 16, 3),
    "counts": lambda: gg.grid(34, 34),  # C(66,33) = 7.2e18
    "last": lambda: gg.er_plus_tree(7084, 3.0, 5),  # the largest that fits
    "past": lambda: gg.er_plus_tree(7085, 3.0, 5),
}


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0))) if y.size else 0.0


@pytest.mark.parametrize("name", list(GRAPHS))
def test_plain_small(gpu_lib, name):
    g = GRAPHS[name]()
    print(f"small plain {name} n={g.n}", flush=True)
    src = gg.sample_sources(g.n, min(g.n, 700), 11)  # groups of three, the last ragged
    src = np.concatenate([src, src[:1]]).astype(np.int32)  # a multiset
    want = oracle.bc(g, sources=src, threads=8)
    with gpu_lib.BC(g, form="plain") as ctx:
        ctx.run(src)
        assert rel_err(ctx.read(), want) <= 1e-12  # FP64 throughout
        ctx.run(src[:1])
        assert rel_err(ctx.read(), want + oracle.bc(g, sources=src[:1])) <= 1e-12
        pick = src[:: max(1, src.size // 5)]
        dist, sigma, delta = ctx.sssp(pick)
    for i, s in enumerate(pick):
        d, sg, dl = oracle.sssp_u64(g, int(s))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)
        assert rel_err(delta[i], dl) <= 1e-12


def test_plain_small_overflow(gpu_lib):
    """Paths of 255 * 2^56 and 2^57 meet: their sum passes 2^64, whichever of
    the two is added last."""
    from test_gpu_many_groups import wrapping_sum
    for _ in range(8):
        with gpu_lib.BC(wrapping_sum(32), form="plain") as ctx:
            ctx.run()
            with pytest.raises(gpu_lib.BCError) as ei:
                ctx.read()
            assert ei.value.status == gpu_lib.BC_ERR_OVERFLOW
            ctx.reset()


BATCHED = {
    "one": lambda: gg.path(1),
    "isolated": lambda: gg.disjoint_union(gg.path(1), gg.cycle(9), gg.path(1), gg.path(70)),
    "deep": lambda: gg.path(1500),
    "hubs": lambda: gg.rmat(12, 16, 3),
    # C(34,17) fits 32 bits with a sum that could wrap; C(38,19) and C(66,33)
    # are run again in 64
    "counts32": lambda: gg.grid(18, 18),
    "counts64": lambda: gg.disjoint_union(gg.grid(34, 34), gg.grid(20, 20), gg.path(3)),
    "last": lambda: gg.er_plus_tree(7084, 3.0, 5),
    "past": lambda: gg.er_plus_tree(7085, 3.0, 5),
}


@pytest.mark.parametrize("form,batch", [("sparse", 64), ("sparse", 512), ("hybrid", 256)])
@pytest.mark.parametrize("name", list(BATCHED))
def test_batched_small(gpu_lib, name, form, batch):
    """The batched forms on small graphs: the LDS sweep against the oracle, and
    against the batched kernels (a host-driven context)."""
    g = BATCHED[name]()
    print(f"small {form} {batch} {name} n={g.n}", flush=True)
    src = gg.sample_sources(g.n, min(g.n, 700), 11)
    src = np.concatenate([src, src[:1]]).astype(np.int32)
    want = oracle.bc(g, sources=src, threads=8)
    pick = src[:: max(1, src.size // 5)][:6]
    with gpu_lib.BC(g, form=form, batch=batch, host_driven=True) as ctx:
        ctx.run(src)
        host, levels = ctx.read(), ctx.info().max_levels
    with gpu_lib.BC(g, form=form, batch=batch) as ctx:
        ctx.run(src)
        assert rel_err(ctx.read(), want) <= 1e-5  # FP32 c(v)
        assert rel_err(ctx.read(), host) <= 1e-5
        assert ctx.info().max_levels == levels and ctx.info().sources_run == src.size
        ctx.reset()
        ctx.run()
        assert rel_err(ctx.read(), oracle.bc(g, threads=8)) <= 1e-5
        dist, sigma, delta = ctx.sssp(pick)
    for i, s in enumerate(pick):
        d, sg, dl = oracle.sssp_u64(g, int(s))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)
        assert rel_err(delta[i], dl) <= 1e-5


@pytest.mark.parametrize("form", ["plain", "sparse"])
def test_small_overflow(gpu_lib, form):
    g = gg.grid(35, 35)  # C(68,34) > 2^64 - 1
    with gpu_lib.BC(g, form=form) as ctx:
        ctx.run()
        with pytest.raises(gpu_lib.BCError) as ei:
            ctx.read()
        assert ei.value.status == gpu_lib.BC_ERR_OVERFLOW
        ctx.reset()
        ctx.run(np.array([600], np.int32))  # near the middle: counts fit
        assert rel_err(ctx.read(), oracle.bc(g, sources=np.array([600], np.int32))) <= 1e-5


@pytest.mark.parametrize("form,batch", [("auto", 0), ("sparse", 512), ("hybrid", 256)])
def test_small_contexts_hold_no_batch_state(gpu_lib, form, batch):
    g = gg.er_plus_tree(300, 6.0, 3)
    print(f"small state {form}", flush=True)
    with gpu_lib.BC(g, form=form, batch=batch) as ctx:
        # a batch's counts alone: 8 bytes for every vertex and source
        assert ctx.info().device_bytes < 8 * g.n * ctx.info().batch
        ctx.run()
        assert rel_err(ctx.read(), oracle.bc(g)) <= 1e-5
        assert ctx.info().batch == (batch or 256)
    for bad in (192, 1024):
        with pytest.raises(gpu_lib.BCError) as ei:
            gpu_lib.BC(g, form="sparse", batch=bad)
        assert ei.value.status == gpu_lib.BC_ERR_INVALID_ARG


COLUMNS = {f"er{n}": (lambda n=n: gg.er_plus_tree(n, 9.0, n)) for n in (255, 256, 257, 512, 513)}
COLUMNS |= {
    "star2049": lambda: gg.star(2050),  # 257 bursts in one row
    "late-hub": lambda: gg.disjoint_union(gg.path(600), gg.star(900)),
    "gaps": lambda: gg.disjoint_union(*[gg.path(1)] * 300, gg.complete(40), *[gg.path(1)] * 300),
}


@pytest.mark.parametrize("order", ["degree", "input"])
@pytest.mark.parametrize("name", list(COLUMNS))
def test_padded_columns(gpu_lib, name, order):
    """Row counts around a workgroup's 256, rows of none and of many bursts, in
    the order of their degrees and as given."""
    g = COLUMNS[name]()
    print(f"small columns {name} {order} n={g.n}", flush=True)
    with gpu_lib.BC(g, form="plain", vertex_order=order) as ctx:
        ctx.run()
        assert rel_err(ctx.read(), oracle.bc(g, threads=8)) <= 1e-12  # FP64 throughout


DEALT = {
    "all-heavy": lambda: gg.er_plus_tree(500, 100.0, 1),
    "few-heavy": lambda: gg.er_plus_tree(1500, 50.0, 2),  # their entries stay together
    "bipartite": lambda: gg.complete_bipartite(900, 20),
    "one-heavy": lambda: gg.disjoint_union(gg.star(66), gg.path(500), gg.star(1200)),
    "hubs": lambda: gg.rmat(11, 16, 5),
}


@pytest.mark.parametrize("form,tol", [("plain", 1e-12), ("sparse", 1e-5)])
@pytest.mark.parametrize("name", list(DEALT))
def test_heavy_rows_dealt(gpu_lib, name, form, tol):
    """Levels of one to more than a workgroup's entries, one source and several
    a group, with the heavy rows dealt to the waves and without."""
    g = DEALT[name]()
    print(f"small dealt {name} {form} n={g.n} heavy={int((g.degrees() > 64).sum())}", flush=True)
    with gpu_lib.BC(g, form=form, batch=64 if form == "sparse" else 0) as ctx:
        for src in (np.arange(g.n, dtype=np.int32), gg.sample_sources(g.n, 20, 3)):
            ctx.reset()
            ctx.run(src)
            assert rel_err(ctx.read(), oracle.bc(g, sources=src, threads=8)) <= tol
        dist, sigma, delta = ctx.sssp(src[:3])
    for i in range(3):
        d, sg, dl = oracle.sssp_u64(g, int(src[i]))
        assert np.array_equal(dist[i], d) and np.array_equal(sigma[i], sg)
        assert rel_err(delta[i], dl) <= tol

"""Runs whose batches are dealt to lanes replaying at the same time: results,
counts and errors must be those of one chain of batches driven from the host,
whichever lane a batch lands in."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

STAR = 7200  # with it a graph is too large for the LDS sweeps

GRAPHS = {
    "er": lambda: gg.er_plus_tree(9000, 5.0, 1),
    "hubs": lambda: gg.rmat(14, 8, 2),
    # 39 levels and counts past 2^32 in a few batches only: handed back
    "deep-wide": lambda: gg.disjoint_union(gg.star(STAR), gg.grid(20, 20), gg.path(250)),
}


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0)))


@pytest.mark.parametrize("form,batch,edges", [("sparse", 64, False), ("sparse", 512, False), ("hybrid", 256, False),
                                              ("algebraic", 256, False), ("sparse", 128, True)])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_lanes_equal_one_chain(gpu_lib, name, form, batch, edges):
    g = GRAPHS[name]()
    print(f"lanes {name} {form} {batch} edges={edges} n={g.n}", flush=True)
    src = gg.sample_sources(g.n, 8 * batch + 31, 3) if g.n > 8 * batch + 31 else np.arange(g.n, dtype=np.int32)
    if name == "deep-wide":  # the grid's and the path's sources among the star's
        src = np.unique(np.concatenate([src, np.arange(STAR, g.n, 3, dtype=np.int32)]))
    want = oracle.edge_bc(g, sources=src, threads=8) if edges else (oracle.bc(g, sources=src, threads=8), None)
    with gpu_lib.BC(g, form=form, batch=batch, edges=edges, host_driven=True) as ctx:
        ctx.run(src)
        host, info = ctx.read(), ctx.info()
    with gpu_lib.BC(g, form=form, batch=batch, edges=edges) as ctx:
        for times in (1, 2, 3):
            ctx.run(src)
            if times != 2:  # two runs without a read between
                assert rel_err(ctx.read(), times * want[0]) <= 1e-5
                assert rel_err(ctx.read(), times * host) <= 1e-5
        if edges:
            assert rel_err(ctx.read_edges(), 3 * want[1]) <= 1e-5
        now = ctx.info()
        assert now.sources_run == 3 * src.size and now.max_levels == info.max_levels
        if form == "algebraic":
            # products per batch and level are the same, whichever lane ran them
            assert now.mfma_ktiles_dense * 2 ** 20 == now.mfma_planes * 2 * batch * (-(-g.n // 256) * 256) ** 2
        ctx.reset()
        assert np.all(ctx.read() == 0.0)
        ctx.run(src[: 2 * batch])
        assert rel_err(ctx.read(), oracle.bc(g, sources=src[: 2 * batch], threads=8)) <= 1e-5


def test_overflow_in_a_lane(gpu_lib):
    g = gg.disjoint_union(gg.star(STAR), gg.grid(35, 35))  # C(68,34) > 2^64 - 1, in the last batches
    with gpu_lib.BC(g, form="sparse", batch=64) as ctx:
        ctx.run()
        with pytest.raises(gpu_lib.BCError) as ei:
            ctx.read()
        assert ei.value.status == gpu_lib.BC_ERR_OVERFLOW
        ctx.reset()
        src = np.arange(2000, dtype=np.int32)
        ctx.run(src)
        assert rel_err(ctx.read(), oracle.bc(g, sources=src, threads=8)) <= 1e-5


def test_lanes_on_a_stream(gpu_lib):
    """The run and everything queued after it on the context's stream are in order."""
    import torch
    g = GRAPHS["er"]()
    want = oracle.bc(g, threads=8)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        with gpu_lib.BC(g, form="sparse", batch=256, stream=stream) as ctx:
            for _ in range(3):
                ctx.run()
                got = ctx.read_device()
                ctx.reset()
                assert rel_err(got.cpu().numpy(), want) <= 1e-5

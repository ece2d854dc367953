"""bc_get_info and bc_get_timing while the context's stream is being captured
into a HIP graph: the capture goes on, and nothing of theirs is in the graph."""
import ctypes

import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_0809_1906_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,n", [("plain", 300), ("sparse", 300), ("hybrid", 300), ("sparse", 9000),
                                    ("algebraic", 600)])
@pytest.mark.parametrize("timing", [0, 1])
def test_info_under_capture(gpu_lib, form, n, timing):
    import torch
    g = gg.er_plus_tree(n, 5.0, 2105)
    stream = torch.cuda.Stream(device=0)
    lib = B.load()
    print(f"capture_info {form} n={n} timing={timing}", flush=True)
    with gpu_lib.BC(g, form=form, stream=stream, timing=timing) as ctx:
        ctx.run()
        known = ctx.info()
        ctx.run()  # replays whose checks are still to be read
        x = torch.zeros(16, device="cuda:0")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        info, ms, launches = B.bc_info(), ctypes.c_double(), ctypes.c_int64()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
            x.add_(1.0)
            got = lib.bc_get_info(ctx.handle, ctypes.byref(info))
            codes = [lib.bc_get_timing(ctx.handle, k, ctypes.byref(ms), ctypes.byref(launches))
                     for k in (b"no such kernel", b"batch_init", b"plain_sweep")]
        assert got == B.BC_OK and codes[0] == B.BC_OK
        timed = {"plain": 2}.get(form, 1) if timing else 0
        assert [i for i, c in enumerate(codes) if c == B.BC_ERR_STATE] == ([timed] if timed else [])
        assert info.n == g.n and info.max_levels == known.max_levels and info.sources_run == 2 * g.n
        if form == "algebraic":
            assert info.mfma_planes == info.mfma_ktiles_run == -1
        for replays in (1.0, 2.0):
            graph.replay()
            torch.cuda.synchronize()
            assert float(x[0]) == replays
        assert np.max(np.abs(ctx.read() - 2 * oracle.bc(g)) / np.maximum(2 * oracle.bc(g), 1.0)) <= 1e-5

"""Work that is still pending on the context's stream: memory that a
stream-ordered allocator hands over while the stream still writes to it, and
device inputs that the stream has yet to write."""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

SLEEP = 20_000_000  # clock ticks: 10 to 200 ms, far longer than the host needs


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0)))


def cases():
    er = gg.er_plus_tree(400, 5.0, 1)
    return {"plain": (er, dict(form="plain")), "small": (er, dict(form="sparse")),
            "sparse": (gg.er_plus_tree(8000, 4.0, 2), dict(form="sparse", batch=256)),
            "edges": (er, dict(form="sparse", edges=True)),
            "weighted": (gg.with_uniform_weights(er, 3, 1, 20), dict()),
            "many": ([er, gg.path(30)], dict())}


@pytest.mark.parametrize("name", list(cases()))
def test_created_in_memory_still_written(gpu_lib, name):
    import torch
    g, kw = cases()[name]
    want = np.concatenate([oracle.bc(x) for x in g]) if isinstance(g, list) else oracle.bc(g, threads=8)
    stream = torch.cuda.Stream()
    print(f"stream_order create {name}", flush=True)
    with torch.cuda.stream(stream):
        held = [torch.empty(1 << k, dtype=torch.uint8, device="cuda:0") for k in range(8, 23) for _ in range(4)]
        torch.cuda.synchronize()
        torch.cuda._sleep(SLEEP)
        for x in held:
            x.fill_(1)
        del held, x  # the allocator may hand these over while they are written
        with gpu_lib.BC(g, stream=stream, **kw) as ctx:
            ctx.run()
            assert rel_err(ctx.read(), want) <= 1e-5


@pytest.mark.parametrize("form", ["plain", "sparse"])
def test_sources_still_to_be_written(gpu_lib, form):
    import torch
    g = gg.er_plus_tree(8000, 4.0, 2)
    src = gg.sample_sources(g.n, 600, 5)
    stream = torch.cuda.Stream()
    print(f"stream_order sources {form}", flush=True)
    with torch.cuda.stream(stream):
        given = torch.from_numpy(src.astype(np.int32)).to("cuda:0")
        later = torch.zeros_like(given)
        with gpu_lib.BC(g, form=form, stream=stream) as ctx:
            torch.cuda.synchronize()
            torch.cuda._sleep(SLEEP)
            later.copy_(given)
            ctx.run(later)
            assert rel_err(ctx.read(), oracle.bc(g, sources=src, threads=8)) <= 1e-5


def test_graph_still_to_be_written(gpu_lib):
    import ctypes

    import torch
    from paper_0809_1906_amd import binding as B
    g = gg.er_plus_tree(400, 5.0, 1)
    other = gg.star(g.n)  # a valid graph of as many vertices, in the arrays before
    stream = torch.cuda.Stream()
    print("stream_order graph", flush=True)
    with torch.cuda.stream(stream):
        row_ptr, col = (torch.from_numpy(x.astype(np.int32)).to("cuda:0") for x in (g.row_ptr, g.col))
        old_ptr, old_col = (torch.from_numpy(x.astype(np.int32)).to("cuda:0") for x in (other.row_ptr, other.col))
        now_ptr = old_ptr.clone()
        now_col = torch.zeros_like(col)
        now_col[: old_col.numel()] = old_col
        opt = B.bc_options_init()
        opt.form = B.FORMS["plain"]
        opt.stream = stream.cuda_stream
        graph = B.bc_graph()
        graph.n, graph.nnz = g.n, g.col.size
        graph.row_ptr, graph.col, graph.weight = now_ptr.data_ptr(), now_col.data_ptr(), None
        graph.mem = B.BC_MEM_DEVICE
        torch.cuda.synchronize()
        torch.cuda._sleep(SLEEP)
        now_ptr.copy_(row_ptr)
        now_col.copy_(col)
        ctx = ctypes.c_void_p()
        st = B.load().bc_create(ctypes.byref(graph), ctypes.byref(opt), ctypes.byref(ctx))
        assert st == B.BC_OK, B.bc_last_error(None)
        out = np.zeros(g.n)
        assert B.load().bc_run(ctx, None, -1, B.BC_MEM_HOST) == B.BC_OK
        assert B.load().bc_read(ctx, out.ctypes.data, B.BC_MEM_HOST) == B.BC_OK
        B.load().bc_destroy(ctx)
    assert rel_err(out, oracle.bc(g)) <= 1e-12

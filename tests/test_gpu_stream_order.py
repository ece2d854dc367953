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

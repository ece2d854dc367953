"""Contexts whose batches run on the device's shared lane streams: several alive
at once, driven from several threads and streams, destroyed in any order."""
import threading

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0)))


def test_contexts_share_lane_streams(gpu_lib):
    import torch
    graphs = [gg.er_plus_tree(n, 5.0, n) for n in (7300, 7900, 8100, 8600)]
    want = [oracle.bc(g, threads=8) for g in graphs]
    streams = [None, torch.cuda.Stream(), None, torch.cuda.Stream()]
    ctxs = [gpu_lib.BC(g, form="sparse", batch=256) for g in graphs]
    errors = {}

    def drive(i):
        with torch.cuda.stream(streams[i]) if streams[i] is not None else torch.cuda.stream(torch.cuda.default_stream()):
            for _ in range(3):
                ctxs[i].reset()
                ctxs[i].run()
            errors[i] = rel_err(ctxs[i].read(), want[i])

    threads = [threading.Thread(target=drive, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert sorted(errors) == [0, 1, 2, 3] and max(errors.values()) <= 1e-5
    ctxs[0].close()  # the others keep the streams
    ctxs[2].close()
    for i in (1, 3):
        ctxs[i].reset()
        ctxs[i].run()
        assert rel_err(ctxs[i].read(), want[i]) <= 1e-5
        ctxs[i].close()
    with gpu_lib.BC(graphs[0], form="sparse", batch=256) as ctx:  # streams anew
        ctx.run()
        assert rel_err(ctx.read(), want[0]) <= 1e-5

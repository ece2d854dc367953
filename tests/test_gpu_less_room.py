"""Runs that cannot have all the device memory they would like: where the
library has a way to go on with less, it does, and the results are the same."""
import ctypes

import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_0809_1906_amd import binding as B
from test_gpu_guards import CountingAllocator, create_raw

pytestmark = pytest.mark.gpu


class Refusing(CountingAllocator):
    """Refuses the requests that refuse(bytes) picks, leaving the HIP error of a
    failed hipMalloc behind, as the library's own allocations do."""

    def __init__(self):
        super().__init__()
        self.refuse = lambda nbytes: False
        self.refused = 0
        lib, grant = B.load(), self.alloc

        def _alloc(nbytes, stream, user):
            if not self.refuse(nbytes):
                return grant(nbytes, stream, user)
            p = ctypes.c_void_p()
            assert lib.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 50)) != 0
            self.refused += 1
            return None

        self.alloc = B.ALLOC_FN(_alloc)


def rel_err(x, y):
    return float(np.max(np.abs(x - y) / np.maximum(np.abs(y), 1.0)))


def context(g, form, batch):
    import torch
    a = Refusing()
    st, ctx = create_raw(g, form, batch, a, torch.cuda.current_stream(0))
    assert st == B.BC_OK
    return a, ctx


def read(ctx, n):
    out = np.zeros(n)
    assert B.load().bc_read(ctx, out.ctypes.data, B.BC_MEM_HOST) == B.BC_OK
    return out


@pytest.mark.parametrize("granted", [0, 1])
def test_lanes_without_their_state(gpu_lib, granted):
    """No memory for the counts of a further lane: the run takes fewer."""
    g = gg.er_plus_tree(9000, 5.0, 1)
    want = oracle.bc(g, threads=8)
    a, ctx = context(g, "sparse", 64)
    asked = []

    def refuse(nbytes):
        if nbytes == g.n * 64 * 8:
            asked.append(nbytes)
            return len(asked) > granted
        return False

    a.refuse = refuse
    print(f"less_room lanes granted={granted}", flush=True)
    for times in (1, 2):
        assert B.load().bc_run(ctx, None, -1, B.BC_MEM_HOST) == B.BC_OK
        assert rel_err(read(ctx, g.n), times * want) <= 1e-5
    assert a.refused > 0
    B.load().bc_destroy(ctx)
    assert not a.live


def test_all_pairs_without_the_far_matrices(gpu_lib):
    """No memory for the two matrices of the far triples at once."""
    g = gg.watts_strogatz(331, 4, 0.05, 9)  # pairs at distance 4 and more
    want = oracle.bc(g)
    a, ctx = context(g, "sparse", 64)
    asked = []

    def refuse(nbytes):
        if nbytes == g.n * 384 * 4:  # rows of a multiple of 64
            asked.append(nbytes)
            return len(asked) == 2
        return False

    a.refuse = refuse
    print("less_room all_pairs", flush=True)
    out = np.zeros(g.n)
    assert B.load().bc_all_pairs(ctx, out.ctypes.data, B.BC_MEM_HOST) == B.BC_OK
    assert a.refused == 1 and rel_err(out, want) <= 1e-12
    B.load().bc_destroy(ctx)
    assert not a.live

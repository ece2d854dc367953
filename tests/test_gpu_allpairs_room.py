"""Algorithm 2 without the memory for the far triples' two matrices: every
triple by the triple sum, the same result; without the memory for what it
always needs, BC_ERR_NOMEM and nothing left behind."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_0809_1906_amd import binding as B
from test_gpu_guards import CountingAllocator, create_raw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["sparse", "plain"])
def test_all_pairs_with_less_room(gpu_lib, form):
    import torch
    g = gg.watts_strogatz(331, 4, 0.05, 9)  # pairs at distance 4 and more
    want = oracle.bc(g)
    lib = B.load()
    failed = []
    for extra in range(10):
        a = CountingAllocator()
        st, ctx = create_raw(g, form, 64 if form == "sparse" else 0, a, torch.cuda.current_stream(0))
        assert st == B.BC_OK
        held, first = len(a.live), a.calls
        a.fail_at = first + extra
        print(f"all_pairs room {form} allocation {extra}", flush=True)
        out = np.zeros(g.n)
        st = lib.bc_all_pairs(ctx, out.ctypes.data, B.BC_MEM_HOST)
        assert len(a.live) == held
        assert st in (B.BC_OK, B.BC_ERR_NOMEM)
        if st == B.BC_OK:
            assert np.max(np.abs(out - want) / np.maximum(want, 1.0)) <= 1e-12
        failed.append(st == B.BC_ERR_NOMEM)
        made = a.calls - first
        lib.bc_destroy(ctx)
        assert not a.live
        if extra >= made:
            break
    # the last two requests of a full run are the far triples' matrices
    assert failed[-1] is False and made >= 8
    assert all(failed[:made - 2]) and not any(failed[made - 2:])

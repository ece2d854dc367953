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


@pytest.mark.parametrize("form", ["sparse", "plain"])
@pytest.mark.parametrize("name", ["deep", "near"])
def test_all_pairs_in_24_bytes_a_pair(gpu_lib, name, form):
    """Distances past a byte leave every triple to the triple sum; so do near
    ones where there is no more memory."""
    g = gg.path(512) if name == "deep" else gg.watts_strogatz(512, 4, 0.05, 9)
    a, ctx = context(g, form, 0 if form == "plain" else 64)
    held = sum(a.live.values())
    room = held + 24 * g.n * g.n + 8 * g.n + 8192  # the result, the sources
    a.refuse = lambda nbytes: sum(a.live.values()) + nbytes > room
    print(f"less_room all_pairs {name} {form}", flush=True)
    out = np.zeros(g.n)
    assert B.load().bc_all_pairs(ctx, out.ctypes.data, B.BC_MEM_HOST) == B.BC_OK
    assert rel_err(out, oracle.bc(g)) <= 1e-12
    assert sum(a.live.values()) == held
    B.load().bc_destroy(ctx)
    assert not a.live


def up256(nbytes):
    return -(-nbytes // 256) * 256


@pytest.mark.parametrize("granted", [0, 1])
def test_lanes_without_their_levels(gpu_lib, granted):
    """A further lane has its state but not the bitmaps of a deep graph's levels."""
    g = gg.watts_strogatz(9000, 4, 0.002, 3)
    want = oracle.bc(g, threads=8)
    level = g.n * 8
    a, ctx = context(g, "sparse", 64)
    asked = []

    def refuse(nbytes):
        # the first state's storage doubles from 16 levels as its search goes on; a
        # lane's is made in one go for the depth that is known by then
        if nbytes > up256(32 * level) and nbytes not in [up256(k * level) for k in (64, 128, 256, 512, 1024, 2048)]:
            asked.append(nbytes)
            return len(asked) > granted
        return False

    a.refuse = refuse
    print(f"less_room levels granted={granted}", flush=True)
    for times in (1, 2):
        assert B.load().bc_run(ctx, None, -1, B.BC_MEM_HOST) == B.BC_OK
        assert rel_err(read(ctx, g.n), times * want) <= 1e-5
    assert a.refused > 0
    B.load().bc_destroy(ctx)
    assert not a.live


def test_lanes_give_way_to_deeper_levels(gpu_lib):
    """A state that has to grow past what is left takes the lanes' memory."""
    star = 7200
    g = gg.disjoint_union(gg.star(star), gg.path(250))
    shallow = np.arange(1, 8 * 64 + 1, dtype=np.int32)
    deep = np.arange(star, g.n, dtype=np.int32)
    a, ctx = context(g, "sparse", 64)
    lib = B.load()
    print("less_room give way", flush=True)
    want = run_until_lanes(ctx, a, shallow) * oracle.bc(g, sources=shallow)
    assert rel_err(read(ctx, g.n), want) <= 1e-5
    # room for a growth to 256 levels beside the 128 before only without the lanes,
    # of which each holds 12 bytes for a vertex and source
    room = sum(a.live.values()) + 16 * g.n * 64 * 2
    a.refuse = lambda nbytes: sum(a.live.values()) + nbytes > room
    assert lib.bc_run(ctx, deep.ctypes.data, deep.size, B.BC_MEM_HOST) == B.BC_OK
    want += oracle.bc(g, sources=deep)
    assert rel_err(read(ctx, g.n), want) <= 1e-5
    assert a.refused > 0
    a.refuse = lambda nbytes: False
    lib.bc_destroy(ctx)
    assert not a.live


def run_until_lanes(ctx, a, src):
    """Runs until the context has set its lanes up (more than a dozen requests
    each); returns how often."""
    for times in range(1, 100):
        calls = a.calls
        assert B.load().bc_run(ctx, src.ctypes.data, src.size, B.BC_MEM_HOST) == B.BC_OK
        if a.calls >= calls + 20:
            return times
    raise AssertionError("no lanes")


def refuse_next(a):
    """Refuses one request."""
    left = [True]
    a.refuse = lambda nbytes: left.pop() if left else False


def readout(ctx, n):
    src, dist = np.zeros(1, np.int32), np.zeros((1, n), np.int32)
    return B.load().bc_read_sssp(ctx, src.ctypes.data, 1, dist.ctypes.data, None, None)


def test_lanes_given_up_leave_their_overflow(gpu_lib):
    g = gg.disjoint_union(gg.star(7200), gg.grid(35, 35))  # C(68,34) > 2^64 - 1
    corners = np.tile(np.array([7200, g.n - 1], np.int32), 4 * 64)
    a, ctx = context(g, "sparse", 64)
    lib = B.load()
    print("less_room overflow", flush=True)
    run_until_lanes(ctx, a, np.arange(1, 8 * 64 + 1, dtype=np.int32))
    for _ in range(2):  # the second run's counts are 64 bits wide from the start
        assert lib.bc_reset(ctx) == B.BC_OK
        assert lib.bc_run(ctx, corners.ctypes.data, corners.size, B.BC_MEM_HOST) == B.BC_OK
    refuse_next(a)
    assert readout(ctx, g.n) == B.BC_OK and a.refused == 1
    out = np.zeros(g.n)
    assert lib.bc_read(ctx, out.ctypes.data, B.BC_MEM_HOST) == B.BC_ERR_OVERFLOW
    assert lib.bc_reset(ctx) == B.BC_OK
    assert not np.any(read(ctx, g.n))
    lib.bc_destroy(ctx)
    assert not a.live


def test_lanes_given_up_leave_their_products(gpu_lib):
    g = gg.er_plus_tree(2500, 20.0, 4)
    lib = B.load()
    seen = []
    gpu_lib.BC(g, form="algebraic", batch=256).close()  # tuned: the contexts below start alike
    for give_up in (False, True):
        print(f"less_room products give_up={give_up}", flush=True)
        a, ctx = context(g, "algebraic", 256)
        run_until_lanes(ctx, a, np.arange(g.n, dtype=np.int32))
        assert lib.bc_run(ctx, None, -1, B.BC_MEM_HOST) == B.BC_OK
        held = B.bc_get_info(ctx).device_bytes
        if give_up:
            refuse_next(a)
        assert readout(ctx, g.n) == B.BC_OK and a.refused == give_up
        info = B.bc_get_info(ctx)
        assert (info.device_bytes < held) == give_up
        seen.append((info.mfma_planes, info.mfma_ktiles_run, info.mfma_ktiles_dense, info.mfma_ktiles_run_fwd,
                     info.mfma_ktiles_dense_fwd))
        lib.bc_destroy(ctx)
        assert not a.live
    assert seen[0] == seen[1] and min(seen[0]) > 0


def test_handed_back_batches_wait_for_memory(gpu_lib):
    """A call without the memory for handed-back batches leaves them to the next."""
    import torch
    # K2s come last in the order of the sources, so the first batch is shallow
    # and the path's are handed back
    g = gg.disjoint_union(gg.star(7200), gg.path(250), *[gg.path(2)] * 60)
    want = oracle.bc(g)
    src = np.array([0, 7300], np.int32)
    dist = torch.empty((2, g.n), dtype=torch.int32, device="cuda:0")
    print("less_room handed back", flush=True)
    with gpu_lib.BC(g, form="sparse", batch=64) as ctx:
        ctx.run()
        for _ in range(2):
            with pytest.raises(gpu_lib.BCError) as ei:
                ctx.sssp_noalloc(src, dist=dist)
            assert ei.value.status == gpu_lib.BC_ERR_NOMEM
        assert rel_err(ctx.read(), want) <= 1e-5
    # a reset while they wait
    a, ctx = context(g, "sparse", 64)
    lib = B.load()
    assert lib.bc_run(ctx, None, -1, B.BC_MEM_HOST) == B.BC_OK
    a.refuse = lambda nbytes: True
    out = np.zeros(g.n)
    assert lib.bc_read(ctx, out.ctypes.data, B.BC_MEM_HOST) == B.BC_ERR_NOMEM
    assert lib.bc_reset(ctx) == B.BC_OK
    assert lib.bc_read(ctx, out.ctypes.data, B.BC_MEM_HOST) == B.BC_OK and not np.any(out)
    a.refuse = lambda nbytes: False
    assert lib.bc_run(ctx, None, -1, B.BC_MEM_HOST) == B.BC_OK
    assert rel_err(read(ctx, g.n), want) <= 1e-5
    lib.bc_destroy(ctx)
    assert not a.live

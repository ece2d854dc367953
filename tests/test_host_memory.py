"""Host allocations that fail inside a C entry (no GPU needed)."""
import os
import subprocess
import sys

from paper_0809_1906_amd import binding as B

NO_HOST_MEMORY = """
import ctypes, resource
import numpy as np
import graphgen as gg
from paper_0809_1906_amd import binding as B
lib = B.load()
g = gg.complete(1500)
rp, col = np.ascontiguousarray(g.row_ptr, np.int32), np.ascontiguousarray(g.col, np.int32)
gs = (B.bc_graph * 40)()
for x in gs:
    x.n, x.nnz, x.row_ptr, x.col, x.weight, x.mem = g.n, col.size, rp.ctypes.data, col.ctypes.data, None, B.BC_MEM_HOST
ctx = ctypes.c_void_p(1)
held = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (held + (60 << 20), resource.RLIM_INFINITY))
status = lib.bc_create_many(gs, len(gs), None, ctypes.byref(ctx))  # 360 MB of columns
print("status", status, ctx.value, lib.bc_last_error(None).decode())
"""


def test_no_host_memory_is_an_error_not_an_exception():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    run = subprocess.run([sys.executable, "-c", NO_HOST_MEMORY], cwd=root, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr[-500:]
    assert f"status {B.BC_ERR_NOMEM} None" in run.stdout

"""Upload of a plan to a device without room for all of it, on a stand-in for the HIP runtime (c_abi/hip_stub.c): the library is
the one that runs on the GPU, its device memory is host memory within a budget."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PROGRAM = r"""
import ctypes, sys
import numpy as np
sys.path.insert(0, sys.argv[1])
from paper_2603_08734_amd import Plan, RshError, binding
from workloads import from_coo
stub = ctypes.CDLL(sys.argv[2])
stub.stub_live.restype = stub.stub_peak.restype = ctypes.c_size_t
stub.stub_budget.argtypes = [ctypes.c_size_t]

rng = np.random.default_rng(3)
rows, cols, N = 1100, 600, int(sys.argv[3])
cells = rng.random((rows, cols)) < 0.12
cells[1024:] = 0                        # 76 rows of the residual part
r, c = np.nonzero(cells)
r = np.concatenate([r, np.repeat(np.arange(1024, rows), 3)])
c = np.concatenate([c, np.tile([5, 77, 500], rows - 1024)])
A = from_coo(r, c, rng.standard_normal(r.size), rows, cols)

def plan(budget):
    stub.stub_budget(budget)
    try:
        p = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, window_rows=256, reorder=0, max_tiles_per_item=8)
    except RshError as e:
        assert e.status == binding.RSH_ERR_OOM, e
        assert stub.stub_live() == 0, "memory kept by a plan that was not made"
        return "none", None, None
    out = "written out" if p.kernels()["cells_written"] else "packed", p.stats(), stub.stub_peak()
    p.destroy()
    assert stub.stub_live() == 0, "memory kept by a plan that is gone"
    return out

most, st, peak = plan(1 << 40)
assert most == "written out" and st["nnz_irregular"] > 0 and st["n_scratch_slots"] > 0 and st["n_split_windows"] > 0
seen = []
for budget in range(peak + 4096, 0, -peak // 160):
    form, stats, _ = plan(budget)
    if not seen or seen[-1] != form:
        seen.append(form)
    if form == "packed":
        less = st["tile_part_bytes"] - stats["tile_part_bytes"]
        assert less > 0 and all(st[k] - stats[k] == less for k in ("plan_bytes", "bytes_method", "bytes_method_element_level"))
        assert all(st[k] == stats[k] for k in ("n_tile_items", "n_scratch_slots", "irregular_part_bytes", "n_combine"))
assert seen == ["written out", "packed", "none"], seen
print("ok")
"""


@pytest.mark.parametrize("N", [130, 256])
def test_a_plan_whose_cells_leave_no_room_takes_the_packed_form(tmp_path, N):
    stub = tmp_path / "libhipstub.so"
    subprocess.check_call(["gcc", "-O1", "-Wall", "-Wextra", "-shared", "-fPIC", "-o", str(stub), os.path.join(HERE, "c_abi", "hip_stub.c")])
    env = dict(os.environ, LD_PRELOAD=" ".join(x for x in (str(stub), os.environ.get("LD_PRELOAD", "")) if x))
    out = subprocess.run([sys.executable, "-c", PROGRAM, os.path.dirname(HERE), str(stub), str(N)], env=env, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stderr[-3000:]

"""Residual rows whose lanes own rows of B or share them (rsh_narrow_kernel, rsh_shared_kernel): what a sum may lose, and what
lanes read past the end of their rows."""
import numpy as np
import pytest

from oracle import spmm as oracle
from workloads import from_coo

pytestmark = pytest.mark.gpu


def product(A, B, lanes, **opts):
    import torch
    from paper_2603_08734_amd import Plan
    N = B.shape[1]
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, force_path=1, **opts)
    assert plan.kernels()["row_lanes"] == lanes
    Bd = torch.from_numpy(B).cuda()
    C = torch.full((A.n_rows, N), float("nan"), dtype=torch.float32, device="cuda")
    plan.spmm(Bd, C)
    torch.cuda.synchronize()
    plan.destroy()
    return C.cpu().numpy().astype(np.float64)


# 32 entries, as many as one lane takes, the first product 1 and the others 2^-25: one behind the other in fp32 none of them would
# count.  Entries are added up in pairs, pairs in 64 bits: a pair's sum and the result are rounded to 2^-24 of themselves.
@pytest.mark.parametrize("N,lanes", [(1, 1), (2, 1), (4, 1), (7, 1), (8, 1), (9, 2), (16, 2), (32, 4), (48, 8)])
def test_entries_of_a_lane_keep_small_products(N, lanes):
    rows, length = 140000, 32
    r = np.repeat(np.arange(rows), length)
    c = np.tile(np.arange(length), rows)
    A = from_coo(r, c, np.where(c == 0, 1.0, 2.0 ** -12), rows, length)
    B = np.full((length, N), 2.0 ** -13, dtype=np.float16)
    B[0] = 1.0
    print(f"case small products N={N}", flush=True)
    got = product(A, B, lanes)
    exact = 1.0 + 31 * 2.0 ** -25
    assert np.abs(got - exact).max() <= 2 * 2.0 ** -24 * exact

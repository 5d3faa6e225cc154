"""GPU parity of the tall-window kernel where its packed units, quads of fragments and window parts end.

Bound as everywhere: |C - C_ref| <= 1e-4 * sum_k |a_ik| |b_kj| elementwise (fp32 chains of at most
1024 + parts additions, 1024 * 2^-24 = 6.1e-5)."""
import numpy as np
import pytest

from oracle import spmm as oracle
from workloads import dense_B, from_coo

pytestmark = pytest.mark.gpu


def random_matrix(rows, cols, density, seed):
    rng = np.random.default_rng(seed)
    m = rng.random((rows, cols)) < density
    r, c = np.nonzero(m)
    return from_coo(r, c, rng.standard_normal(r.size), rows, cols)


# density 1: every lane holds its eight values; 0.3: mask halves of all kinds; 0.02: mostly empty lanes, and
# windows whose columns are not one run.  400 and 130 columns: 13 and 5 fragments, so that the last quad of a
# window is short; 300 rows: a last window that is mostly absent.  Parts of 3 fragments begin inside quads.
@pytest.mark.parametrize("N", [16, 48, 80, 128, 160])
@pytest.mark.parametrize("density,cols", [(1.0, 130), (0.3, 400), (0.02, 1500)])
@pytest.mark.parametrize("window_rows,parts", [(128, 0), (256, 0), (128, 3), (256, 3)])
def test_units_quads_and_parts(N, density, cols, window_rows, parts):
    A = random_matrix(300, cols, density, 5)
    from paper_2603_08734_amd import Plan
    import torch
    print(f"case panel N={N} density={density} cols={cols} W={window_rows} parts={parts}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, window_rows=window_rows, force_path=2, max_tiles_per_item=parts)
    assert plan.stats()["nnz_tile"] == A.nnz
    B = dense_B(A.n_cols, N, "normal", seed=N)
    Bd = torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16)
    C = torch.full((A.n_rows, N), float("nan"), dtype=torch.float32, device="cuda")
    plan.spmm(Bd, C)
    torch.cuda.synchronize()
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    got = C.cpu().numpy()
    assert not np.isnan(got).any()
    assert np.all(np.abs(got.astype(np.float64) - C_ref) <= 1e-4 * S)
    plan.destroy()

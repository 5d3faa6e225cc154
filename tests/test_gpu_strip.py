"""GPU parity of the kernel whose waves divide the columns of tall windows (strip.hpp), in every form it has.

Bound as everywhere: |C - C_ref| <= 1e-4 * sum_k |a_ik| |b_kj| elementwise (a wave's fp32 chain has at most 1024 products, eight
waves and a tree behind it: 1030 * 2^-24 = 6.2e-5)."""
import numpy as np
import pytest

from oracle import spmm as oracle
from workloads import dense_B, from_coo


def matrix(rows, cols, density, seed=3, holes=True):
    """`holes`: the first window lacks a column, so that its columns are not one run; the others' are."""
    rng = np.random.default_rng(seed)
    m = rng.random((rows, cols), dtype=np.float32) < density
    if holes:
        m[:256, cols // 2] = False
    m[np.flatnonzero(~m.any(1)), 0] = True
    r, c = np.nonzero(m)
    return from_coo(r, c, rng.standard_normal(r.size), rows, cols)


A32, B32, A64, B64, B64L, E64 = (32, 1, 8), (32, 2, 4), (64, 1, 8), (64, 2, 8), (64, 2, 8), (64, 2, 4)
# Columns: less than a fragment, less than a quad (waves without work), quads that do not divide among the waves, the most that
# four waves take and one fragment more.  Features: every place in which a row of B or C can end (inside pieces of 8 and 4, odd
# ones, whole panels, one into the next panel).  Rows: a last window with absent groups and half a group.
CASES = [
    (1100, 20, 0.5, 1, A32), (1100, 20, 0.5, 16, A32), (1100, 130, 0.3, 7, A32), (1100, 1100, 0.2, 3, A32), (1100, 1100, 0.2, 8, A32),
    (1100, 1100, 0.2, 15, A32), (1100, 1100, 0.2, 17, A32), (1100, 1100, 0.2, 31, A32), (1100, 1100, 0.2, 32, A32), (1100, 300, 0.2, 33, A32),
    (1100, 300, 0.2, 100, A32), (1100, 300, 0.2, 191, A32), (1030, 8192, 0.15, 24, A32),
    (16500, 40, 0.5, 3, B32), (16500, 130, 0.3, 9, B32), (16500, 130, 0.3, 16, B32), (16500, 300, 0.2, 31, B32), (16500, 4130, 0.1, 13, B32), (16500, 8192, 0.1, 5, B32),
    (4300, 300, 0.2, 64, A64), (4300, 130, 0.3, 50, A64), (4300, 300, 0.2, 63, A64), (1100, 300, 0.2, 350, A64), (1100, 300, 0.2, 257, A64),
    (8300, 300, 0.2, 64, B64), (8300, 130, 0.3, 58, B64), (8300, 20, 0.5, 33, B64), (2143, 300, 0.2, 203, B64),
    (16600, 300, 0.2, 64, E64), (16600, 130, 0.3, 42, E64), (8300, 130, 0.3, 127, E64), (16500, 4130, 0.1, 62, B64L),
]


# Operands at their element's alignment where the width allows it; B is read where it lies but in the two plans whose loads at
# 2-byte boundaries would cost more than a copy.
@pytest.mark.gpu
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("rows,cols,density,N,form", CASES)
def test_waves_that_divide_the_columns(rows, cols, density, N, form, fused):
    product(rows, cols, density, N, form, fused, N % 2, copied=(rows, cols, N) in ((16500, 4130, 13), (16500, 8192, 5)))


# Rows of whole pieces, B at its element's alignment (N = 8) or at 4 bytes: the loads of the kernel of broken pieces.
@pytest.mark.gpu
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("rows,cols,density,N,form,shift", [(1100, 1100, 0.2, 8, A32, 1), (1100, 20, 0.5, 8, A32, 3), (1100, 1100, 0.2, 24, A32, 2), (16500, 300, 0.2, 24, B32, 2),
                                                           (4300, 300, 0.2, 40, A64, 2), (8300, 300, 0.2, 40, B64, 6)])
def test_rows_of_whole_pieces_at_other_alignments(rows, cols, density, N, form, shift, fused):
    product(rows, cols, density, N, form, fused, shift, copied=False)


def product(rows, cols, density, N, form, fused, shift, copied):
    """`shift`: halves by which B lies behind an aligned address; what lies around B is not finite."""
    import torch
    from paper_2603_08734_amd import Plan
    A = matrix(rows, cols, density)
    print(f"case strip rows={rows} cols={cols} N={N} fused={fused} shift={shift}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, force_path=2, reorder=0)
    assert plan.strip() == form and plan.stats()["n_split_windows"] == 0
    B = dense_B(A.n_cols, N, "normal", seed=N)
    odd = N % 2 == 1
    Bf = torch.full((A.n_cols * N + shift + 8,), float("nan"), dtype=torch.float16, device="cuda")
    Bd = Bf[shift:shift + A.n_cols * N].view(A.n_cols, N)
    Bd.copy_(torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16))
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    pad = 65 if odd else 64
    flat = torch.full((A.n_rows * N + 2 * pad,), float("nan"), dtype=torch.float16 if fused else torch.float32, device="cuda")
    C = flat[pad:pad + A.n_rows * N].view(A.n_rows, N)
    assert plan.operand(Bd.data_ptr(), C.data_ptr()) == (copied, (N + 15) // 16 * 16 if copied else N)
    bound = 1e-4 * S
    if fused:
        bias = torch.linspace(-1, 1, N, device="cuda")
        plan.spmm_f16(Bd, C, bias, relu=True)
        C_ref = np.maximum(C_ref + bias.cpu().numpy().astype(np.float64), 0.0)
        # the fp32 bound, the addition of the bias, one rounding to binary16
        bound = bound + 2.0 ** -24 * np.abs(C_ref) + 2.0 ** -11 * np.abs(C_ref) * 1.001 + 2.0 ** -24
    else:
        plan.spmm(Bd, C)
    torch.cuda.synchronize()
    assert bool(torch.isnan(flat[:pad]).all()) and bool(torch.isnan(flat[pad + A.n_rows * N:]).all()), "stores outside C"
    got = C.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any()
    assert np.all(np.abs(got - C_ref) <= bound)
    plan.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("N", [5, 16, 33, 130])
def test_windows_beside_rows_without_entries(N):
    """Empty rows are the residual kernel's, which reads the padded copy of B; both kernels then do."""
    import torch
    from paper_2603_08734_amd import Plan
    A = matrix(1300, 200, 0.3)
    keep = np.arange(1300) % 7 != 3
    r = np.repeat(np.arange(1300), np.diff(A.row_ptr))
    A = from_coo(r[keep[r]], A.col_idx[keep[r]], A.val[keep[r]].astype(np.float64), 1300, 200)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, reorder=0)
    assert plan.strip() is not None and plan.stats()["n_empty_rows"] == np.count_nonzero(~keep)
    B = dense_B(A.n_cols, N, "normal", seed=N)
    C = torch.full((A.n_rows, N), float("nan"), dtype=torch.float32, device="cuda")
    Bd = torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16)
    assert plan.operand(Bd.data_ptr(), C.data_ptr())[0] == (N < 16 or N % 2 == 1)
    plan.spmm(Bd, C)
    torch.cuda.synchronize()
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    assert np.all(np.abs(C.cpu().numpy().astype(np.float64) - C_ref) <= 1e-4 * S)
    plan.destroy()


# Windows that name different columns, from 128 on: an XCD takes the strips of a window one behind the other.  The last window lacks
# row groups; 128 and 130 windows: the last turn of the XCDs is full, or two of them have it alone.
@pytest.mark.gpu
@pytest.mark.parametrize("rows,N,form", [(32700, 64, E64), (33200, 31, B32), (33200, 18, B32), (33200, 16, B32)])
def test_strips_of_a_window_one_behind_the_other(rows, N, form):
    import torch
    from paper_2603_08734_amd import Plan
    rng = np.random.default_rng(4)
    r, c = np.nonzero(rng.random((rows, 512), dtype=np.float32) < 0.3)
    A = from_coo(r, r * (rows - 512) // (rows - 1) + c, rng.standard_normal(r.size), rows, rows)
    print(f"case strips of a band rows={rows} N={N}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, force_path=2, reorder=0)
    st = plan.stats()
    assert plan.strip() == form and st["n_windows"] == -(-rows // 256) >= 128 and 64 * st["n_tiles"] < st["n_windows"] * rows
    B = dense_B(A.n_cols, N, "normal", seed=N)
    C = torch.full((rows, N), float("nan"), dtype=torch.float32, device="cuda")
    plan.spmm(torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16), C)
    torch.cuda.synchronize()
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    got = C.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any() and np.all(np.abs(got - C_ref) <= 1e-4 * S)
    plan.destroy()


# Both sides of the lines up to which strips are taken: short windows in several rounds, rows of B in pieces or whole, long windows of
# many features, the copy of B that whole windows do without.
@pytest.mark.parametrize("rows,cols,density,N,form", [
    (44800, 128, 0.3, 18, None), (44800, 128, 0.3, 16, B32), (44800, 500, 0.1, 18, B32), (30000, 64, 0.4, 18, B32), (44800, 128, 0.3, 31, B32),
    (64000, 300, 0.1, 32, None), (64000, 500, 0.1, 32, B32), (64000, 500, 0.1, 18, None), (64000, 1000, 0.1, 18, B32),
    (64000, 890, 0.1, 18, None), (64000, 910, 0.1, 18, B32), (70000, 890, 0.1, 18, B32), (70000, 700, 0.1, 18, None),
    (64000, 500, 0.1, 31, B32), (64000, 300, 0.1, 31, None), (64000, 300, 0.1, 1, None),
    (22400, 128, 0.3, 50, None), (22400, 160, 0.3, 50, E64), (22400, 128, 0.3, 56, E64),
    (9000, 300, 0.2, 18, B32), (9000, 300, 0.2, 24, A32), (9000, 300, 0.2, 13, B32), (9000, 2500, 0.1, 18, A32), (9000, 2000, 0.1, 18, B32), (9000, 2000, 0.1, 13, A32), (9000, 1900, 0.1, 13, B32),
    (8300, 4700, 0.1, 18, None), (8300, 4500, 0.1, 18, A32), (8300, 4700, 0.1, 24, A32), (11400, 4700, 0.1, 18, A32),
    (1440, 8192, 0.1, 200, None), (1440, 6000, 0.1, 200, A64), (1440, 8192, 0.1, 256, A64),
    (1200, 5000, 0.1, 500, None), (1200, 4500, 0.1, 500, B64), (4800, 6500, 0.1, 128, B64), (4800, 6500, 0.1, 100, None),
    (1200, 3500, 0.1, 1000, None), (1200, 3000, 0.1, 1000, E64), (9600, 4000, 0.1, 128, E64), (9600, 4000, 0.1, 100, None),
    (2000, 8192, 0.1, 1, None), (2000, 6900, 0.1, 1, A32), (2000, 8192, 0.1, 16, A32), (50000, 1000, 0.1, 13, None), (64000, 1000, 0.1, 13, B32),
])
def test_where_strips_end(rows, cols, density, N, form):
    from paper_2603_08734_amd import Plan
    A = matrix(rows, cols, density, holes=False)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, force_path=2, reorder=0, upload=0)
    assert plan.strip() == form
    plan.destroy()


@pytest.mark.parametrize("N,opts,form", [(16, {}, A32), (16, dict(window_rows=256), None), (16, dict(max_tiles_per_item=4), None), (700, {}, B64), (1024, {}, E64),
                                         (4096, {}, None)])
def test_plans_that_take_the_form(N, opts, form):
    """Only where the planner chooses the height and the parts, and while 64 x 64 tiles fill the chip once at most."""
    from paper_2603_08734_amd import Plan
    A = matrix(1100, 300, 0.2)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, force_path=2, reorder=0, upload=0, **opts)
    assert plan.strip() == form
    row_ptr, col_idx, val, path = plan.decode()
    assert np.array_equal(row_ptr, A.row_ptr) and np.array_equal(col_idx, A.col_idx) and np.array_equal(val, np.asarray(A.val).view(np.uint16))
    plan.destroy()

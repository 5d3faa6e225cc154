"""Residual rows whose lanes own rows of B or share them (rsh_narrow_kernel, rsh_shared_kernel): what a sum may lose, what lanes
read past the end of their rows, widths where only plans of rows of medium length take them, and windows beside them."""
import numpy as np
import pytest

from oracle import spmm as oracle
from workloads import from_coo

pytestmark = pytest.mark.gpu


def product(A, B, lanes, windows=False, **opts):
    import torch
    from paper_2603_08734_amd import Plan
    N = B.shape[1]
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, **opts)
    assert plan.kernels()["row_lanes"] == lanes and (plan.stats()["n_tile_items"] > 0) == windows
    Bd = torch.from_numpy(B).cuda()
    C = torch.full((A.n_rows, N), float("nan"), dtype=torch.float32, device="cuda")
    plan.spmm(Bd, C)
    torch.cuda.synchronize()
    plan.destroy()
    return C.cpu().numpy().astype(np.float64)


def rows_of(per_row, cols, seed):
    """Rows of the given numbers of entries, in random columns of 1 .. cols - 1."""
    rng = np.random.default_rng(seed)
    per_row = np.asarray(per_row)
    r = np.repeat(np.arange(per_row.size), per_row)
    step = (cols - 1) // per_row.max()
    c = 1 + np.concatenate([np.arange(k) for k in per_row]) * step + rng.integers(0, step, r.size)
    return r, c, rng.standard_normal(r.size)


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
    got = product(A, B, lanes, force_path=1)
    exact = 1.0 + 31 * 2.0 ** -25
    assert np.abs(got - exact).max() <= 2 * 2.0 ** -24 * exact


# A lane goes on past its row's last entry, through slots that name column 0 and through other rows' entries: rows of B that its
# own row does not name, infinite or not a number, must not count.  Every fiftieth row names them.
@pytest.mark.parametrize("N,lanes", [(1, 1), (3, 1), (4, 1), (8, 1), (11, 2), (16, 2), (32, 4), (31, 4), (48, 8), (64, 8)])
def test_rows_of_b_that_are_not_finite(N, lanes):
    rng = np.random.default_rng(N)
    rows, cols = 24000, 3000
    per_row = np.resize([1, 2, 3, 7, 8, 12, 15, 16, 17, 30, 31, 32, 33, 40], rows)
    r, c, v = rows_of(rng.permutation(per_row), cols, N)
    bad = rng.permutation(np.arange(0, rows, 50))
    r, c, v = np.concatenate([r, bad]), np.concatenate([c, np.zeros(bad.size, int)]), np.concatenate([v, np.ones(bad.size)])
    A = from_coo(r, c, v, rows, cols)
    B = rng.standard_normal((cols, N)).astype(np.float16)
    B[0, ::2], B[0, 1::2] = np.inf, np.nan
    print(f"case not finite N={N}", flush=True)
    got = product(A, B, lanes, force_path=1)
    B[0] = 0
    want, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    names = np.zeros(rows, bool)
    names[bad] = True
    assert np.all(np.abs(got[~names] - want[~names]) <= 1e-4 * S[~names])
    assert np.isposinf(got[names][:, ::2]).all() and np.isnan(got[names][:, 1::2]).all()


# From 33 to 63 features, except 48, eight lanes share rows where half of them are of medium length: rows of C and B that end at
# every even place inside the last lane's eight features, and odd ones beside the padded copy.
@pytest.mark.parametrize("N", [33, 38, 49, 50, 52, 54, 56, 62, 63])
def test_widths_where_half_of_the_rows_are_medium(N):
    rows, cols = 28000, 5000
    A = from_coo(*rows_of(np.resize([12, 9, 20, 0], rows), cols, N), rows, cols)
    B = np.random.default_rng(N).standard_normal((cols, N)).astype(np.float16)
    print(f"case medium rows N={N}", flush=True)
    got = product(A, B, 8, force_path=1)
    want, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    assert np.all(np.abs(got - want) <= 1e-4 * S)


# Windows and lanes in one plan, one after the other and on two streams.
@pytest.mark.parametrize("side_stream", [0, 1])
@pytest.mark.parametrize("N,lanes", [(5, 1), (12, 2), (16, 2), (20, 4), (32, 4), (48, 8), (64, 8)])
def test_windows_beside_lanes(N, lanes, side_stream):
    rng = np.random.default_rng(3)
    rows, cols = 34000, 40000
    r, c, v = rows_of(np.resize([12, 9, 20, 0, 2], rows), cols, 4)
    w = np.nonzero(rng.random((320, 48)) < 0.6)     # windows: 320 further rows, 16 to 48 columns
    r, c = np.concatenate([r, rows + w[0]]), np.concatenate([c, w[0] // 16 * 50 + w[1]])
    A = from_coo(r, c, np.concatenate([v, rng.standard_normal(w[0].size)]), rows + 320, cols)
    B = rng.standard_normal((cols, N)).astype(np.float16)
    print(f"case windows beside lanes N={N} side_stream={side_stream}", flush=True)
    got = product(A, B, lanes, windows=True, side_stream=side_stream, window_rows=16)
    want, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    assert np.all(np.abs(got - want) <= 1e-4 * S)


# Plans of fewer than 2^18 entries read rows of 3, 5 to 7 and 9 to 15 features where they lie, at their element's alignment: the
# last row ends with the allocation and every entry list names it.  Rows of every length, whole and in slices that leave partial
# sums; fp32 and binary16; canaries around C.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("N", [3, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15])
@pytest.mark.parametrize("opts", [{}, dict(max_nnz_per_slice=20), dict(xcd_partition_nnz=24)], ids=["whole", "slices", "xcd"])
def test_small_plans_read_rows_of_any_width_where_they_lie(opts, N, fused):
    import torch
    from paper_2603_08734_amd import Plan
    rng = np.random.default_rng(N)
    rows, cols = 3000, 701
    per_row = rng.permutation(np.resize([0, 1, 2, 3, 7, 16, 31, 33, 64, 65, 130], rows))
    r, c, v = rows_of(per_row, cols - 1, N)
    full = np.flatnonzero(per_row)
    r, c, v = np.concatenate([r, full]), np.concatenate([c, np.full(full.size, cols - 1)]), np.concatenate([v, rng.standard_normal(full.size)])
    A = from_coo(r, c, v, rows, cols)
    print(f"case rows in place N={N} opts={opts} fused={fused}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, cols, N, force_path=1, **opts)
    B = rng.standard_normal((cols, N)).astype(np.float16)
    flat = torch.full((rows * N + 129,), float("nan"), dtype=torch.float16 if fused else torch.float32, device="cuda")
    C = flat[65:65 + rows * N].view(rows, N)
    Bd = torch.empty(cols * N + 1, dtype=torch.float16, device="cuda")[1:].view(cols, N)
    Bd.copy_(torch.from_numpy(B))
    assert plan.operand(Bd.data_ptr(), C.data_ptr()) == (False, N)
    want, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    bound = 1e-4 * S
    if fused:
        bias = torch.linspace(-1, 1, N, device="cuda")
        plan.spmm_f16(Bd, C, bias, relu=True)
        want = np.maximum(want + bias.cpu().numpy().astype(np.float64), 0.0)
        bound = bound + 2.0 ** -24 * np.abs(want) + 2.0 ** -11 * np.abs(want) * 1.001 + 2.0 ** -24   # the bias, one rounding to binary16
    else:
        plan.spmm(Bd, C)
    torch.cuda.synchronize()
    plan.destroy()
    assert bool(torch.isnan(flat[:65]).all()) and bool(torch.isnan(flat[65 + rows * N:]).all()), "stores outside C"
    assert np.all(np.abs(C.cpu().numpy().astype(np.float64) - want) <= bound)


def test_products_go_to_the_current_stream():
    import torch
    from paper_2603_08734_amd import binding
    torch.zeros(1, device="cuda")
    side = torch.cuda.Stream()
    assert binding.current_stream() == torch.cuda.current_stream().cuda_stream != side.cuda_stream
    with torch.cuda.stream(side):
        assert binding.current_stream() == side.cuda_stream
    assert binding.current_stream() == torch.cuda.current_stream().cuda_stream

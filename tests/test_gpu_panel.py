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


# Beyond 128 features windows of 256 rows run on cells written out (at 1 / 16 of them and more).  Fragments per window: 1 and
# 3 (fewer than a turn of the loop), 5, 33 (one past the second level of sums), 36; the last one full or with one column; parts
# of 3 and 7 fragments begin anywhere; gathered columns and runs.  Widths: one feature into the second panel, rows of B that
# end at every place inside a 16-byte piece, odd ones beside the padded copy, a whole last panel.  Canaries around C.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("N", [129, 130, 132, 134, 136, 160, 255, 256, 300])
@pytest.mark.parametrize("rows,cols,parts,density", [(256, 32, 0, 0.5), (300, 65, 0, 0.3), (520, 160, 3, 1.0), (257, 1025, 0, 0.15), (256, 1152, 7, 0.08)])
def test_cells_written_out(rows, cols, parts, density, N, fused):
    import torch
    from paper_2603_08734_amd import Plan
    A = random_matrix(rows, cols, density, 7)
    print(f"case wide rows={rows} cols={cols} parts={parts} N={N} fused={fused}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, window_rows=256, force_path=2, max_tiles_per_item=parts)
    st = plan.stats()
    assert st["nnz_tile"] * 16 >= st["n_tiles"] * 32 * 256 and st["tile_part_bytes"] >= 8192 * (2 * st["n_tiles"] + 1)
    B = dense_B(A.n_cols, N, "normal", seed=N)
    Bd = torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16)
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    pad = 64
    flat = torch.full((A.n_rows * N + 2 * pad,), float("nan"), dtype=torch.float16 if fused else torch.float32, device="cuda")
    C = flat[pad:pad + A.n_rows * N].view(A.n_rows, N)
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


# Even widths that are not multiples of 16 run without copies of the operands: rows end inside 16-byte pieces of
# B (8 features) and of C (4 features), inside a feature panel, and one or two pieces into one.  Every kernel takes
# them: windows of 16 rows, tall windows (128-row ones in panels of their own), residual rows of all kinds with
# their combine pass, empty rows.  B and C end with their allocation's last row, canaries follow C.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("N", [16, 18, 22, 50, 100, 124, 126, 130, 134, 258, 300])
@pytest.mark.parametrize("opts", [dict(force_path=2), dict(force_path=2, window_rows=128), dict(force_path=2, window_rows=256, max_tiles_per_item=3),
                                  dict(force_path=1, max_nnz_per_slice=40), dict(force_path=1, xcd_partition_nnz=32)],
                         ids=["tile", "w128", "w256", "residual", "xcd"])
def test_even_widths_without_copies(opts, N, fused):
    import torch
    from paper_2603_08734_amd import Plan
    rng = np.random.default_rng(11)
    dense = rng.random((90, 333)) < np.linspace(0.0, 0.4, 90)[:, None]     # row 0 is empty, rows of every length
    r, c = np.nonzero(dense)
    A = from_coo(r, c, rng.standard_normal(r.size), 90, 333)
    print(f"case width N={N} opts={opts} fused={fused}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, **opts)
    B = dense_B(A.n_cols, N, "normal", seed=N)
    Bd = torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16)
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    dtype, pad = (torch.float16 if fused else torch.float32), 64
    flat = torch.full((A.n_rows * N + pad,), float("nan"), dtype=dtype, device="cuda")
    C = flat[:A.n_rows * N].view(A.n_rows, N)
    if fused:
        bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32)).cuda()
        plan.spmm_f16(Bd, C, bias, relu=True)
        C_ref = np.maximum(C_ref + bias.cpu().numpy().astype(np.float64), 0.0)
        # the fp32 bound, the addition of the bias, one rounding to binary16
        bound = 1e-4 * S + 2.0 ** -24 * np.abs(C_ref) + 2.0 ** -11 * np.abs(C_ref) * 1.001 + 2.0 ** -24
    else:
        plan.spmm(Bd, C)
        bound = 1e-4 * S
    torch.cuda.synchronize()
    assert bool(torch.isnan(flat[A.n_rows * N:]).all()), "stores past the end of C"
    got = C.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any()
    assert np.all(np.abs(got - C_ref) <= bound)
    plan.destroy()


# Odd widths, widths below 16 and operands aligned to their element only: B is copied to the run width, rows of C are
# written as they are.  Rows end inside the pieces of 4 (fp32) and 8 (binary16) features, with one feature in the
# last panel, and with whole panels; C and B begin one element past a 16-byte boundary, canaries stand on both sides
# of C, and the bias ends with its allocation's last element.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("N", [1, 2, 3, 5, 8, 15, 17, 33, 64, 65, 127, 129, 257])
@pytest.mark.parametrize("opts", [dict(force_path=2), dict(force_path=2, window_rows=64, max_tiles_per_item=2),
                                  dict(force_path=2, window_rows=128), dict(force_path=2, window_rows=256, max_tiles_per_item=3),
                                  dict(force_path=1, max_nnz_per_slice=40), dict(force_path=1, xcd_partition_nnz=32)],
                         ids=["tile", "w64", "w128", "w256", "residual", "xcd"])
def test_rows_of_c_of_any_width_and_alignment(opts, N, fused):
    import torch
    from paper_2603_08734_amd import Plan
    rng = np.random.default_rng(13)
    dense = rng.random((90, 333)) < np.linspace(0.0, 0.4, 90)[:, None]     # row 0 is empty, rows of every length
    r, c = np.nonzero(dense)
    A = from_coo(r, c, rng.standard_normal(r.size), 90, 333)
    print(f"case any width N={N} opts={opts} fused={fused}", flush=True)
    run_width = N if N % 16 else N + 16     # a chosen run width takes multiples of 16 through the copy as well
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, run_width=(run_width + 15) // 16 * 16, **opts)
    B = dense_B(A.n_cols, N, "normal", seed=N)
    Bd = torch.empty(A.n_cols * N + 1, dtype=torch.float16, device="cuda")[1:].view(A.n_cols, N)
    Bd.copy_(torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16))
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    dtype, pad = (torch.float16 if fused else torch.float32), 65
    flat = torch.full((A.n_rows * N + 2 * pad,), float("nan"), dtype=dtype, device="cuda")
    C = flat[pad:pad + A.n_rows * N].view(A.n_rows, N)
    if fused:
        bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32)).cuda()
        plan.spmm_f16(Bd, C, bias, relu=True)
        C_ref = np.maximum(C_ref + bias.cpu().numpy().astype(np.float64), 0.0)
        # the fp32 bound, the addition of the bias, one rounding to binary16
        bound = 1e-4 * S + 2.0 ** -24 * np.abs(C_ref) + 2.0 ** -11 * np.abs(C_ref) * 1.001 + 2.0 ** -24
    else:
        plan.spmm(Bd, C)
        bound = 1e-4 * S
    torch.cuda.synchronize()
    assert bool(torch.isnan(flat[:pad]).all()) and bool(torch.isnan(flat[pad + A.n_rows * N:]).all()), "stores outside C"
    got = C.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any()
    assert np.all(np.abs(got - C_ref) <= bound)
    plan.destroy()


# Partial sums of windows' rows of up to 16 features are added by teams of lanes, several rows to a wave (16 features: 16,
# one to four features: 64); wider ones and those of long rows' slices take a wave a row.  600 rows of three or more parts fill several workgroups
# and leave the last one ragged at every width.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("N", [1, 4, 5, 8, 9, 16, 17, 32, 128])
@pytest.mark.parametrize("opts", [dict(force_path=2, max_tiles_per_item=3), dict(force_path=1, max_nnz_per_slice=16)], ids=["windows", "rows"])
def test_partial_sums_of_several_rows_in_a_wave(opts, N, fused):
    import torch
    from paper_2603_08734_amd import Plan
    A = random_matrix(600, 400, 0.2, 17)
    print(f"case partial sums N={N} opts={opts} fused={fused}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, **opts)
    assert plan.stats()["n_combine"] >= 500
    B = dense_B(A.n_cols, N, "normal", seed=N)
    Bd = torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16)
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    C = torch.full((A.n_rows, N), float("nan"), dtype=torch.float16 if fused else torch.float32, device="cuda")
    if fused:
        plan.spmm_f16(Bd, C, None, False)
        bound = 1e-4 * S + 2.0 ** -11 * np.abs(C_ref) * 1.001 + 2.0 ** -24   # the fp32 bound and one rounding to binary16
    else:
        plan.spmm(Bd, C)
        bound = 1e-4 * S
    torch.cuda.synchronize()
    got = C.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any()
    assert np.all(np.abs(got - C_ref) <= bound)
    plan.destroy()


# Windows that the planner cuts into different numbers of parts, and not at all, in one product.
@pytest.mark.parametrize("N", [1, 128, 300])
@pytest.mark.parametrize("window_rows", [128, 256])
def test_windows_cut_into_different_numbers_of_parts(window_rows, N):
    import torch
    from paper_2603_08734_amd import Plan, binding
    rng = np.random.default_rng(23)
    dense = rng.random((5 * window_rows - 7, 3000)) < np.repeat([0.1, 0.001, 0.02, 0.0002, 0.01], window_rows)[:-7, None]
    r, c = np.nonzero(dense)
    A = from_coo(r, c, rng.standard_normal(r.size), dense.shape[0], 3000)
    print(f"case uneven W={window_rows} N={N}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, window_rows=window_rows, force_path=2, reorder=0)
    parts = np.bincount(plan.array(binding.RSH_ARR_TILE_ITEM).reshape(-1, 4)[:, 0])
    assert len(set(parts)) >= 4 and parts.min() == window_rows // 128
    B = dense_B(A.n_cols, N, "normal", seed=N)
    Bd = torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16)
    C = torch.full((A.n_rows, N), float("nan"), dtype=torch.float32, device="cuda")
    plan.spmm(Bd, C)
    torch.cuda.synchronize()
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    got = C.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any()
    assert np.all(np.abs(got - C_ref) <= 1e-4 * S)
    plan.destroy()


# More than 2048 waves of fragments: a narrower last panel of features then takes a launch of its own (fewer go along with
# the others).  Its panel ends with the row: at 130 and 146 features it begins at an even feature inside the panel before, at
# 160 behind it; 65 and 257 features run beside a padded copy of B, of which the last panel holds one feature that counts.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("N", [65, 130, 146, 160, 257])
@pytest.mark.parametrize("window_rows", [16, 64])
def test_a_narrower_last_panel_in_a_launch_of_its_own(window_rows, N, fused):
    import torch
    from paper_2603_08734_amd import Plan
    from workloads import stencil27
    A = stencil27(40)
    print(f"case last panel W={window_rows} N={N} fused={fused}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, window_rows=window_rows, force_path=2)
    assert plan.stats()["n_tile_items"] * (window_rows // 16) > 2048
    B = dense_B(A.n_cols, N, "normal", seed=N)
    Bd = torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16)
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    dtype, pad = (torch.float16 if fused else torch.float32), 64
    flat = torch.full((A.n_rows * N + 2 * pad,), float("nan"), dtype=dtype, device="cuda")
    C = flat[pad:pad + A.n_rows * N].view(A.n_rows, N)
    if fused:
        bias = torch.linspace(-1, 1, N, device="cuda")
        plan.spmm_f16(Bd, C, bias, relu=True)
        C_ref = np.maximum(C_ref + bias.cpu().numpy().astype(np.float64), 0.0)
        # the fp32 bound, the addition of the bias, one rounding to binary16
        bound = 1e-4 * S + 2.0 ** -24 * np.abs(C_ref) + 2.0 ** -11 * np.abs(C_ref) * 1.001 + 2.0 ** -24
    else:
        plan.spmm(Bd, C)
        bound = 1e-4 * S
    torch.cuda.synchronize()
    assert bool(torch.isnan(flat[:pad]).all()) and bool(torch.isnan(flat[pad + A.n_rows * N:]).all()), "stores outside C"
    got = C.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any()
    assert np.all(np.abs(got - C_ref) <= bound)
    plan.destroy()


# Rows of up to 16 features (lanes own rows, or share them in pairs).  Rows of 0 .. 2000 entries: empty, one to a lane with an odd
# and an even number of entries, at both sides of every doubling of the lanes that share one, sliced with partial sums; few rows (a
# lane takes two entries) and many (16); column groups; beside windows that read a copy of 16 features.  B and C begin one element
# past a 16-byte boundary in `odd`: then widths that are a power of two go through the copy too.
# From 17 features on four or eight lanes share a row, in plans of 2^18 entries and more: widths that fill the lanes, end at
# every place inside the last one's eight features, and odd ones beside the padded copy.
FEW = [(90, {}), (90, dict(max_nnz_per_slice=40)), (90, dict(xcd_partition_nnz=32)), (90, dict(window_rows=16, min_reuse=0.0))]
MANY = [(20000, dict(force_path=1)), (20000, dict(force_path=1, max_nnz_per_slice=20)), (20000, dict(force_path=1, xcd_partition_nnz=32))]


@pytest.mark.parametrize("fused,odd", [(False, 0), (False, 1), (True, 0)])
@pytest.mark.parametrize("rows,opts,N", [(*p, n) for p in FEW + MANY[:1] for n in (1, 2, 3, 4, 5, 8, 9, 16)] +
                         [(*p, n) for p in MANY for n in (17, 18, 24, 30, 31, 32, 34, 47, 48, 64)])
def test_narrow_rows(rows, opts, N, fused, odd):
    import torch
    from paper_2603_08734_amd import Plan
    rng = np.random.default_rng(13)
    lengths = np.array([0, 1, 2, 3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 128, 129, 500, 2000])
    if rows > 100:
        lengths = lengths[lengths <= 65]
    per_row = rng.permutation(np.resize(lengths, rows))
    r = np.repeat(np.arange(rows), per_row)
    c = np.concatenate([rng.choice(3000, k, replace=False) if k > 100 else (rng.integers(0, 2900) + rng.permutation(100)[:k]) for k in per_row])
    A = from_coo(r, c, rng.standard_normal(r.size), rows, 3000)
    if N % 16 == 0 and odd:
        pytest.skip("rows of a multiple of 16 features have to be 16-byte aligned")
    print(f"case narrow rows={rows} {opts} N={N} fused={fused} odd={odd}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, **opts)
    assert plan.kernels()["row_lanes"] == (1 if N <= 8 else 2 if N <= 16 else 4 if N <= 32 else 8)
    assert plan.stats()["nnz_irregular"] == A.nnz or rows < 100
    assert plan.stats()["n_scratch_slots"] > 0 or "max_nnz_per_slice" not in opts and "xcd_partition_nnz" not in opts
    B = dense_B(A.n_cols, N, "normal", seed=N)
    Bd = torch.empty(B.size + odd, dtype=torch.float16, device="cuda")[odd:].view(A.n_cols, N)
    Bd.copy_(torch.from_numpy(B.view(np.float16) if B.dtype != np.float16 else B))
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    pad = 64
    flat = torch.full((rows * N + 2 * pad,), float("nan"), dtype=torch.float16 if fused else torch.float32, device="cuda")
    C = flat[pad + odd:pad + odd + rows * N].view(rows, N)
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
    assert bool(torch.isnan(flat[:pad + odd]).all()) and bool(torch.isnan(flat[pad + odd + rows * N:]).all()), "stores outside C"
    got = C.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any()
    assert np.all(np.abs(got - C_ref) <= bound)
    plan.destroy()


# Tall windows read rows of fewer than 16 features where they lie: runs of columns and gathered ones, up to the last row of B,
# whose eight features are read where they end with it; 9 columns of 1 feature are hardly more than one piece, 7 less.  An empty
# row makes a residual part, beside which B is copied.
@pytest.mark.parametrize("fused,odd", [(False, 0), (False, 1), (True, 1)])
@pytest.mark.parametrize("N", [1, 2, 3, 7, 8, 9, 11, 15])
@pytest.mark.parametrize("window_rows", [128, 256])
@pytest.mark.parametrize("cols,density,empty", [(400, 0.3, False), (1500, 0.02, False), (9, 1.0, False), (7, 1.0, False), (130, 0.3, True)])
def test_tall_windows_of_narrow_rows(cols, density, empty, window_rows, N, fused, odd):
    import torch
    from paper_2603_08734_amd import Plan
    rng = np.random.default_rng(9)
    cells = rng.random((300, cols)) < density
    cells[:, -1] = True
    if empty:
        cells[17] = False
    r, c = np.nonzero(cells)
    A = from_coo(r, c, rng.standard_normal(r.size), 300, cols)
    print(f"case tall narrow cols={cols} W={window_rows} N={N} fused={fused} odd={odd}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, window_rows=window_rows, force_path=2)
    B = dense_B(A.n_cols, N, "normal", seed=N)
    Bd = torch.empty(B.size + odd, dtype=torch.float16, device="cuda")[odd:].view(A.n_cols, N)
    Bd.copy_(torch.from_numpy(B.view(np.float16) if B.dtype != np.float16 else B))
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    pad = 64
    flat = torch.full((300 * N + 2 * pad,), float("nan"), dtype=torch.float16 if fused else torch.float32, device="cuda")
    C = flat[pad + odd:pad + odd + 300 * N].view(300, N)
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
    assert bool(torch.isnan(flat[:pad + odd]).all()) and bool(torch.isnan(flat[pad + odd + 300 * N:]).all()), "stores outside C"
    got = C.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any()
    assert np.all(np.abs(got - C_ref) <= bound)
    plan.destroy()


# A chosen run width above 16 beside few features: B is copied to it, and lanes that share a row read the copy.
@pytest.mark.parametrize("run_width", [32, 64])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 7])
def test_chosen_run_width_of_few_features(N, run_width):
    import torch
    from paper_2603_08734_amd import Plan
    rng = np.random.default_rng(4)
    rows, cols = 24000, 20000
    r = np.repeat(np.arange(rows), 12)
    A = from_coo(r, 1600 * np.tile(np.arange(12), rows) + rng.integers(0, 1600, r.size), rng.standard_normal(r.size), rows, cols)
    print(f"case run width {run_width} N={N}", flush=True)
    plan = Plan(A.row_ptr, A.col_idx, A.val, cols, N, run_width=run_width, force_path=1)
    assert plan.kernels()["row_lanes"] == 4
    B = dense_B(cols, N, "normal", seed=N)
    Bd = torch.from_numpy(B.view(np.int16)).cuda().view(torch.float16)
    assert plan.operand(Bd.data_ptr(), 4096) == (True, run_width)
    pad = 64
    flat = torch.full((rows * N + 2 * pad,), float("nan"), dtype=torch.float32, device="cuda")
    C = flat[pad:pad + rows * N].view(rows, N)
    plan.spmm(Bd, C)
    torch.cuda.synchronize()
    C_ref, S, _ = oracle.spmm(A.row_ptr, A.col_idx, A.val, B)
    assert bool(torch.isnan(flat[:pad]).all()) and bool(torch.isnan(flat[pad + rows * N:]).all()), "stores outside C"
    assert np.all(np.abs(C.cpu().numpy().astype(np.float64) - C_ref) <= 1e-4 * S)
    plan.destroy()

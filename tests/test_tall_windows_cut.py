"""How tall windows (128 or 256 rows) are cut into work items when the caller leaves it open (host plans, no GPU)."""
import numpy as np
import pytest

from paper_2603_08734_amd import Plan, binding


def plan_of(blocks, cols, N, window_rows):
    """Plan of a matrix of blocks (rows, about so many entries a row), in the given row order."""
    rng = np.random.default_rng(1)
    rows = [np.unique(rng.integers(0, cols, per_row)).astype(np.int32) for n, per_row in blocks for _ in range(n)]
    row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    col_idx = np.concatenate(rows)
    return Plan(row_ptr, col_idx, np.ones(len(col_idx), np.float16), cols, N, window_rows=window_rows, force_path=2, reorder=0, upload=0)


def item_lengths(plan):
    """{window: fragments of its items}"""
    out = {}
    for w, b, e, _ in plan.array(binding.RSH_ARR_TILE_ITEM).reshape(-1, 4):
        out.setdefault(int(w), []).append(int(e) - int(b))
    return out


# a launch lasts as long as its longest item: windows three and nine times longer than the rest, at one and at several
# feature panels; and windows without much in them behind long ones
@pytest.mark.parametrize("N", [1, 128, 512])
@pytest.mark.parametrize("blocks,cols", [([(16 * 256, 41), (240 * 256, 8)], 8192), ([(8 * 256, 400), (120 * 256, 4)], 8192),
                                         ([(2560, 400), (1536, 2)], 8192)])
def test_uneven_tall_windows_are_cut_by_their_own_length(blocks, cols, N):
    plan = plan_of(blocks, cols, N, 256)
    items, st = item_lengths(plan), plan.stats()
    assert st["window_rows"] == 256
    # no item above one and a half times what every one of 256 workgroups gets, or the start and end of three
    load = st["n_tiles"] * -(-N // 128) / 256
    assert max(max(v) for v in items.values()) <= max(64, 1.5 * load)
    for v in items.values():     # cut between quads of fragments, and no part below four of them (the last may be ragged)
        assert sum(v) == 0 or all(x % 4 == 0 for x in v[:-1])
        assert len(v) == 1 or (min(v[:-1]) >= 16 and v[-1] >= 13)
    plan.destroy()


def test_two_workgroups_of_128_rows_share_a_compute_unit():
    plan = plan_of([(56 * 128, 205)], 4096, 128, 128)      # 56 windows of 128 fragments
    lengths = [x for v in item_lengths(plan).values() for x in v]
    assert plan.stats()["n_windows"] == 56 and 256 < len(lengths) <= 512 and max(lengths) == 16
    plan.destroy()


def test_panels_of_64_features_count_as_workgroups():
    """Rows of B that end inside a 16-byte piece run in panels of 64 features where the window has 128 rows."""
    wide, ragged = (plan_of([(56 * 128, 205)], 4096, N, 128) for N in (104, 100))
    assert ragged.stats()["n_tile_items"] * 2 <= 512 < wide.stats()["n_tile_items"] * 2
    for p in (wide, ragged):
        p.destroy()


def test_chosen_parts_fit_the_library_owned_array():
    """Parts that the planner chooses by itself keep no product from rsh_spmm_noalloc (64 MiB of partial sums)."""
    plan = plan_of([(70 * 256, 480)], 32000, 256, 256)
    st = plan.stats()
    assert st["n_split_windows"] > 0 and st["n_scratch_slots"] * st["N"] * 4 <= 64 << 20
    plan.destroy()


# 40 equal windows at seven panels of features are 35 workgroups for every 32 compute units: a second round, which ends
# sooner when its windows are cut; at one panel all parts run at once
@pytest.mark.parametrize("N,cut", [(896, True), (770, True), (128, False)])
def test_the_last_windows_of_a_part_are_cut_further_where_a_round_is_left_nearly_empty(N, cut):
    plan = plan_of([(40 * 256, 150)], 4096, N, 256)
    items = item_lengths(plan)
    counts = {len(v) for v in items.values()}
    assert (len(counts) > 1) == cut and all(sum(v) == 128 for v in items.values())
    if cut:      # whole windows first in every eighth of the list
        parts = [len(items[w]) for w in dict.fromkeys(plan.array(binding.RSH_ARR_TILE_ITEM).reshape(-1, 4)[:, 0].tolist())]
        assert min(parts) == 1 and all(parts[5 * x] == 1 and parts[5 * x + 4] > 1 for x in range(8))
    plan.destroy()

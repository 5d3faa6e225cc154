"""bench.py may quote counter traffic only from a profile summary made for exactly the workload,
feature width, plan options and library sources it is timing (paper_2603_08734_amd/profiles.py)."""
import json

import numpy as np
import pytest

import bench
from paper_2603_08734_amd import Plan, build, profiles
from workloads import from_coo


def _write(dirname, name, **over):
    data = {"workload": "w", "N": 128, "plan_options": {}, "library_sources": build.source_digest(),
            "bench_args": "--config 2",
            "kernels": {"rsh::rsh_irregular_kernel<16, rsh::OutFused, false>": {"fetched_bytes": 7, "written_bytes": 1},
                        "rsh::rsh_irregular_kernel<16, rsh::OutPlain, false>": {"fetched_bytes": 100, "written_bytes": 20},
                        "rsh::rsh_combine_kernel<rsh::OutPlain>": {"fetched_bytes": 5, "written_bytes": 5}}}
    data.update(over)
    (dirname / name).write_text("# summary\n\n" + profiles._MARK + "\n```json\n" + json.dumps(data) + "\n```\n")


def test_lookup_matches_workload_width_options_and_sources(tmp_path, monkeypatch):
    monkeypatch.setattr(profiles, "PROFILE_DIR", str(tmp_path))
    _write(tmp_path, "a.md")
    (tmp_path / "notes.md").write_text("no data block here\n")
    got = profiles.lookup("w", 128, {}, "rsh_irregular_kernel")
    assert got == (120, "a.md", "rsh::rsh_irregular_kernel<16, rsh::OutPlain, false>")
    assert profiles.lookup("w", 64, {}, "rsh_irregular_kernel") is None
    assert profiles.lookup("other", 128, {}, "rsh_irregular_kernel") is None
    assert profiles.lookup("w", 128, {"min_reuse": "1.0"}, "rsh_irregular_kernel") is None
    assert profiles.lookup("w", 128, {}, "rsh_tile_kernel") is None


def test_lookup_refuses_a_summary_of_other_sources(tmp_path, monkeypatch):
    monkeypatch.setattr(profiles, "PROFILE_DIR", str(tmp_path))
    _write(tmp_path, "a.md", library_sources="0" * 64)
    assert profiles.lookup("w", 128, {}, "rsh_irregular_kernel") is None


def test_lookup_prefers_the_plain_command(tmp_path, monkeypatch):
    monkeypatch.setattr(profiles, "PROFILE_DIR", str(tmp_path))
    _write(tmp_path, "a_epilogue.md", bench_args="--config 2 --epilogue")
    _write(tmp_path, "b.md")
    assert profiles.lookup("w", 128, {}, "rsh_irregular_kernel")[1] == "b.md"


def test_committed_summaries_parse():
    names = [name for name, data in profiles._blocks() if {"workload", "N", "plan_options", "kernels"} <= set(data)]
    assert names, "profiles/ holds no summary in the format bench.py reads"


def test_kernel_names_keep_what_follows_an_anonymous_namespace():
    assert profiles._short("void rsh::(anonymous namespace)::rsh_panel_kernel<4, 8, false, rsh::OutPlainT<false> >(uint4 const*, int)") == \
        "rsh::rsh_panel_kernel<4, 8, false, rsh::OutPlainT<false> >"
    assert profiles._short("rsh::rsh_copy_probe_kernel(uint4 const*)") == "rsh::rsh_copy_probe_kernel"


@pytest.mark.parametrize("lengths,N,opts,names", [
    ({5: 60000}, 48, dict(force_path=1), ("rsh_tile_kernel", "rsh_irregular_kernel")),      # 2^18 entries, no row of medium length
    ({12: 30000}, 56, dict(force_path=1), ("rsh_tile_kernel", "rsh_shared_kernel")),
    ({12: 300}, 12, dict(force_path=1), ("rsh_tile_kernel", "rsh_shared_kernel")),
    ({12: 300}, 8, dict(force_path=1), ("rsh_tile_kernel", "rsh_narrow_kernel")),
    ({300: 512}, 256, dict(window_rows=256, force_path=2), ("rsh_wide_kernel", "rsh_irregular_kernel")),
    ({300: 512}, 256, dict(window_rows=128, force_path=2), ("rsh_panel_kernel", "rsh_irregular_kernel")),
])
def test_bench_names_the_kernels_that_the_plan_runs(lengths, N, opts, names):
    rng = np.random.default_rng(1)
    per_row = np.repeat(list(lengths), list(lengths.values()))
    r = np.repeat(np.arange(per_row.size), per_row)
    c = np.concatenate([np.arange(k) for k in per_row]) * 4 + rng.integers(0, 4, r.size)
    A = from_coo(r, c, rng.standard_normal(r.size), per_row.size, 2000)
    plan = Plan(A.row_ptr, A.col_idx, A.val, A.n_cols, N, upload=0, reorder=0, **opts)
    assert bench.kernel_names(plan) == names
    plan.destroy()

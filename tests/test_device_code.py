"""Checks on the compiled gfx950 code of the kernels (no GPU needed: hipcc cross-compiles).

The streaming-store hint on rows of C is easy to lose -- the compiler folds a hinted store with an
unhinted one on a sibling path and keeps neither hint -- and a change in register pressure can
push a kernel into scratch memory without any test of results noticing.  Both show in the
assembly."""
import os
import re
import subprocess

import pytest

from paper_2603_08734_amd import build as B


@pytest.fixture(scope="module")
def kernels_asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("isa") / "kernels.s"
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-shared")]
    src = os.path.join(B.CSRC, "kernels.hip")
    inc = os.path.join(B.HERE, "..", "include")
    subprocess.check_call([B.HIPCC, *flags, "-I", inc, "-S", "--cuda-device-only", "-o", str(out), src],
                          stderr=subprocess.DEVNULL)
    text = out.read_text()
    kernels = {}
    for chunk in re.split(r"\n\s*\.globl\s+", text)[1:]:
        name = chunk.split("\n", 1)[0].strip()
        end = chunk.find(".end_amdhsa_kernel")
        if end < 0:
            continue
        kernels[name] = chunk[:end]
    return kernels


def _stores(body):
    st = [l for l in body.splitlines() if "global_store_dwordx4" in l]
    return len(st), sum(" nt" in l for l in st)


def test_rows_of_c_leave_with_the_streaming_hint(kernels_asm):
    tile = {n: b for n, b in kernels_asm.items() if "rsh_tile_kernel" in n}
    irregular = {n: b for n, b in kernels_asm.items() if "rsh_irregular_kernel" in n}
    combine = {n: b for n, b in kernels_asm.items() if "rsh_combine_kernel" in n}
    # every kernel exists twice: fp32 sums (OutPlain) and the fused binary16 epilogue (OutFused);
    # the irregular kernel, for teams of four, eight and sixteen lanes, once more for a partial last feature panel
    assert len(tile) >= 60 and len(irregular) == 12 and len(combine) == 2
    for name, body in tile.items():
        n, nt = _stores(body)
        if "OutFused" in name:
            # scratch path: one ordinary store per 16-feature chunk; C path: the wave's 16 rows of
            # binary16 leave as 16 * (2 * chunks) 16-byte pieces, 64 per streaming store
            nch = int(re.search(r"rsh_tile_kernelILi(\d+)E", name).group(1))
            assert n - nt == nch and nt == max(1, nch // 2), f"{name}: {nt} streaming of {n} stores"
        else:
            assert n > 0 and nt * 2 == n, f"{name}: {nt} of {n} stores are streaming (C path streaming, scratch path ordinary)"
    for name, body in irregular.items():
        n, nt = _stores(body)
        assert n > 0 and nt == n, f"{name}: {nt} of {n} stores are streaming"
    for name, body in combine.items():
        st = [l for l in body.splitlines() if "global_store_dword" in l]
        want = "global_store_dwordx2" if "OutFused" in name else "global_store_dwordx4"
        assert st and all(want in l and " nt" in l for l in st), f"{name}: {st}"


def test_rows_of_even_widths_leave_with_the_streaming_hint(kernels_asm):
    """The kernels for rows that are not a multiple of 16 features keep the hint as those above do."""
    seen = {"fragment_even": 0, "residual_even": 0, "sum_even": 0}
    for name, body in kernels_asm.items():
        kind = next((k for k in seen if f"rsh_{k}_kernel" in name), None)
        if kind is None:
            continue
        seen[kind] += 1
        st = [l for l in body.splitlines() if "global_store_dwordx" in l]
        nt = sum(" nt" in l for l in st)
        # fragments: partial sums leave with ordinary stores, one per 16-feature chunk
        ordinary = int(re.search(r"rsh_fragment_even_kernelILi(\d+)E", name).group(1)) if kind == "fragment_even" else 0
        assert nt > 0 and len(st) - nt == ordinary, f"{name}: {nt} of {len(st)} stores are streaming"
    assert seen["fragment_even"] >= 60 and seen["residual_even"] == 6 and seen["sum_even"] == 2


def test_kernels_keep_their_registers(kernels_asm):
    for name, body in kernels_asm.items():
        m = re.search(r"\.amdhsa_private_segment_fixed_size\s+(\d+)", body)
        assert m, name
        spill = int(m.group(1))
        limit = 24 if "rsh_irregular_kernel" in name else 0     # a few registers of the 8-wave irregular kernel, outside its gather loops
        assert spill <= limit, f"{name} uses {spill} bytes of scratch per lane"


def test_tile_loop_waits_do_not_drain_global_loads(kernels_asm):
    """Inside the fragment loop of the 16-row tile kernels no wait may be vmcnt(0) together with
    outstanding prefetches: the generic fences did exactly that.  The loop is the code between the
    loop header label and its backward branch; it must contain MFMA and no `s_barrier`-less
    `vmcnt(0)` beyond the one that precedes staging of the single in-flight fragment."""
    name = next(n for n in kernels_asm if "rsh_tile_kernelILi8ELi4ELi2ELi32E" in n)   # 64-row windows, ring of two
    body = kernels_asm[name]
    loop = body[body.index("Inner Loop Header"):]
    loop = loop[:loop.index("s_endpgm")] if "s_endpgm" in loop else loop
    waits = re.findall(r"s_waitcnt vmcnt\((\d+)\)", loop[:loop.index("s_cbranch_scc")])
    assert waits and all(int(w) > 0 for w in waits), waits


def test_panel_kernels_use_the_32_row_mfma_and_transposing_reads(kernels_asm):
    """Windows of 128 or 256 rows: the product is formed by v_mfma_f32_32x32x16_f16 with the staged
    B tile read through the transposing LDS load, entries arrive as 16-byte loads, and rows of C
    leave as streaming 16-byte stores (partial sums as ordinary ones)."""
    panel = {n: b for n, b in kernels_asm.items() if "rsh_panel_kernel" in n or "rsh_wide_kernel" in n}
    assert panel and sum("rsh_wide_kernel" in n for n in panel) == 6
    for name, body in panel.items():
        assert "v_mfma_f32_32x32x16_f16" in body and "ds_read_b64_tr_b16" in body, name
        assert "global_load_dwordx4" in body and ("ds_write_b16" in body or "rsh_wide_kernel" in name), name
        n, nt = _stores(body)   # each kernel holds both ends: rows of C (streaming) and partial sums (ordinary)
        if "OutPlain" in name:
            assert n > 0 and nt * 2 == n, f"{name}: {nt} of {n} stores are streaming"
        else:   # binary16 rows of C are half as wide
            assert any("global_store_dword" in l and " nt" in l for l in body.splitlines()), name


def test_strips_leave_with_the_streaming_hint(kernels_asm):
    """Every store of a strip is one of C: no partial sums pass through memory."""
    strips = {n: b for n, b in kernels_asm.items() if "rsh_strip_kernel" in n}
    assert len(strips) == 40   # five forms, broken pieces or none, rows of even or any width, fp32 or binary16
    for name, body in strips.items():
        st = [l for l in body.splitlines() if "global_store" in l]
        assert st and all(" nt" in l for l in st), f"{name}: {st}"
        assert "v_mfma_f32_32x32x16_f16" in body and "ds_read_b64_tr_b16" in body, name


def _registers(operand):
    m = re.match(r"([va])(?:(\d+)|\[(\d+):(\d+)\])$", operand)
    return {(m.group(1), i) for i in range(int(m.group(2) or m.group(3)), int(m.group(2) or m.group(4)) + 1)} if m else set()


def test_no_register_is_restored_for_some_lanes_only(kernels_asm):
    """A value that is copied away and copied back with fewer lanes running in between is lost in the others; nested
    conditions that end together have made the compiler do that to the row numbers that lanes take from each other."""
    copy = re.compile(r"(?:v_mov_b32_e32|v_accvgpr_write_b32|v_accvgpr_read_b32|v_accvgpr_mov_b32) ([va]\d+), ([va]\d+)$")
    for name, body in kernels_asm.items():
        if not any(k in name for k in ("rsh_wide_kernel", "rsh_panel_kernel", "rsh_strip_kernel")):
            continue
        held = {}      # register: (copied from, conditions opened since)
        for line in (l.strip() for l in body.splitlines()):
            if line.startswith(("s_and_b64 exec, exec", "s_and_saveexec")):
                held = {r: (src, n + 1) for r, (src, n) in held.items()}
            elif line.startswith(("s_or_b64 exec, exec", "s_mov_b64 exec")):
                held = {r: (src, max(0, n - 1)) for r, (src, n) in held.items()}
            m = copy.match(line)
            if m:
                kept = held.get(m.group(2))
                assert not (kept and kept[0] == m.group(1) and kept[1] > 0), f"{name}: {line}"
            if line.startswith("v_") or "_load" in line or line.startswith("ds_read") or line.startswith("ds_bpermute"):
                for kind, i in _registers(line.split(None, 1)[1].split(",")[0]) if " " in line else ():
                    held.pop(f"{kind}{i}", None)
            if m:
                held[m.group(1)] = (m.group(2), 0)

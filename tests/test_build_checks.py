"""Checks on the generated gfx950 code that no GPU is needed for."""
import functools
import re

import pytest

from paper_2505_21036_amd import build

device_assembly = functools.lru_cache(maxsize=None)(build.device_assembly)


@pytest.mark.parametrize("source", ["rf_attn.hip", "rf_arm.hip"])
def test_m0_is_used_only_by_the_tile_loads(source):
    """The attention and ARM kernels issue its global->LDS tile loads from inline assembly, which writes
    the LDS address to M0 behind the compiler's back.  That is only sound while the compiler
    itself has no use for M0 in those files: every mention of M0 in the generated code must be
    the assembly's own  s_mov_b32 m0 / s_nop / global_load_lds  triple, and there must be no
    compiler-generated LDS load (which would set M0 itself) left."""
    m0_write = r"s_mov_b32 m0, (s\d+|vcc_lo|vcc_hi)"  # the assembly's own write: any scalar source register
    lines = [l.strip() for l in device_assembly(source).splitlines()]
    code = [l for l in lines if l and not l.startswith((";", ".", "//"))]
    loads = 0
    for i, l in enumerate(code):
        if "global_load_lds" in l:
            assert re.fullmatch(r"global_load_lds_dwordx4 v\[\d+:\d+\], off", l), l
            assert code[i - 1] == "s_nop 0" and re.fullmatch(m0_write, code[i - 2]), code[i - 2:i + 1]
            loads += 1
        elif re.search(r"\bm0\b", l):
            assert re.fullmatch(m0_write, l) and code[i + 1] == "s_nop 0" and "global_load_lds" in code[i + 2], l
    assert loads > 0
    # every explicit wait of the pipeline is still there: one vmcnt wait per tile-loop barrier at least
    assert sum("s_waitcnt vmcnt(0)" in l for l in code) >= (4 if source == "rf_attn.hip" else 2)


def _tile_loops(asm, kernel, mfmas=32):
    """Instruction lists of the innermost loops of `kernel` that hold one tile's MFMAs."""
    lines = asm.splitlines()
    start = next(i for i, l in enumerate(lines) if l.startswith(kernel + ":"))
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    lines = lines[start:end]
    label_at = {m.group(1): i for i, l in enumerate(lines) for m in [re.match(r"^(\.LBB\d+_\d+):", l)] if m}
    loops = []
    for i, l in enumerate(lines):
        m = re.search(r"s_c?branch\w*\s+(\.LBB\d+_\d+)", l)
        if m and label_at.get(m.group(1), len(lines)) < i:
            body = [x.strip() for x in lines[label_at[m.group(1)]:i + 1]]
            body = [x for x in body if x and not x.startswith((";", "."))]
            if sum(x.startswith("v_mfma") for x in body) == mfmas:
                loops.append(body)
    return loops


def test_tile_loops_keep_operand_reads_ahead_of_the_mfmas():
    """Performance guard on the generated code of the eight-wavefront kernel (head_dim 128, 256-row blocks):
    in every tile loop the LDS operand reads run ahead of the MFMAs that use them, which shows as
    waits for all-but-3 / all-but-4 outstanding LDS operations.  (A schedule that reads, waits for
    everything and then issues one MFMA costs ~9 % and has appeared from unrelated edits.)"""
    asm = device_assembly("rf_attn.hip")
    loops = _tile_loops(asm, "_ZN2rf11attn_kernelILi128ELi8ELi0EEEvNS_8AttnArgsE")
    assert len(loops) >= 3  # every-tile walk (dense / packed), compacted walk, listed walk
    for body in loops:
        waits = [x for x in body if x.startswith("s_waitcnt") and "lgkmcnt" in x]
        ahead = sum("lgkmcnt(3)" in x or "lgkmcnt(4)" in x for x in waits)
        assert ahead >= 24, (ahead, len(waits))
        assert not any(x.startswith("scratch_") for x in body)  # no spills inside a tile loop


def test_twelve_wavefront_kernel_fits_its_registers():
    """The kernel of the headline configuration (head_dim 128, 384-row blocks, twelve wavefronts) is
    held to 168 registers so that three wavefronts share a SIMD.  A reload from scratch waits for every
    vector-memory operation in flight, the tile loads included, so the loops that run on every tile
    must hold none; the listed loop may reload lane offsets on its rare path (tiles that are not 64
    consecutive rows), at most two."""
    asm = device_assembly("rf_attn.hip")
    loops = _tile_loops(asm, "_ZN2rf11attn_kernelILi128ELi12ELi0EEEvNS_8AttnArgsE")
    assert len(loops) >= 4
    spills = sorted(sum(x.startswith("scratch_") for x in body) for body in loops)
    assert spills[:-1] == [0] * (len(loops) - 1) and spills[-1] <= 2, spills
    m = re.search(r"\.amdhsa_kernel _ZN2rf11attn_kernelILi128ELi12ELi0EEEvNS_8AttnArgsE.*?\.amdhsa_next_free_vgpr\s+(\d+)", asm, re.S)
    assert m and int(m.group(1)) <= 168


@pytest.mark.parametrize("D,waves", [(64, 3), (96, 2), (128, 2)])
def test_whether_a_tile_is_its_rows_is_asked_once(D, waves):
    """Performance guard: a tile's scores and its softmax are one block.  As two, each behind the same question, every step of
    every kernel took two more branches and the scores' registers were copied (1 % with the keys split two ways, 2 % with 128 rows
    and from queues).  Looked at in the walk of a compacted sequence, the plainest that asks."""
    loops = _tile_loops(device_assembly("rf_attn.hip"), "_ZN2rf16attn_item_kernelILi%dELi2ELi2ELi0ELi%dEEEvNS_8AttnArgsE" % (D, waves), D // 4)
    gathered = [b for b in loops if any(x.startswith("ds_read") and "tr" not in x and "b128" not in x for x in b)]
    plainest = min(gathered, key=len)
    assert sum("s_cbranch" in x for x in plainest) <= 16  # 18 as two blocks


@pytest.mark.parametrize("D", [64, 96, 128])
def test_gathered_rows_are_asked_for_without_waiting_for_the_tile_before(D):
    """Performance guard: wavefronts with tiles of their own ask for the next K as soon as the scores are formed.  A row number
    put in LDS between the scores' MFMAs and those loads would wait for every load, of which V is on its way; and the row
    numbers are read for K alone, once per load."""
    loops = _tile_loops(device_assembly("rf_attn.hip"), "_ZN2rf16attn_item_kernelILi%dELi1ELi4ELi0ELi2EEEvNS_8AttnArgsE" % D, D // 4)
    reads = [[x for x in b if re.match(r"ds_read\w*_b(32|64) ", x) and "tr" not in x] for b in loops]
    assert any(reads)
    for body, rows in zip(loops, reads):
        if not rows:
            continue
        events = "".join("M" if x.startswith("v_mfma") else "L" if "global_load_lds" in x else "w" if x.startswith("ds_write_b32") else "" for x in body)
        assert "Mw" not in events, events
        assert sum(2 if "read2" in x else 1 for x in rows) == D // 8, rows  # loads per tensor


def test_no_tile_loop_reloads_from_scratch():
    """The same for every kernel instance of both files: the tile loops of the attention (D / 4 MFMAs per tile and 32
    query rows) and of the ARM (D / 8) hold no access to scratch.  The pipelined loop for 64-row wavefronts, which runs
    only under its flag, is left out."""
    for source, kinds in (("rf_attn.hip", ("attn_item_kernel", "attn_kernel")), ("rf_arm.hip", ("arm_recall_kernel",))):
        asm = device_assembly(source)
        seen = 0
        for name in re.findall(r"\.amdhsa_kernel (\S+)", asm):
            m = re.search(r"(%s)ILi(\d+)E((?:L[ib]\d+E)+)" % "|".join(kinds), name)
            if not m:
                continue
            D, args = int(m.group(2)), [int(x) for x in re.findall(r"L[ib](\d+)E", m.group(3))]
            if m.group(1) == "attn_kernel" and args[1] == 1:  # RF_FLAG_WIDE_ROWS
                continue
            halves = 2 if m.group(1) == "attn_kernel" and args[1] == 2 else 1
            loops = _tile_loops(asm, name, D // 8 if source == "rf_arm.hip" else D // 4 * halves)
            assert loops, name
            for body in loops:
                assert not any(x.startswith("scratch_") for x in body), name
            seen += 1
        assert seen >= 9, (source, seen)


def test_raised_priority_ends_with_the_tile_loop():
    """Where P V is worked at raised priority the wavefront leaves its tile loop with it: what follows (the rows' store, the
    next item) must begin with the default priority again, before anything is stored."""
    asm = device_assembly("rf_attn.hip").splitlines()
    seen = 0
    for i, l in enumerate(asm):
        m = re.match(r"_ZN2rf\d+(attn_kernel|attn_item_kernel)I\S*:", l)
        if not m:
            continue
        end = next(j for j in range(i, len(asm)) if asm[j].startswith(".Lfunc_end"))
        raised = False
        for x in (y.strip() for y in asm[i:end]):
            if x.startswith("s_setprio"):
                raised = x.split()[1] != "0"
            if x.startswith("global_store_dwordx2"):
                assert not raised, l
                seen += 1
    assert seen > 0

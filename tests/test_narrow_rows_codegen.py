"""Generated gfx950 code of the products of few rows (no GPU needed: hipcc cross-compiles): no spill code, loops without a wait for all
loads, the wait states of loads into LDS, and the order of the reads that a barrier counts on."""
import re

import pytest

from test_kernel_codegen import _Code, _blocks, _device_asm, _functions, _meta, _scalars


@pytest.fixture(scope="module")
def asm():
    return _device_asm("gemm_narrow.hip")


def _kernel(asm):
    (name, body), = _functions(asm, "_ZN4alch18k_gemm_narrow_rows")
    return name, body


def _first_reads(body, landed):
    """From the wait for the first stages of a tile (so many loads may be on their way behind them) to the first matrix instruction."""
    at = [m.start() for m in re.finditer(r"s_waitcnt vmcnt\(%d\)\n" % landed, body)]
    assert len(at) == 1, at
    return body[at[0]:body.index("v_mfma_", at[0])]


def test_first_stage_is_read_before_the_second(asm):
    """64x64 tiles: the first step waits until twelve reads are left and loads into stage 0 behind the barrier, so the twelve
    of stage 0 have to be issued ahead of the twelve of stage 1 (stages of 16 KB; the stage is in the offset)."""
    reads = [int(m.group(1) or 0) for m in re.finditer(r"ds_read_b\S+ v\[[^\]]*\], v\d+(?: offset:(\d+))?\n", _first_reads(_kernel(asm)[1], 28))]
    assert len(reads) == 24 and all(o < 32768 for o in reads), reads
    assert [o // 16384 for o in reads] == [0] * 12 + [1] * 12, reads


def test_first_fragments_wait_for_two_stages_only(asm):
    for landed in (28, 8):  # loads of the other stages, 64x64 and 128x128 tiles
        first = _first_reads(_kernel(asm)[1], landed)
        assert "ds_read_b" in first and not re.search(r"vmcnt\((?!%d\)|24\))\d+\)" % landed, first), first


def test_narrow_rows(asm):
    name, body = _kernel(asm)
    assert _meta(asm, name, "vgpr_spill_count") == 0 and _meta(asm, name, "private_segment_fixed_size") == 0
    assert _meta(asm, name, "group_segment_fixed_size") <= 160 * 1024
    loops = [txt for _, txt in _blocks(body) if txt.count("v_mfma_") >= 4 and "s_barrier" in txt]
    assert loops and not any("scratch_" in txt or "vmcnt(0)" in txt for txt in loops)
    code = _Code(body)
    loads = code.loads_into_lds()
    assert loads
    for i in loads:
        assert not code.within(i, 1, lambda op, rest: op.startswith("s_") and rest.split(",")[0] == "m0"), code.ins[i]
        src = _scalars(code.ins[i][1].partition(",")[2])
        assert not code.within(i, 5, lambda op, rest: op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")) and
                               _scalars(rest.split(",")[0]) & src), code.ins[i]

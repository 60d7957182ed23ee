"""Generated gfx950 code of the products of few rows (no GPU needed: hipcc cross-compiles): no spill code, loops without a wait for all
loads, and the wait states of loads into LDS."""
from test_kernel_codegen import _Code, _blocks, _device_asm, _functions, _meta, _scalars


def test_narrow_rows():
    asm = _device_asm("gemm_narrow.hip")
    (name, body), = _functions(asm, "_ZN4alch18k_gemm_narrow_rows")
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

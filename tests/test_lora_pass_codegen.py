"""Generated gfx950 code of the adapter kernels that stream an activation once: no spilled register (the reload of an address
waits for every load before it: the pass over [dG | dU] and Act took 225 us for 113) and the wait state of loads into LDS."""
import pytest

from test_kernel_codegen import B, _Code, _device_asm, _functions, _meta, _scalars


@pytest.fixture(scope="module")
def text():
    import os
    import shutil
    if not (shutil.which(B._hipcc()) or os.path.exists(B._hipcc())):
        pytest.skip("hipcc not found")
    return _device_asm("lora_pass.hip")


@pytest.mark.parametrize("prefix,count", [("_ZN4alch14k_lora_up_mfma", 1), ("_ZN4alch11k_lora_both", 2)])
def test_kernels_that_stream_an_activation(text, prefix, count):
    seen = 0
    for name, body in _functions(text, prefix):
        assert _meta(text, name, "vgpr_spill_count") == 0 and _meta(text, name, "private_segment_fixed_size") == 0, name
        assert _meta(text, name, "vgpr_count") <= 256 and _meta(text, name, "group_segment_fixed_size") <= 80 * 1024, name
        code = _Code(body)
        loads = code.loads_into_lds()
        assert len(loads) >= 16, name
        for i in loads:
            assert not code.within(i, 1, lambda op, rest: op.startswith("s_") and rest.split(",")[0] == "m0"), (name, code.ins[i])
            src = _scalars(code.ins[i][1].partition(",")[2])
            assert not code.within(i, 5, lambda op, rest: op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")) and
                                   _scalars(rest.split(",")[0]) & src), (name, code.ins[i])
        seen += 1
    assert seen == count

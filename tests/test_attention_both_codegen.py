"""Generated gfx950 code of the launch of both attention gradients: no spill code (no GPU needed: hipcc cross-compiles)."""
import pytest

from test_kernel_codegen import _blocks, _device_asm, _functions, _meta


@pytest.mark.parametrize("source", ["attn_mfma.hip", "attn_mfma_d64.hip"])
def test_no_spills(source):
    asm = _device_asm(source)
    names = [n for n, _ in _functions(asm, "_ZN4alch21k_both_gradients_mfma")] + [n for n, _ in _functions(asm, "_ZN4alch11k_row_delta")]
    assert len(names) == 2, names
    for n in names:
        assert _meta(asm, n, "vgpr_spill_count") == 0 and _meta(asm, n, "private_segment_fixed_size") == 0, n
    for name, body in _functions(asm, "_ZN4alch21k_both_gradients_mfma"):
        for lab, txt in _blocks(body):
            if txt.count("v_mfma_") >= 16:
                assert "scratch_" not in txt, (name, lab)

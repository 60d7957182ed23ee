"""RoPE bases of one and below (every pair turns by the position, or faster than the first): legal, and the backward turns the
gradients back by the same angles, in every attention kernel."""
import pytest

import synth_inputs as synth
from helpers import f64
from oracle import layer_backward_reuse
from test_gpu_layer import compare, make_case, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base", [1.0, 0.5])
@pytest.mark.parametrize("shape_name,dtype", [("config1", "f32"), ("odd", "f32"), ("medium64", "bf16"), ("medium", "bf16")])
@pytest.mark.parametrize("lens", [[3, 40, 25], [700, 65]])  # (the second: two launches in fp32, cut key blocks in bf16)
def test_backward(monkeypatch, shape_name, dtype, base, lens):
    monkeypatch.setitem(synth.SHAPES, "base", synth.SHAPES[shape_name][:6] + (base,))
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case("base", dtype, cu, 11, "drawn", dy_std=0.01)
    compare(run_gpu(shp, dtype, cu, W, rec, dY), layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY), dtype)

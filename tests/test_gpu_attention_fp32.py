"""fp32 attention: heads that fill their 32-column blocks and heads that do not, both gradients in one launch (few
work-groups) and in two, ragged, grouped heads, prefixes, against the fp64 oracle."""
import numpy as np
import pytest

import synth_inputs as synth
from helpers import f64
from oracle import layer_backward_reuse
from test_gpu_layer import compare, make_case, run_gpu

pytestmark = pytest.mark.gpu

# hidden, query heads, key/value heads, head size, ffn, rms eps, rope base
SHAPES = {"d32": (64, 4, 2, 32, 96, 1e-5, 10000.0), "d40": (64, 2, 1, 40, 96, 1e-5, 10000.0), "d64": (128, 4, 2, 64, 160, 1e-5, 10000.0),
          "d128": (128, 2, 1, 128, 160, 1e-5, 10000.0), "d160": (96, 1, 1, 160, 128, 1e-5, 10000.0)}


@pytest.mark.parametrize("shape_name", list(SHAPES))
@pytest.mark.parametrize("lens", [[1, 31, 33], [64, 0, 65, 128], [150] * 13])  # (the last: more work-groups than compute units)
def test_gradients(monkeypatch, shape_name, lens):
    monkeypatch.setitem(synth.SHAPES, shape_name, SHAPES[shape_name])
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case(shape_name, "f32", cu, 17, "drawn", dy_std=0.01)
    ref = layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY)
    first, second = [run_gpu(shp, "f32", cu, W, rec, dY) for _ in range(2)]
    compare(first, ref, "f32")
    for k in first:
        assert np.array_equal(first[k], second[k]), k

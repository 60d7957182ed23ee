"""Attention backward of batches with few or unequal key blocks, whose dK/dV sums are cut over the query heads of a
group: groups that divide evenly and not, both head sizes, blocks that are cut beside blocks that are not, prefixes."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import f64
from oracle import layer_backward_reuse
from test_gpu_layer import compare, make_case, run_gpu

pytestmark = pytest.mark.gpu

# hidden, query heads, key/value heads, head size, ffn, rms eps, rope base
SHAPES = {"group of 5": (320, 5, 1, 64, 704, 1e-5, 10000.0), "group of 8": (512, 8, 1, 128, 1024, 1e-5, 500000.0),
          "group of 7": (896, 7, 1, 128, 512, 1e-5, 10000.0)}


@pytest.mark.parametrize("shape_name,lens", [("medium", [129, 500, 64, 0, 257]), ("medium64", [321, 1, 400]),
                                             ("group of 5", [256, 200, 130, 31]), ("group of 8", [128, 63, 449]),
                                             ("group of 7", [127, 385])])
def test_cut_key_blocks(monkeypatch, shape_name, lens):
    if shape_name in SHAPES:
        monkeypatch.setitem(synth.SHAPES, shape_name, SHAPES[shape_name])
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case(shape_name, "bf16", cu, 31, "drawn", dy_std=0.01)
    ref = layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY)
    first = run_gpu(shp, "bf16", cu, W, rec, dY)
    compare(first, ref, "bf16")
    second = run_gpu(shp, "bf16", cu, W, rec, dY)
    for k in first:
        assert np.array_equal(first[k], second[k]), k  # the parts are added in a fixed order

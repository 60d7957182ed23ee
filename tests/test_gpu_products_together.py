"""A data gradient and the weight gradient that runs beside it in one launch (dH2 with dWd, dO with [dWg; dWu], dH1 with
dWo): tokens below, at and beyond a tile, tiles cut along the contraction beside whole ones, tiles that do not fill a
work-group, accumulation."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import to_dev, f64, alch_shape
from oracle import layer_backward_reuse, WEIGHT_KEYS
from test_gpu_layer import REC, compare, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape_name,dtype,lens", [("medium", "bf16", [1]), ("medium", "bf16", [127, 2]), ("medium", "bf16", [256, 1]),
                                                   ("medium64", "bf16", [600]), ("config1", "f32", [16]), ("config1", "f32", [48, 80]),
                                                   ("config1", "f32", [528])])
def test_products_in_one_launch(shape_name, dtype, lens):
    import paper_2503_01066_amd as A
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case(shape_name, dtype, cu, 21, "drawn", dy_std=0.01)
    ref = layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY)
    dW = {k: to_dev(v, dtype) for k, v in W.items()}
    drec = {k: to_dev(rec[k], dtype) for k in REC}
    drec["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    once = A.alch_layer_backward(alch_shape(shp, dtype), A.Batch(cu), drec, dW, to_dev(dY, dtype), want=WEIGHT_KEYS)
    once = {k: v.clone() for k, v in once.items()}
    torch.cuda.synchronize()
    compare({k: v.double().cpu().numpy() for k, v in once.items()}, ref, dtype)
    grads = {k: v.clone() for k, v in once.items() if k != "dX"}
    twice = A.alch_layer_backward(alch_shape(shp, dtype), A.Batch(cu), drec, dW, to_dev(dY, dtype), grads=grads, accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(twice["dX"], once["dX"])
    for k in grads:
        # once more of the same, one rounding of the sum on top of the one that `once` carries
        want, eps = 2 * once[k].double(), 2.0 ** (-8 if dtype == "bf16" else -23)
        assert bool(((twice[k].double() - want).abs() <= 2 * eps * want.abs() + 1e-30).all()), k

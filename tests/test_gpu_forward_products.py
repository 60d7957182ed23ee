"""Layer forward, whose q/k/v and gate/up products run as one where the widths allow it and whose residual additions
are the products' own: widths that are and are not multiples of a tile, row counts at tile edges, both types."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, alch_shape, f64, oracle_shape, rel_err, to_dev, to_np
from oracle import layer_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape_name,dtype", [("medium", "bf16"), ("medium64", "bf16"), ("tiny", "bf16"), ("config1", "f32")])
@pytest.mark.parametrize("lens", [[1], [100, 28], [255, 2], [300, 0, 212, 257]])
def test_forward_against_the_oracle(shape_name, dtype, lens):
    # medium: q/k/v 1024 + 256 + 256 columns, gate/up 1536 each, all in one product; medium64: q 384, on its own
    import paper_2503_01066_amd as A
    shp = synth.shape_dict(shape_name)
    cu = synth.ragged_cu(lens)
    W = synth.layer_weights(shp, 3, dtype, gain_std=0.1)
    X = synth.activations(int(cu[-1]), shp["hidden"], 4, dtype)
    Y64, rec64 = layer_forward(oracle_shape(shp), cu, None, X.astype(np.float64), f64(W))
    dX = to_dev(X, dtype)
    Y, rec = A.alch_layer_forward(alch_shape(shp, dtype), A.Batch(cu), dX, {k: to_dev(v, dtype) for k, v in W.items()})
    torch.cuda.synchronize()
    assert torch.equal(dX, to_dev(X, dtype))
    assert rel_err(to_np(Y), Y64) <= TOL[dtype]
    for k in ("X2", "Q", "K", "V", "O", "G", "U", "LSE"):
        assert rel_err(to_np(rec[k]), rec64[k]) <= TOL[dtype], k

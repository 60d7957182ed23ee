"""Attention backward of short batches: dQ and dK/dV in one launch, behind one that forms delta.  Sequences beside key blocks of 128 and tiles
of 64, with and without cut key blocks, batches whose work-groups just find and just do not find compute units, against the definition."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, alch_shape, f64, rel_err, to_dev, to_np
from oracle import layer_backward_reuse
from test_gpu_layer import REC, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1], [64], [65, 1], [128], [129], [200, 0, 57], [320], [500], [513], [128] * 6, [128] * 8, [1000]])
@pytest.mark.parametrize("heads", [(32, 8, 128), (32, 8, 64), (4, 4, 128), (32, 1, 64)])
def test_short_batches(monkeypatch, lens, heads):
    import paper_2503_01066_amd as A
    n_q, n_kv, D = heads
    monkeypatch.setitem(synth.SHAPES, "both", (256, n_q, n_kv, D, 256, 1e-5, 10000.0))
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case("both", "bf16", cu, 7, "drawn", dy_std=0.01)
    ref = layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY.astype(np.float64))
    d = {k: to_dev(rec[k], "bf16") for k in REC}
    d["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    batch = A.Batch(cu)
    batch.c.max_seqlen = int(cu[-1]) + 300  # (a bound: any number that is not below the longest)
    out = A.alch_layer_backward(alch_shape(shp, "bf16"), batch, d, {k: to_dev(v, "bf16") for k, v in W.items()}, to_dev(dY, "bf16"))
    torch.cuda.synchronize()
    for k in ("dX", "dWq", "dWk", "dWv"):
        assert rel_err(to_np(out[k]), ref[k]) <= TOL["bf16"], (k, rel_err(to_np(out[k]), ref[k]))


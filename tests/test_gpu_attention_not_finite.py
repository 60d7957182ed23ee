"""A NaN or an infinity in one token reaches the tokens that see it, or that it sees, and no others: not those that merely share
a tile with it.  Keys and values: later tokens; queries and output gradients: earlier tokens; never another sequence's."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, alch_shape, rel_err, to_dev, to_np
from test_gpu_layer import REC, make_case

pytestmark = pytest.mark.gpu

SHAPES = {"d40": (64, 2, 1, 40, 96, 1e-5, 10000.0), "d160": (96, 1, 1, 160, 128, 1e-5, 10000.0), "group of 5": (320, 5, 1, 64, 704, 1e-5, 10000.0)}


@pytest.mark.parametrize("shape_name,dtype", [("config1", "f32"), ("d40", "f32"), ("d160", "f32"), ("d40", "bf16"), ("medium64", "bf16"),
                                              ("group of 5", "bf16")])
@pytest.mark.parametrize("lens,t", [([70, 40], 45), ([65, 700], 65 + 333), ([150] * 13, 151)])
@pytest.mark.parametrize("where", ["K", "V", "Q", "dY"])
def test_reach(monkeypatch, shape_name, dtype, lens, t, where):
    import paper_2503_01066_amd as A
    if shape_name in SHAPES:
        monkeypatch.setitem(synth.SHAPES, shape_name, SHAPES[shape_name])
    cu = synth.ragged_cu(lens)
    shp, _, W, rec, dY = make_case(shape_name, dtype, cu, 23, "drawn", dy_std=0.01)
    dW, batch = {k: to_dev(v, dtype) for k, v in W.items()}, A.Batch(cu)

    def run(bad):
        r, g = {k: to_dev(rec[k], dtype) for k in REC}, to_dev(dY, dtype)
        r["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
        if bad is not None:
            (g if where == "dY" else r[where])[t, 3] = bad
        O, lse = A.alch_attention_forward(alch_shape(shp, dtype), batch, r["Q"], r["K"], r["V"])
        dX = A.alch_layer_backward(alch_shape(shp, dtype), batch, r, dW, g, want=())["dX"]
        torch.cuda.synchronize()
        return to_np(O), to_np(lse), to_np(dX)

    seq = int(np.searchsorted(cu, t, side="right")) - 1
    rows = np.arange(cu[-1])
    later, earlier = (rows > t) & (rows < cu[seq + 1]), (rows < t) & (rows >= cu[seq])
    clean = run(None)
    for bad in (float("nan"), float("inf")):
        O, lse, dX = run(bad)
        fwd_free = (rows != t) if where in "Q" else np.ones_like(later) if where == "dY" else ~later & (rows != t)
        bwd_free = (~later if where in "KV" else ~earlier) & (rows != t)
        for got, want, free in ((O, clean[0], fwd_free), (lse, clean[1], fwd_free), (dX, clean[2], bwd_free)):
            assert np.isfinite(got[free]).all()
            assert rel_err(got[free], want[free]) <= TOL[dtype]
        assert not np.isfinite(dX[t]).any()

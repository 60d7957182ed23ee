"""bf16 layers: the partial rows of both RMSNorm gains added by one launch where those of g1 find room in the activation's buffer.  Batches of
fewer rows than the row kernels may leave and of more, feed-forward widths that just give the room and just do not, hidden sizes either
side of each row kernel."""
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, alch_shape, f64, rel_err, to_dev, to_np
from oracle import layer_backward_reuse
from test_gpu_layer import REC, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 5, 255, 257, 513])
@pytest.mark.parametrize("hidden,ffn", [(256, 512), (256, 504), (260, 520), (2056, 4112), (4104, 8200)])
def test_gains(monkeypatch, hidden, ffn, T):
    import paper_2503_01066_amd as A
    monkeypatch.setitem(synth.SHAPES, "gains", (hidden, 4, 4, 64, ffn, 1e-5, 10000.0))
    cu = synth.ragged_cu([min(200, T - a) for a in range(0, T, 200)])
    shp, osh, W, rec, dY = make_case("gains", "bf16", cu, 11, "drawn", dy_std=0.01)
    ref = layer_backward_reuse(osh, cu, None, f64(rec), f64(W), f64({"dY": dY})["dY"])
    d = {k: to_dev(rec[k], "bf16") for k in REC}
    d["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    out = A.alch_layer_backward(alch_shape(shp, "bf16"), A.Batch(cu), d, {k: to_dev(v, "bf16") for k, v in W.items()}, to_dev(dY, "bf16"))
    torch.cuda.synchronize()
    for k in ("dX", "dg1", "dg2"):
        assert rel_err(to_np(out[k]), ref[k]) <= TOL["bf16"], (k, rel_err(to_np(out[k]), ref[k]))

"""max_seqlen is a bound on the lengths and may be any number above them, up to the largest of its type: the attention kernels
size their launches by the lengths themselves and give the same bits."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import alch_shape, to_dev
from test_gpu_layer import REC, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape_name,dtype", [("config1", "f32"), ("odd", "f32"), ("medium64", "bf16")])
@pytest.mark.parametrize("lens,bound", [([3, 40, 25], 131072), ([200, 0, 130], 2 ** 31 - 1), ([150] * 13, 2 ** 31 - 40)])
def test_loose_bound(shape_name, dtype, lens, bound):
    import paper_2503_01066_amd as A
    cu = synth.ragged_cu(lens)
    shp, _, W, rec, dY = make_case(shape_name, dtype, cu, 19, "drawn", dy_std=0.01)
    dW, drec = {k: to_dev(v, dtype) for k, v in W.items()}, {k: to_dev(rec[k], dtype) for k in REC}
    drec["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    outs = []
    for n in (max(lens), bound):
        batch = A.Batch(cu)
        batch.c.max_seqlen = n
        O, lse = A.alch_attention_forward(alch_shape(shp, dtype), batch, drec["Q"], drec["K"], drec["V"])
        outs.append(dict(A.alch_layer_backward(alch_shape(shp, dtype), batch, drec, dW, to_dev(dY, dtype)), O=O, LSE=lse))
    torch.cuda.synchronize()
    for k in outs[0]:
        assert torch.equal(outs[0][k], outs[1][k]) and bool(torch.isfinite(outs[0][k]).all()), k

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


@pytest.mark.parametrize("shape_name", ["medium", "medium64", "group of 5", "group of 7"])
@pytest.mark.parametrize("prompts,responses", [([300, 65], [[70, 129], [100, 200]]), ([130, 500], [[40, 75, 1], [257]])])
def test_cut_key_blocks_of_shared_prompts(monkeypatch, shape_name, prompts, responses):
    # the keys of a prompt meet its own queries and those of its responses: blocks long enough to be cut, in either head size
    from helpers import alch_shape, rel_err, TOL, to_dev, to_np
    from oracle import WEIGHT_KEYS
    from oracle.prefix import layer_backward_reuse_prefix
    from test_gpu_prefix import dev_record, make
    import paper_2503_01066_amd as A
    if shape_name in SHAPES:
        monkeypatch.setitem(synth.SHAPES, shape_name, SHAPES[shape_name])
    shp, osh, b, W, _, _, _, rec, dY = make("bf16", shape_name, prompts, responses, 9)
    ref = layer_backward_reuse_prefix(osh, b["cu"], b["prefix"], f64(rec), f64(W), dY)
    batch = A.Batch(b["cu"], positions=b["positions"], prefix=b["prefix"])
    outs = [A.alch_layer_backward(alch_shape(shp, "bf16"), batch, dev_record(rec, "bf16"), {k: to_dev(v, "bf16") for k, v in W.items()},
                                  to_dev(dY, "bf16")) for _ in range(2)]
    torch.cuda.synchronize()
    for k in ["dX"] + ["d" + w for w in WEIGHT_KEYS]:
        assert torch.equal(outs[0][k], outs[1][k]), k
        assert rel_err(to_np(outs[0][k]), ref[k]) <= TOL["bf16"], k

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


@pytest.mark.parametrize("D,Hkv,lens", [(64, 4, [128, 128]), (64, 4, [300, 1, 723]), (128, 2, [300, 1, 723]), (256, 2, [1024]), (32, 8, [1, 1023])])
def test_sums_round_no_more_often_than_a_tree(D, Hkv, lens):
    # Scores are sums of D products of order 1 and lose what their order of addition costs.  With the terms paired (log2 D
    # roundings each) O was within 1.6e-7 of its norm at 2 x 128 tokens and 2.5e-7 .. 3.3e-7 at 1024, dQ of the short
    # sequences within 3.6e-7; one sum over the whole head made it 2.0e-7, 2.0e-7 .. 4.4e-7 and 4.3e-7.  The bounds are the
    # paired sums' errors (of 1024 tokens the smallest).
    import torch
    import paper_2503_01066_amd as A
    from helpers import alch_shape, to_dev, to_np
    from test_gpu_attention_d64 import attention_fp64, exposed_case, run_exposed
    cu = synth.ragged_cu(lens)
    T = int(cu[-1])
    shp, W, rec, dY = exposed_case(cu, Hkv, D, 10000.0, np.random.default_rng(7), "f32")
    ref = attention_fp64(shp, cu, rec, dY)
    O, _ = A.alch_attention_forward(alch_shape(shp, "f32"), A.Batch(cu), *[to_dev(rec[k], "f32") for k in "QKV"])
    torch.cuda.synchronize()
    err = np.linalg.norm(to_np(O) - ref["O"]) / np.linalg.norm(ref["O"])
    assert err <= (1.6e-7 if T == 256 else 2.5e-7), err
    if T == 256:
        got = run_exposed(shp, W, rec, ref["LSE"], dY, cu, dtype="f32")
        for k, bound in (("dQ", 3.65e-7), ("dK", 3.2e-7), ("dV", 2.6e-7)):
            err = np.linalg.norm(got[k] - ref[k]) / np.linalg.norm(ref[k])
            assert err <= bound, (k, err)


@pytest.mark.parametrize("shape_name", ["d32", "d40", "d64", "d128"])
@pytest.mark.parametrize("prompts,responses", [([33, 64], [[20, 31], [1, 40]]), ([130, 97], [[60, 75], [200, 33, 1]])])  # (one launch; two)
def test_shared_prompts(monkeypatch, shape_name, prompts, responses):
    import torch
    import paper_2503_01066_amd as A
    from helpers import TOL, alch_shape, rel_err, to_dev, to_np
    from oracle import WEIGHT_KEYS
    from oracle.prefix import layer_backward_reuse_prefix
    from test_gpu_prefix import dev_record, make
    monkeypatch.setitem(synth.SHAPES, shape_name, SHAPES[shape_name])
    shp, osh, b, W, _, _, _, rec, dY = make("f32", shape_name, prompts, responses, 9)
    ref = layer_backward_reuse_prefix(osh, b["cu"], b["prefix"], f64(rec), f64(W), dY)
    batch = A.Batch(b["cu"], positions=b["positions"], prefix=b["prefix"])
    out = A.alch_layer_backward(alch_shape(shp, "f32"), batch, dev_record(rec, "f32"), {k: to_dev(v, "f32") for k, v in W.items()}, to_dev(dY, "f32"))
    O, lse = A.alch_attention_forward(alch_shape(shp, "f32"), batch, *[to_dev(rec[k], "f32") for k in "QKV"])
    torch.cuda.synchronize()
    for k in ["dX"] + ["d" + w for w in WEIGHT_KEYS]:
        assert rel_err(to_np(out[k]), ref[k]) <= TOL["f32"], k
    assert rel_err(to_np(O), rec["O"]) <= 1e-5 and rel_err(to_np(lse), rec["LSE"]) <= 1e-5

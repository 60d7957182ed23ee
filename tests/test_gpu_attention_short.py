"""Batches of many sequences of a few tokens, whose attention is formed a row at a time: lengths around the limits of the rows
(8, 16 and 24 tokens by head size), empty sequences and long ones among them, given positions, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, alch_shape, f64, rel_err, to_dev, to_np
from oracle import attention_lse, layer_backward_reuse
from test_gpu_attention_d64 import attention_fp64
from test_gpu_layer import compare, make_case, run_gpu

pytestmark = pytest.mark.gpu

# hidden, query heads, key/value heads, head size, ffn, rms eps, rope base
SHAPES = {"d64": (64, 6, 2, 64, 96, 1e-5, 10000.0), "d20": (64, 4, 2, 20, 96, 1e-5, 10000.0), "d80": (64, 5, 1, 80, 96, 1e-5, 10000.0),
          "d160": (64, 2, 2, 160, 96, 1e-5, 10000.0)}


@pytest.mark.parametrize("shape_name,dtype", [("d64", "bf16"), ("d64", "f32"), ("d20", "f32"), ("d80", "bf16"), ("d80", "f32"), ("d160", "bf16")])
@pytest.mark.parametrize("lens,turned", [([1] * 800, False), ([1, 2, 0, 7, 8, 9, 3, 5] * 100 + [70, 33], True),
                                         ([15, 16, 17, 1, 23, 24, 25, 4] * 90, False)])
def test_short_sequences(monkeypatch, shape_name, dtype, lens, turned):
    import paper_2503_01066_amd as A
    monkeypatch.setitem(synth.SHAPES, shape_name, SHAPES[shape_name])
    cu = synth.ragged_cu(lens)
    T = int(cu[-1])
    shp, osh, W, rec, dY = make_case(shape_name, dtype, cu, 29, "drawn", dy_std=0.01)
    positions = np.random.default_rng(2).integers(0, 3000, T).astype(np.int32) if turned else None
    ref = layer_backward_reuse(osh, cu, positions, f64(rec), f64(W), dY)
    compare(run_gpu(shp, dtype, cu, W, rec, dY, positions=positions), ref, dtype)
    O, lse = A.alch_attention_forward(alch_shape(shp, dtype), A.Batch(cu), *[to_dev(rec[k], dtype) for k in "QKV"])
    want = attention_fp64(shp, cu, rec, np.zeros_like(rec["O"]))
    assert rel_err(to_np(O), want["O"]) <= (TOL["bf16"] if dtype == "bf16" else 1e-5) and rel_err(to_np(lse), want["LSE"]) <= 1e-5


# Heads of 64 in large groups: the row kernels take the short sequences, and the key blocks of the long one are cut into parts.
# (query heads to one key/value head, lengths, whose long sequence is first, last or between the short ones)
CUT = [(64, [1000] + [4] * 64), (32, [4] * 128 + [1000]), (64, [3, 8] * 20 + [900] + [1, 0, 5] * 16)]


@pytest.mark.parametrize("heads,lens", CUT)
def test_short_sequences_beside_cut_key_blocks(monkeypatch, heads, lens):
    monkeypatch.setitem(synth.SHAPES, "cut", (64, heads, 1, 64, 1024, 1e-5, 10000.0))
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case("cut", "bf16", cu, 31, "drawn", dy_std=0.01)
    ref = layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY)
    compare(run_gpu(shp, "bf16", cu, W, rec, dY), ref, "bf16")

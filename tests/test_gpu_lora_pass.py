"""Adapter products that share one pass over an activation: rows that do not fill a step of 32 or a block of 128, widths that do not
fill 128 or 512 columns, more than four groups of eight rank columns, gradients that are not asked for, and shapes and batches that take
two passes."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, f64, rel_err, to_dev
from oracle.lora import layer_backward_reuse_lora
from test_gpu_lora import compare, make_case, run_gpu

pytestmark = pytest.mark.gpu


def case(monkeypatch, T, rank, hidden, ffn, projections=synth.PROJECTIONS):
    monkeypatch.setitem(synth.SHAPES, "pass", (hidden, 4, 2, 64, ffn, 1e-5, 10000.0))
    cu = synth.ragged_cu([min(61, T - a) for a in range(0, T, 61)])
    shp, osh, W, lora, lora64, rec, dY, scale = make_case("pass", "bf16", cu, 17, rank, projections, record="drawn", dy_std=0.01)
    return cu, shp, W, lora, rec, dY, scale, layer_backward_reuse_lora(osh, cu, None, f64(rec), f64(W), lora64, scale, dY)


@pytest.mark.parametrize("T,rank,hidden,ffn", [(1, 8, 256, 512), (33, 24, 320, 576), (95, 40, 256, 1088), (161, 64, 320, 576),
                                               (1030, 8, 512, 1536), (5500, 8, 256, 704),  # blocks of 256 rows
                                               (5500, 8, 64, 192),    # more partial sums than scratch: two passes
                                               (130, 8, 264, 520)])   # widths that the matrix cores do not take: two passes
def test_rows_widths_and_ranks(monkeypatch, T, rank, hidden, ffn):
    cu, shp, W, lora, rec, dY, scale, ref = case(monkeypatch, T, rank, hidden, ffn)
    gpu = run_gpu(shp, "bf16", cu, W, lora, rank, scale, rec, dY)
    assert len(gpu) == 15
    compare(gpu, ref, "bf16")


@pytest.mark.parametrize("wanted", ["A", "B", "gdBdA", ""])
@pytest.mark.parametrize("projections", [synth.PROJECTIONS, ("d", "u", "k"), ("g", "o")])
def test_gradients_that_are_not_asked_for(monkeypatch, wanted, projections):
    import paper_2503_01066_amd as A
    cu, shp, W, lora, rec, dY, scale, ref = case(monkeypatch, 130, 16, 256, 576, projections)
    take = {"A": lambda p, m: m == "A", "B": lambda p, m: m == "B", "": lambda p, m: False,
            "gdBdA": lambda p, m: (p, m) in (("g", "B"), ("d", "A"))}[wanted]
    bufs = {"d" + m + p: torch.zeros(lora[p][m == "B"].shape, dtype=torch.bfloat16, device="cuda") for p in projections for m in "AB" if take(p, m)}
    gpu = run_gpu(shp, "bf16", cu, W, lora, 16, scale, rec, dY, lora_grads=bufs)
    assert sorted(gpu) == sorted(list(bufs) + ["dX"])
    compare(gpu, ref, "bf16")


# Tokens in one pass and tokens for whose partial sums the scratch has no room, the parts of t2 16, 8 and 4
BITS_SHAPE = (64, 2, 2, 64, 320, 1e-5, 10000.0)
BITS = [(8, 880, 1000), (8, 1480, 1600), (8, 2480, 2600)]


@pytest.mark.parametrize("rank,in_one,apart", BITS)
def test_data_gradient_keeps_its_bits_in_one_pass(monkeypatch, rank, in_one, apart):
    """The tokens of a batch that takes one pass, alone and at the front of one that takes two: t2, and so dX, is the same sum (no
    product of this shape is long enough to be cut, and no sequence depends on another)."""
    import paper_2503_01066_amd as A
    monkeypatch.setitem(synth.SHAPES, "pass", BITS_SHAPE)
    cu = synth.uniform_cu(apart // 40, 40)
    shp, osh, W, lora, lora64, rec, dY, scale = make_case("pass", "bf16", cu, 31, rank, synth.PROJECTIONS, record="drawn", dy_std=0.01)
    both = run_gpu(shp, "bf16", cu, W, lora, rank, scale, rec, dY)["dX"]
    front = run_gpu(shp, "bf16", synth.uniform_cu(in_one // 40, 40), W, lora, rank, scale, {k: v[:in_one] for k, v in rec.items()}, dY[:in_one])["dX"]
    assert np.array_equal(front, both[:in_one])

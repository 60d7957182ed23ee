"""Layers with adapters under a loss mask: where Act, dG and dU take one pass, everything from the MLP to the output projection runs on
the kept rows, whose number only the device knows.  Counts beside steps of 32 and blocks of 128 and 256 rows, none, one and all,
against the dense call on a dY whose masked rows are zero (which the tests of adapters hold against the definition)."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import alch_shape, to_dev
from oracle import WEIGHT_KEYS
from test_gpu_lora import REC, make_case

pytestmark = pytest.mark.gpu


CASES = [(1000, 8, 2048, 8192, True, False), (4000, 24, 1088, 3904, False, True), (5500, 8, 1024, 2816, True, True),  # blocks of 256 rows
         (700, 8, 512, 1024, False, False)]
ALL_ROWS = [700]  # too few to gain


@pytest.mark.parametrize("T,rank,hidden,ffn,frozen,accumulate", CASES)
def test_kept_counts(monkeypatch, T, rank, hidden, ffn, frozen, accumulate):
    import paper_2503_01066_amd as A
    monkeypatch.setitem(synth.SHAPES, "kept", (hidden, 4, 2, 64, ffn, 1e-5, 10000.0))
    cu = synth.ragged_cu([min(61, T - a) for a in range(0, T, 61)])
    shp, _, W, lora, _, rec, dY, scale = make_case("kept", "bf16", cu, 19, rank, synth.PROJECTIONS, record="drawn", dy_std=0.01)
    d = {k: to_dev(rec[k], "bf16") for k in REC}
    d["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    Wd, dYd = {k: to_dev(v, "bf16") for k, v in W.items()}, to_dev(dY, "bf16")
    dl = {p: (to_dev(a, "bf16"), to_dev(b, "bf16")) for p, (a, b) in lora.items()}
    old = 0.001 if accumulate else float("nan")  # (not accumulated: every element is written)
    start = lambda: {} if frozen else {"d" + k: torch.full_like(Wd[k], old) for k in WEIGHT_KEYS}
    start_lora = lambda: {"d" + m + p: torch.full_like(ab[m == "B"], old) for p, ab in dl.items() for m in "AB"}
    order = np.random.default_rng(7).permutation(T)
    for kept in (0, 1, 31, 33, 127, 128, 129, 255, 257, T - 1, T):
        mask = np.zeros(T, np.uint8)
        mask[order[:kept]] = 1
        m = torch.from_numpy(mask).cuda()
        run = lambda dy, lm: A.alch_layer_backward_lora(alch_shape(shp, "bf16"), A.Batch(cu), d, Wd, dl, rank, scale, dy, loss_mask=lm,
                                                        grads=start(), lora_grads=start_lora(), accumulate=accumulate)
        got, want = run(dYd, m), run(dYd * m[:, None].to(dYd.dtype), None)
        torch.cuda.synchronize()
        assert sorted(got) == sorted(want)
        for k in want:
            a, b = got[k].float(), want[k].float()
            assert torch.isfinite(a).all(), (kept, k)
            # the two differ in the order of fp32 sums, and so in where a bf16 rounding falls: at most four roundings, one
            # behind the other (dG/dU, dH2, dX2, the output), each 2^-9 of the norm
            assert float((a - b).norm()) <= 2 ** -7 * float(b.norm()), (kept, k, float((a - b).norm() / b.norm()))


def test_rows_too_wide_for_device_counts_run_as_before(monkeypatch):
    """[dG | dU] rows of more than 2^21 elements: no kernel takes such a product with its row count on the device."""
    import paper_2503_01066_amd as A
    T, H, F, rank, g = 256, 64, (1 << 20) + 64, 8, torch.Generator(device="cuda").manual_seed(5)
    shape = A.make_shape(H, 1, 1, 64, F, 1e-5, 10000.0, "bf16")
    draw = lambda *s, std=1.0: torch.randn(s, generator=g, device="cuda").mul_(std).to(torch.bfloat16)
    d = {k: draw(T, F if k in "GU" else H) for k in REC}
    d["LSE"] = torch.full((T, 1), 5.0, device="cuda")
    W = {"W" + k: draw(F if k in "gu" else H, F if k == "d" else H, std=0.02) for k in "qkvogud"}
    W["g1"], W["g2"] = draw(H), draw(H)
    lora = {p: (draw(rank, W["W" + p].shape[1], std=0.05), draw(W["W" + p].shape[0], rank, std=0.05)) for p in synth.PROJECTIONS}
    dY = draw(T, H, std=0.01)
    mask = (torch.rand(T, generator=g, device="cuda") < 0.3).to(torch.uint8)
    run = lambda dy, m: A.alch_layer_backward_lora(shape, A.Batch(np.array([0, 100, T])), d, W, lora, rank, 2.0, dy, loss_mask=m, grads={})
    got, want = run(dY, mask), run(dY * mask[:, None].to(dY.dtype), None)
    torch.cuda.synchronize()
    for k in want:
        assert torch.equal(got[k], want[k]), k

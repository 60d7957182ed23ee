"""Products sized by the number of rows that a loss mask keeps: which kernel takes them, and whether their tiles are cut along
the contraction, is settled on the device.  Kept counts at edges of the 128- and 256-row tiles, none, one and all, in a batch where
the counts reach whole and cut tiles of the 128x256 kernel and whole ones of the 256x256 kernel (which cuts none of these), against
the dense call on a dY whose masked rows are zero.  Weight gradients that contract the kept rows choose for half of the tokens: short
ones run on the 128x256 kernel, those of the long batch on the other."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import alch_shape, to_dev
from oracle import WEIGHT_KEYS
from test_gpu_layer import REC, make_case

pytestmark = pytest.mark.gpu
COUNTS = (0, 1, 128, 129, 257, 700, 1025, 1281, 2049, 2305, 4159, 4160)
LONG, LONG_T = (4096, 4, 2, 64, 2048, 1e-5, 10000.0), 7040


@pytest.mark.parametrize("accumulate", [False, True])
def test_kept_counts(monkeypatch, accumulate):
    monkeypatch.setitem(synth.SHAPES, "kept", (2048, 16, 4, 128, 8192, 1e-5, 10000.0))
    compare_kept_counts(synth.uniform_cu(65, 64), COUNTS, accumulate)


@pytest.mark.parametrize("accumulate", [False, True])
def test_kept_counts_of_a_long_batch(monkeypatch, accumulate):
    # [dWg; dWu] of 4096 x 4096: counts beside a k-tile, odd numbers of them, ragged ends, other remainders by the ten of the rings
    monkeypatch.setitem(synth.SHAPES, "kept", LONG)
    compare_kept_counts(synth.uniform_cu(LONG_T // 64, 64), (0, 1, 31, 32, 33, 159, 161, 3525, 7039, 7040), accumulate)


def compare_kept_counts(cu, counts, accumulate):
    import paper_2503_01066_amd as A
    T = int(cu[-1])
    shp, _, W, rec, dY = make_case("kept", "bf16", cu, 29, "drawn", dy_std=0.01)
    d = {k: to_dev(rec[k], "bf16") for k in REC}
    d["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    Wd, dYd, old = {k: to_dev(v, "bf16") for k, v in W.items()}, to_dev(dY, "bf16"), 0.001
    start = lambda: {"d" + k: torch.full_like(Wd[k], old) for k in WEIGHT_KEYS}
    order = np.random.default_rng(7).permutation(T)
    for kept in counts:
        mask = np.zeros(T, np.uint8)
        mask[order[:kept]] = 1
        m = torch.from_numpy(mask).cuda()
        run = lambda dy, lm: A.alch_layer_backward(alch_shape(shp, "bf16"), A.Batch(cu), d, Wd, dy, loss_mask=lm, grads=start(),
                                                   accumulate=accumulate)
        got, want = run(dYd, m), run(dYd * m[:, None].to(dYd.dtype), None)
        torch.cuda.synchronize()
        for k in want:
            a, b = got[k].float(), want[k].float()
            assert torch.isfinite(a).all(), (kept, k)
            # the two differ in the order of fp32 sums, and so in where a bf16 rounding falls: at most four roundings, one
            # behind the other (dG/dU, dH2, dX2, the output), each 2^-9 of the norm
            assert float((a - b).norm()) <= 2 ** -7 * float(b.norm()), (kept, k, float((a - b).norm() / b.norm()))


def test_products_of_kept_rows_are_traced_without_work(monkeypatch):
    """A record of the launch trace counts the operations of products whose sizes the host knows: with a mask those behind the
    attention, dH1 and d[Wq; Wk; Wv], and not dWo, which contracts the kept rows, where it shares the launch of dH1."""
    import paper_2503_01066_amd as A
    H, QKV = 2048, 3072
    monkeypatch.setitem(synth.SHAPES, "kept", (H, 16, 4, 128, 8192, 1e-5, 10000.0))
    cu = synth.uniform_cu(65, 64)
    T = int(cu[-1])
    shp, _, W, rec, dY = make_case("kept", "bf16", cu, 29, "drawn", dy_std=0.01)
    d = {k: to_dev(rec[k], "bf16") for k in REC}
    d["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    mask = torch.from_numpy(synth.keep_mask(T, 0.25, 3)).cuda()
    A.alch_trace_enable(True)
    A.alch_layer_backward(alch_shape(shp, "bf16"), A.Batch(cu), d, {k: to_dev(v, "bf16") for k, v in W.items()}, to_dev(dY, "bf16"),
                          loss_mask=mask, want=WEIGHT_KEYS)
    torch.cuda.synchronize()
    A.alch_trace_enable(False)
    work = [(flops, nbytes) for kind, flops, nbytes, ms in A.alch_trace_collect() if kind == "gemm_mfma"]
    known = (2.0 * T * H * QKV, 2.0 * (T * QKV + QKV * H + T * H))  # of either: the three matrices are the same sizes
    assert sorted(w for w in work if w != (0.0, 0.0)) == [known, known], work
    assert len(work) == 7, work  # dAct, dWd, dH2, [dWg; dWu], dO without work; dH1 with dWo, d[Wq; Wk; Wv]

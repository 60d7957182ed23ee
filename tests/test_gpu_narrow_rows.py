"""Stacks of several layers under a loss mask: the data gradients of the head and of the top layer, sized by the kept rows, run whole in
tiles of 64x64 or 128x128 where no compute unit has a second one.  Kept counts beside both tiles, columns that are no whole large tile,
with and without the SwiGLU gradient behind the product, against the definition in 64 bits."""
import numpy as np
import pytest

import synth_inputs as synth
from helpers import f64
from oracle import stack_backward_reuse
from test_gpu_stack import check_stack, make_stack, run_stack

pytestmark = pytest.mark.gpu


# 64x64 tiles throughout; of dAct 130 x 8256 387 of them, 130 of 128x128; of dHf and dH2 1100 x 1088 306 and 81
@pytest.mark.parametrize("hidden,ffn,V,T,kept,wstd", [(320, 640, 4160, 300, k, 0.05) for k in (1, 63, 64, 65, 129, 250)] +
                         [(320, 8256, 512, 200, k, 0.05) for k in (128, 130)] + [(1088, 512, 320, 1300, k, 0.03) for k in (1024, 1025, 1100)])
def test_kept_counts(monkeypatch, hidden, ffn, V, T, kept, wstd):
    monkeypatch.setitem(synth.SHAPES, "narrow", (hidden, 4, 2, 64, ffn, 1e-5, 10000.0))
    cu = synth.ragged_cu([T // 3, 1, T - T // 3 - 1])
    shp, osh, Ws, recs, Xf, gf, Wlm, labels = make_stack("narrow", "bf16", cu, 2, V, 17, wstd)
    mask = np.zeros(T, np.uint8)
    mask[np.random.default_rng(kept).permutation(np.flatnonzero(labels >= 0))[:kept]] = 1
    ref = stack_backward_reuse(osh, cu, None, [f64(r) for r in recs], [f64(W) for W in Ws], Xf.astype(np.float64), gf.astype(np.float64),
                               Wlm.astype(np.float64), labels, mask)
    check_stack(run_stack(shp, "bf16", cu, Ws, recs, Xf, gf, Wlm, labels, mask), ref, "bf16", 2)

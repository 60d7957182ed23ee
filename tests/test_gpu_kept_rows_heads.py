"""Head of a stack under a loss mask: its products are sized by the kept rows, which the device counts, and those of few rows are
cut along the contraction (the vocabulary in dHf).  Kept counts beside tiles of 128 rows, none, one and all, against the definition in 64 bits."""
import numpy as np
import pytest

import synth_inputs as synth
from test_gpu_stack import _check_head, _head_case

pytestmark = pytest.mark.gpu


KEPT = [1, 127, 128, 129, 300, 698]
SIZES = [(256, 20032), (1088, 4160)]


@pytest.mark.parametrize("kept", KEPT)
@pytest.mark.parametrize("hidden,V", SIZES)
def test_kept_counts(monkeypatch, hidden, V, kept):
    monkeypatch.setitem(synth.SHAPES, "head", (hidden, 4, 2, 64, 512, 1e-5, 10000.0))
    shp, cu, Xf, gf, Wlm, labels = _head_case("head", V, [300, 1, 400], 41, wstd=0.05)
    may = np.flatnonzero(labels >= 0)
    mask = np.zeros(int(cu[-1]), np.uint8)
    mask[np.random.default_rng(kept).permutation(may)[:kept]] = 1
    _check_head(shp, cu, Xf, gf, Wlm, labels, mask, "head V=%d kept=%d" % (V, kept))

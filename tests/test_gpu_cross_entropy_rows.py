"""The cross-entropy kernel that keeps a row of logits on the chip and fetches the next one meanwhile: vocabularies at the
edges of its three sizes, fewer and more rows than work-groups, labels in the first and last chunk, ignored rows."""
import numpy as np
import pytest

import synth_inputs as synth
from test_gpu_stack import _check_head, _head_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,rows", [(8, 70), (8192, 600), (32760, 1100), (32768, 33), (32776, 300), (65536, 260), (65544, 40),
                                    (131072, 520)])
@pytest.mark.parametrize("keep", [None, 0.6])
def test_rows(monkeypatch, V, rows, keep):
    monkeypatch.setitem(synth.SHAPES, "narrow", (128, 2, 1, 64, 128, 1e-5, 10000.0))
    shp, cu, Xf, gf, Wlm, labels = _head_case("narrow", V, [rows - 9, 9], 41, wstd=0.1)
    labels[:4] = [0, V - 1, V // 2, -1]
    mask = None if keep is None else synth.keep_mask(rows, keep, 7)
    _check_head(shp, cu, Xf, gf, Wlm, labels, mask, "rows V=%d" % V)

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


@pytest.mark.parametrize("V", [8200, 65536, 128256])
@pytest.mark.parametrize("counted", ["none", "first", "last", "every third", "first half"])
def test_rows_that_do_not_count(monkeypatch, V, counted):
    # (300 rows: the last work-groups' second row is the first they work on, or the other way round)
    monkeypatch.setitem(synth.SHAPES, "narrow", (128, 2, 1, 64, 128, 1e-5, 10000.0))
    shp, cu, Xf, gf, Wlm, labels = _head_case("narrow", V, [300], 43, wstd=0.1)
    rows = np.arange(300)
    keep = {"none": rows < 0, "first": rows == 0, "last": rows == 299, "every third": rows % 3 == 1, "first half": rows < 150}[counted]
    labels[:] = np.where(keep, np.random.default_rng(5).integers(0, V, 300), np.where(rows % 2, -1, V))
    _check_head(shp, cu, Xf, gf, Wlm, labels, None, "counted: " + counted, oracle_labels=np.where(keep, labels, -1))


def test_rows_that_do_not_count_are_not_read():
    # 4096 rows of 128,256 logits: read and written when they count, only cleared when they do not.  The reads are 1.05 GB,
    # 205 us at the rate of a large copy; half of that has to show in the time of the pass, whose other kernels do the same work.
    import torch
    import paper_2503_01066_amd as A
    from helpers import alch_shape
    shp = dict(hidden=128, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=128, rms_eps=1e-5, rope_base=10000.0)
    V, T = 128256, 4096
    g = torch.Generator(device="cuda").manual_seed(1)
    X, gf, Wlm = [torch.randn(*s, device="cuda", generator=g).to(torch.bfloat16) for s in ((T, 128), (128,), (V, 128))]
    batch, ignored = A.Batch(np.array([0, T], np.int32)), torch.full((T,), -1, dtype=torch.int32, device="cuda")
    ignored[0] = 5
    times = [[], []]
    for _ in range(12):
        for t, labels in zip(times, (torch.randint(0, V, (T,), dtype=torch.int32, device="cuda"), ignored)):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            A.alch_stack_backward(alch_shape(shp, "bf16"), batch, [], [], X, gf, Wlm, labels)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b) * 1e3)
    counted, cleared = [sorted(t)[3] for t in times]
    print("%.0f us when they count, %.0f us when they do not" % (counted, cleared))
    assert counted - cleared > 100, (counted, cleared)

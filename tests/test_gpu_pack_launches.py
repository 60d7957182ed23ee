"""Capture/pack around the limits of its launches: scan and gather in one (up to 4096 tokens, with and without a
work-group per stream), a scan of one work-group per 4096 tokens, boundaries on and beside the edges of both."""
import numpy as np
import pytest

import synth_inputs as synth
from oracle import gather_pack
from test_gpu_pack import run_pack, streams_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1], [15, 1], [16, 1], [256], [257, 0], [0, 4095], [4000, 96], [4096, 0, 0], [4097], [4096, 4096],
                                  [4080, 16, 1, 0, 4095, 0], [12288, 0, 17], [65536, 4464, 1]])
@pytest.mark.parametrize("keep,part", [(0.0, 1.0), (0.3, 0.5), (1.0, 1.0), (1.0, 0.9)])
def test_scan_and_gather(lens, keep, part):
    cu = synth.ragged_cu(lens)
    T = int(cu[-1])
    rng = np.random.default_rng(T)
    mask = (rng.random(T) < keep).astype(np.uint8) * rng.integers(1, 256, size=T).astype(np.uint8)
    capacity = max(1, int(T * part))
    for widths in ((8, 24, 2048), (6, 3 * 8)):  # 16-byte and 4-byte pieces
        srcs = streams_for(T, rng, widths=widths)
        kept, cu_kept, status, dsts = run_pack(cu, mask, srcs, capacity=capacity)
        ok, ocu, opacked = gather_pack(mask, cu, srcs)
        n = min(len(ok), capacity)
        assert status[0] == len(ok) and status[1] == (len(ok) > capacity)
        assert np.array_equal(cu_kept, ocu) and np.array_equal(kept[:n], ok[:n])
        for d, o in zip(dsts, opacked):
            assert np.array_equal(d[:n], o[:n].view(d.dtype))


@pytest.mark.parametrize("lens", [[1] * 3967, [3, 0, 14, 16, 1] * 200, [1, 2] * 3000])
@pytest.mark.parametrize("n_streams", [1, 20])
def test_many_boundaries(lens, n_streams):
    # more boundaries than threads, at every place inside the sixteen tokens of a thread, in either scan
    cu = synth.ragged_cu(lens)
    T = int(cu[-1])
    rng = np.random.default_rng(T)
    mask = (rng.random(T) < 0.4).astype(np.uint8)
    srcs = streams_for(T, rng, widths=(8,) * n_streams)
    kept, cu_kept, status, dsts = run_pack(cu, mask, srcs, capacity=T)
    ok, ocu, opacked = gather_pack(mask, cu, srcs)
    assert status[0] == len(ok) and np.array_equal(cu_kept, ocu) and np.array_equal(kept[:len(ok)], ok)
    for d, o in zip(dsts, opacked):
        assert np.array_equal(d[:len(ok)], o.view(d.dtype))

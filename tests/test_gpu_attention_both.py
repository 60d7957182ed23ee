"""Attention backward of short batches: dQ and dK/dV in one launch, behind one that forms delta.  Sequences beside key blocks of 128 and tiles
of 64, with and without cut key blocks, batches whose work-groups just find and just do not find compute units, against the definition."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, alch_shape, f64, rel_err, to_dev, to_np
from oracle import layer_backward_reuse
from test_gpu_layer import REC, make_case

pytestmark = pytest.mark.gpu


LENS = [[1], [64], [65, 1], [128], [129], [200, 0, 57], [320], [500], [513], [128] * 6, [128] * 8, [1000]]
HEADS = [(32, 8, 128), (32, 8, 64), (4, 4, 128), (32, 1, 64)]
FFN = 256
APART = [(h, lens) for h in HEADS if h != (4, 4, 128) for lens in LENS[-2:]]  # (too many work-groups)
# A feed-forward width that leaves room for the partial sums of cut key blocks (at 256 those of (32, 1, 64) alone find it)
WIDE_FFN, WIDE_LENS = 8192, [[100], [150], [201], [70, 70], [3, 130], [320], [513]]


@pytest.mark.parametrize("heads,lens,ffn", [(h, lens, FFN) for h in HEADS for lens in LENS] +
                         [(h, lens, WIDE_FFN) for h in HEADS[:2] for lens in WIDE_LENS])
def test_short_batches(monkeypatch, heads, lens, ffn):
    import paper_2503_01066_amd as A
    n_q, n_kv, D = heads
    monkeypatch.setitem(synth.SHAPES, "both", (256, n_q, n_kv, D, ffn, 1e-5, 10000.0))
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case("both", "bf16", cu, 7, "drawn", dy_std=0.01)
    ref = layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY.astype(np.float64))
    d = {k: to_dev(rec[k], "bf16") for k in REC}
    d["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    batch = A.Batch(cu)
    batch.c.max_seqlen = int(cu[-1]) + 300  # (a bound: any number that is not below the longest)
    out = A.alch_layer_backward(alch_shape(shp, "bf16"), batch, d, {k: to_dev(v, "bf16") for k, v in W.items()}, to_dev(dY, "bf16"))
    torch.cuda.synchronize()
    for k in ("dX", "dWq", "dWk", "dWv"):
        assert rel_err(to_np(out[k]), ref[k]) <= TOL["bf16"], (k, rel_err(to_np(out[k]), ref[k]))


# Stacks of several layers cut the key blocks of both launches alike, so that a sequence's gradients have the same bits whichever it is in.
# The same sequences alone, and beside so many others that dQ and dK/dV are launches of their own; nothing is counted in the others, and the
# sizes are such that no key block is cut and the products are cut alike.
BITS = [((32, 8, 128), [201]), ((32, 8, 64), [300]), ((32, 8, 128), [65, 130, 1]), ((32, 1, 64), [500]), ((32, 1, 64), [70, 300])]
OTHERS, BITS_FFN = [128] * 8, 64


@pytest.mark.parametrize("heads,lens", BITS)
def test_same_bits_as_two_launches(heads, lens):
    import paper_2503_01066_amd as A
    n_q, n_kv, D = heads
    g = torch.Generator(device="cuda").manual_seed(13)
    draw = lambda *s, std=1.0: torch.randn(s, generator=g, device="cuda").mul_(std).to(torch.bfloat16)
    own, T, hidden, V = sum(lens), sum(lens + OTHERS), 256, 512
    width = dict(X=hidden, X2=hidden, Q=n_q * D, K=n_kv * D, V=n_kv * D, O=n_q * D, G=BITS_FFN, U=BITS_FFN)
    size = dict(Wq=(n_q * D, hidden), Wk=(n_kv * D, hidden), Wv=(n_kv * D, hidden), Wo=(hidden, n_q * D), Wg=(BITS_FFN, hidden),
                Wu=(BITS_FFN, hidden), Wd=(hidden, BITS_FFN), g1=(hidden,), g2=(hidden,))
    recs = [dict({k: draw(T, w) for k, w in width.items()}, LSE=torch.full((T, n_q), 6.0, device="cuda")) for _ in range(2)]
    Ws = [{k: draw(*s, std=0.05) for k, s in size.items()} for _ in range(2)]
    X, gain, W_lm = draw(T, hidden), draw(hidden), draw(V, hidden, std=0.05)
    labels = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    labels[own:] = -1

    def gradient(cu):
        n = int(cu[-1])
        return A.alch_stack_backward(A.make_shape(hidden, n_q, n_kv, D, BITS_FFN, 1e-5, 10000.0, "bf16"), A.Batch(cu),
                                     [{k: v[:n] for k, v in r.items()} for r in recs], Ws, X[:n], gain, W_lm, labels[:n], want=())["dX_embed"]
    one, two = gradient(synth.ragged_cu(lens)), gradient(synth.ragged_cu(lens + OTHERS))
    assert torch.isfinite(one.float()).all() and float(one.float().abs().max()) > 0 and float(two[own:].float().abs().max()) == 0
    assert torch.equal(one, two[:own]), float((one.float() - two[:own].float()).norm() / one.float().norm())

"""Stacks of several layers under a loss mask: the data gradients of the head and of the top layer, sized by the kept rows, run whole in
tiles of 64x64 or 128x128 where no compute unit has a second one.  Kept counts beside both tiles, columns that are no whole large tile,
with and without the SwiGLU gradient behind the product, against the definition in 64 bits."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import f64
from oracle import stack_backward_reuse
from test_gpu_stack import check_stack, make_stack, run_stack

pytestmark = pytest.mark.gpu


QD = 256
# 64x64 tiles throughout; of dAct 130 x 8256 387 of them, 130 of 128x128; of dHf and dH2 1100 x 1088 306 and 81
CASES = ([(320, 640, 4160, 300, k, 0.05) for k in (1, 63, 64, 65, 129, 250)] + [(320, 8256, 512, 200, k, 0.05) for k in (128, 130)] +
         [(1088, 512, 320, 1300, k, 0.03) for k in (1024, 1025, 1100)])


@pytest.mark.parametrize("hidden,ffn,V,T,kept,wstd", CASES)
def test_kept_counts(monkeypatch, hidden, ffn, V, T, kept, wstd):
    monkeypatch.setitem(synth.SHAPES, "narrow", (hidden, 4, 2, 64, ffn, 1e-5, 10000.0))
    cu = synth.ragged_cu([T // 3, 1, T - T // 3 - 1])
    shp, osh, Ws, recs, Xf, gf, Wlm, labels = make_stack("narrow", "bf16", cu, 2, V, 17, wstd)
    mask = np.zeros(T, np.uint8)
    mask[np.random.default_rng(kept).permutation(np.flatnonzero(labels >= 0))[:kept]] = 1
    ref = stack_backward_reuse(osh, cu, None, [f64(r) for r in recs], [f64(W) for W in Ws], Xf.astype(np.float64), gf.astype(np.float64),
                               Wlm.astype(np.float64), labels, mask)
    check_stack(run_stack(shp, "bf16", cu, Ws, recs, Xf, gf, Wlm, labels, mask), ref, "bf16", 2)


# Kept rows of which the first count runs in 64x64 or 128x128 tiles and the second in 128x256 or 256x256 ones.  The loss is a mean over the
# kept rows and the counts are a power of two apart, so a row's gradients differ by that factor and by nothing else.
BITS_SHAPE, BITS_V, BITS_T = (2048, 4, 2, 64, 4096, 1e-5, 10000.0), 4160, 6200
BITS = [(63, 4032), (250, 4000), (500, 4000), (1000, 4000), (1537, 6148), (2048, 4096)]


@pytest.fixture(scope="module")
def single_tokens():
    """Two layers over sequences of one token: no row of a gradient depends on another row."""
    import paper_2503_01066_amd as A
    hidden, n_q, n_kv, D, ffn = BITS_SHAPE[:5]
    g = torch.Generator(device="cuda").manual_seed(9)
    draw = lambda *s, std=1.0: torch.randn(s, generator=g, device="cuda").mul_(std).to(torch.bfloat16)
    width = dict(X=hidden, X2=hidden, Q=n_q * D, K=n_kv * D, V=n_kv * D, O=n_q * D, G=ffn, U=ffn)
    size = dict(Wq=(n_q * D, hidden), Wk=(n_kv * D, hidden), Wv=(n_kv * D, hidden), Wo=(hidden, n_q * D), Wg=(ffn, hidden), Wu=(ffn, hidden),
                Wd=(hidden, ffn), g1=(hidden,), g2=(hidden,))
    recs = [dict({k: draw(BITS_T, w) for k, w in width.items()}, LSE=torch.zeros((BITS_T, n_q), device="cuda")) for _ in range(2)]
    Ws = [{k: draw(*s, std=0.05) for k, s in size.items()} for _ in range(2)]
    head = draw(BITS_T, hidden), draw(hidden), draw(BITS_V, hidden, std=0.05)
    labels = torch.randint(0, BITS_V, (BITS_T,), generator=g, device="cuda", dtype=torch.int32)
    batch, shape = A.Batch(np.arange(BITS_T + 1)), A.make_shape(*BITS_SHAPE, "bf16")

    def gradients(rows):
        mask = torch.zeros(BITS_T, dtype=torch.uint8, device="cuda")
        mask[rows] = 1
        return A.alch_stack_backward(shape, batch, recs, Ws, *head, labels, loss_mask=mask, want=())["dX_embed"][rows].float()
    return gradients


@pytest.mark.parametrize("few,many", BITS)
def test_same_bits_as_whole_large_tiles(single_tokens, few, many):
    rows = torch.from_numpy(np.sort(np.random.default_rng(few).permutation(BITS_T)[:many])).cuda()
    chosen = torch.from_numpy(np.sort(np.random.default_rng(many).permutation(many)[:few])).cuda()
    a, b = single_tokens(rows[chosen]), single_tokens(rows)[chosen]
    assert float(a.abs().min(1).values.max()) > 0 and torch.isfinite(a).all()
    assert torch.equal(a, b * (many // few)), float((a - b * (many // few)).norm() / a.norm())

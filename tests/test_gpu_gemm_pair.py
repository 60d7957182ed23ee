"""The 128x256-tile contraction kernel (two work-groups per compute unit) and the choice between it and the 256x256 one:
tile edges, remainders of the contraction, tiles cut along it, accumulate, column ranges that are cut, the order of either
kernel's sums."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import rel_err, to_dev, to_np
from test_gpu_gemm import operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,Ks", [(4104, 2048, (1024, 64)), (4104, 2304, (2048,)), (6000, 2048, (1024,))])
@pytest.mark.parametrize("a_k,b_k", [(True, False), (False, False)])
def test_whole_tiles_beside_cut_ones(a_k, b_k, M, N, Ks):
    # a little more than one tile for every compute unit: 33, 38 and 47 tiles for the 32 units of an XCD
    import paper_2503_01066_amd as A_
    rng = np.random.default_rng(M + N)
    terms, ref = [], 0.0
    for K in Ks:
        A, B, r = operands(rng, M, N, K, a_k, b_k, "bf16")
        terms.append((to_dev(A, "bf16"), to_dev(B, "bf16"), K))
        ref = ref + r
    ws = torch.empty(A_.lib().alch_gemm_workspace_bytes(), dtype=torch.uint8, device="cuda")
    outs = []
    for _ in range(2):
        C = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        A_.alch_gemm(M, N, terms, a_k, b_k, out=C, workspace=ws)
        torch.cuda.synchronize()
        assert rel_err(to_np(C), ref) < 6e-3  # one bf16 rounding of the output
        outs.append(C)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("a_k,b_k", [(True, False), (False, False), (True, True), (False, True)])
@pytest.mark.parametrize("M,N,Ks", [(8, 8, (64,)), (128, 256, (64, 128)), (136, 264, (192,)), (120, 520, (1024,)),
                                    (1000, 2048, (704,)),       # 8 x 8 tiles, no part of the contraction long enough to cut
                                    (488, 1032, (4096, 512)),   # 20 tiles, cut over both operand pairs
                                    (2056, 4360, (1024,))])     # 17 x 18 tiles: rounds of 64 per XCD and a remainder
def test_short_products(a_k, b_k, M, N, Ks):
    # a token-major operand alone also takes contractions that end inside a step of 32
    import paper_2503_01066_amd as A_
    if not (a_k or b_k):
        Ks = tuple(K - 13 for K in Ks)
    rng = np.random.default_rng(M + N + sum(Ks))
    terms, ref = [], 0.0
    for K in Ks:
        A, B, r = operands(rng, M, N, K, a_k, b_k, "bf16")
        terms.append((to_dev(A, "bf16"), to_dev(B, "bf16"), K))
        ref = ref + r
    C0 = synth.quantize(rng.standard_normal((M, N)).astype(np.float32) * 20, "bf16")
    ws = torch.empty(A_.lib().alch_gemm_workspace_bytes(), dtype=torch.uint8, device="cuda")
    for acc in (False, True):
        outs = []
        for w in (None, ws, ws):
            # the output is a column slice of a wider buffer whose other columns must stay untouched
            wide = torch.full((M, N + 16), 7.0, dtype=torch.bfloat16, device="cuda")
            C = wide[:, 8:N + 8]
            C.copy_(to_dev(C0, "bf16"))
            A_.alch_gemm(M, N, terms, a_k, b_k, out=C, accumulate=acc, workspace=w)
            torch.cuda.synchronize()
            assert rel_err(to_np(C), ref + C0 if acc else ref) < 6e-3   # one bf16 rounding of the output
            assert bool((wide[:, :8] == 7).all()) and bool((wide[:, N + 8:] == 7).all())
            outs.append(C.clone())
        assert torch.equal(outs[1], outs[2])                            # deterministic


@pytest.mark.parametrize("a_k,b_k,N,K", [(True, False, 4096, 8192), (False, False, 4096, 8192), (True, True, 4096, 28672)])
def test_both_kernels_add_in_the_same_order(a_k, b_k, N, K):
    # Few rows take the 128x256 kernel and 8192 the 256x256 one (long contractions; 8 tiles of 256 x 256 to an XCD against
    # 64).  Without scratch neither cuts the contraction, and the products of a row do not depend on the other rows: the
    # same bits, which is what stacks, cut alike in either kernel, rely on.
    import paper_2503_01066_amd as A_
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.randn(*((8192, K) if a_k else (K, 8192)), device="cuda", generator=g).to(torch.bfloat16)
    B = torch.randn(*((N, K) if b_k else (K, N)), device="cuda", generator=g).to(torch.bfloat16)
    whole = A_.alch_gemm(8192, N, [(A, B, K)], a_k, b_k)
    for rows in (256, 1000):
        few = A_.alch_gemm(rows, N, [(A[:rows] if a_k else A[:, :rows], B, K)], a_k, b_k)
        torch.cuda.synchronize()
        assert torch.equal(few, whole[:rows]), rows


@pytest.mark.parametrize("hidden,Hq,Hkv,D,ffn,rows", [(2048, 16, 8, 128, 1024, 300),    # 128x256 tiles, cut: 6 to an XCD of 16 parts
                                                      (1024, 8, 2, 128, 1536, 130),
                                                      (8192, 64, 8, 128, 512, 1792)])   # 35 tiles of 256x256 to an XCD, three of them cut
def test_column_ranges_that_are_cut(hidden, Hq, Hkv, D, ffn, rows):
    # q/k/v and gate/up of a layer forward as one product each, contractions long enough to be cut.  All positions are zero,
    # so that q and k come out as the product leaves them.
    import paper_2503_01066_amd as A_
    shape = A_.make_shape(hidden, Hq, Hkv, D, ffn, 1e-5, 10000.0, "bf16")
    g = torch.Generator(device="cuda").manual_seed(hidden + rows)
    rn = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)
    QD, KD = Hq * D, Hkv * D
    W = dict(Wq=rn(QD, hidden, std=0.02), Wk=rn(KD, hidden, std=0.02), Wv=rn(KD, hidden, std=0.02), Wo=rn(hidden, QD, std=0.02),
             Wg=rn(ffn, hidden, std=0.02), Wu=rn(ffn, hidden, std=0.02), Wd=rn(hidden, ffn, std=0.02), g1=rn(hidden), g2=rn(hidden))
    X = rn(rows, hidden)
    cu = np.minimum(np.arange(0, rows + 256, 256), rows).astype(np.int32)
    _, rec = A_.alch_layer_forward(shape, A_.Batch(cu, positions=np.zeros(rows, np.int32)), X, W)
    torch.cuda.synchronize()
    norm = lambda x, gain: (x.float() * torch.rsqrt(x.float().pow(2).mean(1, keepdim=True) + 1e-5) * gain.float()).to(torch.bfloat16).float()
    h1, h2 = norm(X, W["g1"]), norm(rec["X2"], W["g2"])
    for k, h, w in (("Q", h1, "Wq"), ("K", h1, "Wk"), ("V", h1, "Wv"), ("G", h2, "Wg"), ("U", h2, "Wu")):
        assert rel_err(to_np(rec[k]), to_np(h @ W[w].float().T)) < 8e-3, k  # one bf16 rounding, and a last bit of the rows' own

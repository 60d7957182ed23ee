"""The 128x256-tile contraction kernel (two work-groups per compute unit) and the choice between it and the 256x256 one:
tile edges, remainders of the contraction, tiles cut along it, several outputs, accumulate, device-resident sizes."""
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

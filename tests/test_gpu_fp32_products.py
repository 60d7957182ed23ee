"""fp32 products whose contractions are whole chunks (loads without conditions): fewer chunks than slices, several operand
pairs, ragged outputs, rows that do and do not allow loads of four elements, against fp64."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import rel_err, to_dev, to_np
from test_gpu_gemm import operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a_k,b_k", [(True, False), (False, False), (True, True), (False, True)])
@pytest.mark.parametrize("M,N,Ks", [(1, 1, (16,)), (15, 17, (64, 16)), (33, 31, (512,)), (352, 384, (8, 24)), (352, 330, (512, 16)),
                                    (47, 65, (1024, 256)), (256, 1024, (256,)), (353, 385, (1040,))])
def test_products_of_whole_chunks(M, N, Ks, a_k, b_k):
    # (error bound: as for the plain products, 1e-6 of the largest element for K <= 1025, times sqrt(1280 / 1025))
    import paper_2503_01066_amd as A_
    rng = np.random.default_rng(M + N + sum(Ks))
    terms, ref = [], 0.0
    for K in Ks:
        A, B, r = operands(rng, M, N, K, a_k, b_k, "f32")
        terms.append((to_dev(A, "f32"), to_dev(B, "f32"), K))
        ref = ref + r
    C0 = rng.standard_normal((M, N)).astype(np.float32)
    for acc in (False, True):
        C = to_dev(C0, "f32")
        A_.alch_gemm(M, N, terms, a_k, b_k, out=C, accumulate=acc)
        torch.cuda.synchronize()
        assert rel_err(to_np(C), ref + C0 if acc else ref) < 2e-6

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


@pytest.mark.parametrize("a_k,b_k", [(True, False), (False, False), (True, True), (False, True)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", [(5, 9, 0), (352, 384, 0), (1537, 1665, 0), (40, 24, 64), (352, 384, 512), (40, 24, 1024)])
def test_pairs_of_length_zero(a_k, b_k, M, N, K, dtype):
    # legal with NULL operands, alone (the product is zero) and beside a pair of whole chunks: nothing is read through them
    import ctypes
    import paper_2503_01066_amd as A_
    from paper_2503_01066_amd.binding import CGemmTerm
    A, B, ref = operands(np.random.default_rng(M + K), M, N, max(K, 1), a_k, b_k, dtype)
    dA, dB = to_dev(A, dtype), to_dev(B, dtype)
    empty = CGemmTerm(0, 0, 0, 0 if a_k else M, 0 if b_k else N)
    terms = [empty] if K == 0 else [empty, CGemmTerm(dA.data_ptr(), dB.data_ptr(), K, dA.stride(0), dB.stride(0)), empty]
    C0 = synth.quantize(np.random.default_rng(1).standard_normal((M, N)).astype(np.float32), dtype)
    for acc in (0, 1):
        C = to_dev(C0, dtype)
        rc = A_.lib().alch_gemm(0 if dtype == "f32" else 1, M, N, int(a_k), int(b_k), len(terms), (CGemmTerm * len(terms))(*terms),
                                ctypes.c_void_p(C.data_ptr()), C.stride(0), acc, None)
        torch.cuda.synchronize()
        want = (ref if K else 0.0 * ref) + (C0 if acc else 0)
        assert rc == 0 and rel_err(to_np(C), want) < (2e-6 if dtype == "f32" else 6e-3)


@pytest.mark.parametrize("a_k,b_k", [(True, False), (False, False), (True, True)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K,shift", [(1664, 1668, 16, 8), (1537, 1792, 40, 4), (1700, 1669, 33, 8), (1664, 1664, 65, 2)])
def test_tiles_leave_whole(a_k, b_k, M, N, K, shift, dtype):
    # 182 .. 196 tiles of 128x128 whose rows leave in pieces of four (N and the output's alignment allow it, or not), edge
    # tiles among them, into a column slice of a wider buffer whose other columns stay untouched
    import paper_2503_01066_amd as A_
    A, B, ref = operands(np.random.default_rng(M + N), M, N, K, a_k, b_k, dtype)
    C0 = synth.quantize(np.random.default_rng(1).standard_normal((M, N)).astype(np.float32), dtype)
    for acc in (False, True):
        wide = torch.full((M, (N + 2 * shift + 3) // 4 * 4), 7.0, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
        C = wide[:, shift:shift + N]
        C.copy_(to_dev(C0, dtype))
        A_.alch_gemm(M, N, [(to_dev(A, dtype), to_dev(B, dtype), K)], a_k, b_k, out=C, accumulate=acc)
        torch.cuda.synchronize()
        assert rel_err(to_np(C), ref + C0 if acc else ref) < (2e-6 if dtype == "f32" else 6e-3)
        assert bool((wide[:, :shift] == 7).all()) and bool((wide[:, shift + N:] == 7).all())

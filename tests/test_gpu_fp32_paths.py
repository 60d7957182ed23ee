"""The fp32-arithmetic kernels (fp32 storage, and bf16 problems the bf16 matrix-core kernels do not take) at the edges of
their tiles and on both sides of the choices between them, against fp64."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, f64, rel_err, to_dev, to_np
from oracle import attention_lse, layer_backward_reuse
from test_gpu_gemm import operands
from test_gpu_layer import REC, compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a_k,b_k", [(True, False), (False, False), (True, True), (False, True)])
@pytest.mark.parametrize("M,N,Ks", [(1, 1, (1,)), (15, 17, (63, 1)), (33, 31, (511, 514)), (352, 384, (40,)), (352, 330, (513, 7)),
                                    (1530, 1668, (65, 31)), (1537, 1665, (33,))])
def test_plain_products(M, N, Ks, a_k, b_k):
    # 16x16 tiles below 128 tiles of 32x32, those up to 159 tiles of 128x128, then 128x128; 4, 8 or 16 slices of the
    # contraction.  fp32: a sum of K products of order 1, each partial sum rounded to 2^-24: error well below
    # K^(1/2) 2^-23 of the result's norm in the random-sign case; 1e-6 of the largest element covers K <= 1025
    import paper_2503_01066_amd as A_
    rng = np.random.default_rng(M + N + sum(Ks))
    for dtype in ("f32", "bf16"):
        terms, ref = [], 0.0
        for K in Ks:
            A, B, r = operands(rng, M, N, K, a_k, b_k, dtype)
            terms.append((to_dev(A, dtype), to_dev(B, dtype), K))
            ref = ref + r
        C0 = synth.quantize(rng.standard_normal((M, N)).astype(np.float32), dtype)
        for acc in (False, True):
            C = to_dev(C0, dtype)
            A_.alch_gemm(M, N, terms, a_k, b_k, out=C, accumulate=acc)
            torch.cuda.synchronize()
            assert rel_err(to_np(C), ref + C0 if acc else ref) < (2e-6 if dtype == "f32" else 6e-3), (dtype, acc)


@pytest.mark.parametrize("D,lens", [(12, [1, 31, 33]), (32, [32, 65]), (64, [31, 97, 0, 2]), (70, [40, 33]), (128, [64, 130]), (256, [70, 3])])
def test_fp32_attention_head_sizes(D, lens):
    # every number of 32-column blocks, heads that are no multiple of four, sequences around the 32-row blocks and longer
    # than the four wavefronts of a work-group cover in one turn
    import paper_2503_01066_amd as A
    shp = dict(hidden=48, n_q_heads=4, n_kv_heads=2, head_dim=D, ffn=64, rms_eps=1e-5, rope_base=10000.0)
    from helpers import alch_shape, oracle_shape
    cu, osh = synth.ragged_cu(lens), oracle_shape(shp)
    T = int(cu[-1])
    W = synth.layer_weights(shp, 3, "f32", std=0.1)
    rec = synth.drawn_record(shp, T, 4, "f32")
    rec["LSE"] = attention_lse(osh, cu, rec["Q"].astype(np.float64), rec["K"].astype(np.float64)).astype(np.float32)
    dY = synth.activations(T, 48, 5, "f32", std=0.01)
    compare(run_gpu(shp, "f32", cu, W, rec, dY), layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY), "f32")
    O, lse = A.alch_attention_forward(alch_shape(shp, "f32"), A.Batch(cu), *[to_dev(rec[k], "f32") for k in "QKV"])
    Q, K, V = [rec[k].astype(np.float64).reshape(T, -1, D) for k in "QKV"]
    ref = np.zeros((T, 4, D))
    for a, b in zip(cu[:-1], cu[1:]):
        for h in range(4):
            S = np.where(np.tril(np.ones((b - a, b - a), bool)), Q[a:b, h] @ K[a:b, h // 2].T / np.sqrt(D), -np.inf)
            P = np.exp(S - S.max(axis=1, keepdims=True, initial=-np.inf))
            ref[a:b, h] = (P / P.sum(axis=1, keepdims=True)) @ V[a:b, h // 2]
    assert rel_err(to_np(O), ref.reshape(T, -1)) < 1e-5 and rel_err(to_np(lse), rec["LSE"]) < 1e-5

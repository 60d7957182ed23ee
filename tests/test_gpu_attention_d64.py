"""Attention with heads of 64 on the matrix cores: forward and backward at the edges of its tiles (32-key and 32-query
blocks, 64-row tiles, 128-row work-groups), ragged, grouped heads, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, alch_shape, f64, oracle_shape, rel_err, to_dev, to_np
from oracle import attention_lse, layer_backward_reuse
from test_gpu_layer import compare, make_case, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1, 31, 32, 33], [63, 64, 65, 0, 2], [127, 128, 129], [500, 191, 193]])
def test_heads_of_64_at_tile_edges(lens):
    import paper_2503_01066_amd as A
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case("medium64", "bf16", cu, 21, "drawn", dy_std=0.01)
    # forward: O and LSE from the drawn Q, K, V
    O, lse = A.alch_attention_forward(alch_shape(shp, "bf16"), A.Batch(cu), *[to_dev(rec[k], "bf16") for k in "QKV"])
    Hq, Hkv, D = shp["n_q_heads"], shp["n_kv_heads"], shp["head_dim"]
    ref = np.zeros((int(cu[-1]), Hq, D))
    Q, K, V = [rec[k].astype(np.float64).reshape(int(cu[-1]), -1, D) for k in "QKV"]
    for s in range(len(lens)):
        a, b = cu[s], cu[s + 1]
        for h in range(Hq):
            S = np.where(np.tril(np.ones((b - a, b - a), bool)), Q[a:b, h] @ K[a:b, h // (Hq // Hkv)].T / np.sqrt(D), -np.inf)
            P = np.exp(S - S.max(axis=1, keepdims=True, initial=-np.inf))
            ref[a:b, h] = (P / P.sum(axis=1, keepdims=True)) @ V[a:b, h // (Hq // Hkv)]
    assert rel_err(to_np(O), ref.reshape(to_np(O).shape)) <= TOL["bf16"]
    assert rel_err(to_np(lse), attention_lse(osh, cu, rec["Q"].astype(np.float64), rec["K"].astype(np.float64))) <= 1e-3
    # backward
    compare(run_gpu(shp, "bf16", cu, W, rec, dY), layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY), "bf16")

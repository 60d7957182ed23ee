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


def exposed_case(cu, Hkv, D, base, rng, dtype="bf16"):
    """A layer whose weight gradients are its attention's gradients: X, Wo and the normalised rows are the identity (hidden =
    tokens, a square number of them; gain 1 / sqrt(hidden), eps 0), Wd is zero, so that dO = dY and dWq = dQ^T, element for
    element.  Returns shape, weights, record without LSE, dY (fp32 numpy, rounded to dtype)."""
    T = int(cu[-1])
    assert int(np.sqrt(T)) ** 2 == T and T % (D * Hkv) == 0
    n = lambda *s, std=1.0: synth.quantize(rng.standard_normal(s).astype(np.float32) * np.float32(std), dtype)
    shp = dict(hidden=T, n_q_heads=T // D, n_kv_heads=Hkv, head_dim=D, ffn=128, rms_eps=0.0, rope_base=base)
    I = np.eye(T, dtype=np.float32)
    W = dict(Wq=n(T, T), Wk=n(Hkv * D, T), Wv=n(Hkv * D, T), Wo=I, Wg=n(128, T), Wu=n(128, T), Wd=np.zeros((T, 128), np.float32),
             g1=np.full(T, T ** -0.5, np.float32), g2=np.ones(T, np.float32))
    rec = dict(X=I, X2=n(T, T), Q=n(T, T), K=n(T, Hkv * D), V=n(T, Hkv * D), O=n(T, T, std=0.2), G=n(T, 128), U=n(T, 128))
    return shp, W, rec, n(T, T, std=0.01)


def attention_fp64(shp, cu, rec, dO, positions=None):
    """O, LSE and (from the LSE rounded to fp32, as a record holds it) dQ, dK, dV with the RoPE backward, in 64 bits."""
    Hq, Hkv, D = shp["n_q_heads"], shp["n_kv_heads"], shp["head_dim"]
    T = int(cu[-1])
    Q, K, V, O, g = [x.astype(np.float64).reshape(T, -1, D) for x in (rec["Q"], rec["K"], rec["V"], rec["O"], dO)]
    out = dict(O=np.zeros((T, Hq, D)), LSE=np.zeros((T, Hq)), dQ=np.zeros((T, Hq, D)), dK=np.zeros((T, Hkv, D)), dV=np.zeros((T, Hkv, D)))
    for a, b in zip(cu[:-1], cu[1:]):
        keep = np.tril(np.ones((b - a, b - a), bool))
        for h in range(Hq) if b > a else ():
            kv = h // (Hq // Hkv)
            S = np.where(keep, Q[a:b, h] @ K[a:b, kv].T / np.sqrt(D), -np.inf)
            mx = S.max(axis=1, keepdims=True)
            lse = mx + np.log(np.exp(S - mx).sum(axis=1, keepdims=True))
            out["LSE"][a:b, h] = lse[:, 0]
            out["O"][a:b, h] = np.exp(S - lse) @ V[a:b, kv]
            P = np.exp(S - lse.astype(np.float32).astype(np.float64))
            dS = P * (g[a:b, h] @ V[a:b, kv].T - (g[a:b, h] * O[a:b, h]).sum(axis=1, keepdims=True)) / np.sqrt(D)
            out["dQ"][a:b, h] = dS @ K[a:b, kv]
            out["dK"][a:b, kv] += dS.T @ Q[a:b, h]
            out["dV"][a:b, kv] += P.T @ g[a:b, h]
    pos = np.concatenate([np.arange(n) for n in np.diff(cu)]) if positions is None else positions
    ang = np.asarray(pos, np.float64)[:, None, None] * shp["rope_base"] ** (-2.0 * np.arange(D // 2) / D)
    for k in ("dQ", "dK"):
        lo, hi = out[k][..., :D // 2], out[k][..., D // 2:]
        out[k] = np.concatenate([lo * np.cos(ang) + hi * np.sin(ang), hi * np.cos(ang) - lo * np.sin(ang)], axis=-1)
    return {k: v.reshape(T, -1) for k, v in out.items()}


def run_exposed(shp, W, rec, lse, dY, cu, positions=None, dtype="bf16"):
    import paper_2503_01066_amd as A
    drec = {k: to_dev(v, dtype) for k, v in rec.items()}
    drec["LSE"] = torch.from_numpy(lse.astype(np.float32)).cuda()
    out = A.alch_layer_backward(alch_shape(shp, dtype), A.Batch(cu, positions=positions), drec, {k: to_dev(v, dtype) for k, v in W.items()},
                                to_dev(dY, dtype))
    torch.cuda.synchronize()
    return {k: to_np(out[w]).T for k, w in (("dQ", "dWq"), ("dK", "dWk"), ("dV", "dWv"))}


@pytest.mark.parametrize("Hkv,lens", [(4, [300, 1, 723]), (16, [128] * 8), (2, [1024])])
def test_heads_of_64_lose_nothing_but_the_rounding_of_their_results(Hkv, lens):
    import paper_2503_01066_amd as A
    cu = synth.ragged_cu(lens)
    shp, W, rec, dY = exposed_case(cu, Hkv, 64, 500000.0, np.random.default_rng(len(lens)))
    ref = attention_fp64(shp, cu, rec, dY)
    got = run_exposed(shp, W, rec, ref["LSE"], dY, cu)
    O, lse = A.alch_attention_forward(alch_shape(shp, "bf16"), A.Batch(cu), *[to_dev(rec[k], "bf16") for k in "QKV"])
    got["O"] = to_np(O)
    # Probabilities and dS that carry 16 bits put an error of about 2^-17 of its norm into a result, 0.5 % of that of the
    # one rounding to bf16 (1.6e-3): the two together are 1.00001 times the rounding.  Rounded to bf16 themselves they made
    # it 1.2 to 1.4 times.
    for k, v in got.items():
        err, rounding = np.linalg.norm(v - ref[k]), np.linalg.norm(synth.quantize(ref[k].astype(np.float32), "bf16") - ref[k])
        assert err <= 1.01 * rounding, (k, err / rounding)
    # one fp32 rounding of a number up to |LSE|, and that of the normaliser's sum and logarithm
    assert np.abs(to_np(lse) - ref["LSE"]).max() <= 2.0 ** -24 * np.abs(ref["LSE"]).max() + 2.0 ** -21


def test_more_sequences_than_a_grid_holds():
    # 65,538 sequences, all but two of one token: beyond the 65,535 of the matrix-core kernels' grid, and the same tokens in two
    # batches that fit it.  Outputs of a token depend on its own sequence alone.
    import paper_2503_01066_amd as A
    shp = dict(hidden=64, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=64, rms_eps=1e-5, rope_base=10000.0)
    lens = [1] * 32768 + [37] + [1] * 32768 + [70]
    T, rng = sum(lens), np.random.default_rng(3)
    W = {k: to_dev(v, "bf16") for k, v in synth.layer_weights(shp, 1, "bf16").items()}
    rec = {k: to_dev(v, "bf16") for k, v in synth.drawn_record(shp, T, 2, "bf16").items() if k != "LSE"}
    dY = to_dev(synth.activations(T, 64, 3, "bf16", std=0.01), "bf16")
    sh, half = alch_shape(shp, "bf16"), 32768 + 37

    def run(lens, rows):
        batch = A.Batch(synth.ragged_cu(lens))
        part = {k: v[rows].contiguous() for k, v in rec.items()}
        O, part["LSE"] = A.alch_attention_forward(sh, batch, part["Q"], part["K"], part["V"])
        dX = A.alch_layer_backward(sh, batch, part, W, dY[rows].contiguous(), want=())["dX"]
        torch.cuda.synchronize()
        return to_np(O), to_np(part["LSE"]), to_np(dX)

    whole = run(lens, slice(0, T))
    parts = [run(lens[:32769], slice(0, half)), run(lens[32769:], slice(half, T))]
    for i, tol in enumerate((TOL["bf16"], 1e-5, TOL["bf16"])):
        assert rel_err(whole[i], np.concatenate([p[i] for p in parts])) <= tol, i
    assert np.array_equal(whole[0][:32768], to_np(rec["V"])[:32768].repeat(2, 0).reshape(32768, -1))  # one key: O = V

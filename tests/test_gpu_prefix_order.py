"""Query blocks on a shared prompt are handed out by the keys they meet: every block of every sequence has to come up once,
also where the prompt is empty, where its blocks are whole, and where one rank is reached by a single sequence.  A prompt's
key blocks meet the tiles that need a mask first: whole and ragged tiles, own and of responses, more than 64 sequences on."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import TOL, to_dev, to_np, f64, rel_err, alch_shape, oracle_shape
from oracle.prefix import layer_backward_reuse_prefix, layer_forward_prefix
from test_gpu_prefix import REC, dev_record, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape_name,prompts,responses", [
    ("medium", [0, 129], [[2, 130], [1]]),             # nothing in front of the first two responses
    ("medium", [128, 256], [[128, 129], [256]]),       # whole blocks
    ("medium", [1, 385], [[400], [1]]),                # a response longer than its prompt; the last rank has one row
    ("medium64", [257, 1], [[1, 1], [130]]),
    ("medium", [385, 3], [[300, 20], [129]]),          # more ranks asked for than the longest sequence has blocks
    ("medium", [333, 320], [[64, 128, 0], [65, 192]]),  # ragged and whole tiles past the diagonal
    ("medium", [130, 70], [[33] * 66, [64, 65]]),
])
def test_every_query_and_key_block(shape_name, prompts, responses):
    import paper_2503_01066_amd as A
    shp, osh, b, W, X, _, _, rec, dY = make("bf16", shape_name, prompts, responses, 11)
    ref = layer_backward_reuse_prefix(osh, b["cu"], b["prefix"], f64(rec), f64(W), dY)
    batch = A.Batch(b["cu"], positions=b["positions"], prefix=b["prefix"])
    out = A.alch_layer_backward(alch_shape(shp, "bf16"), batch, dev_record(rec, "bf16"),
                                {k: to_dev(v, "bf16") for k, v in W.items()}, to_dev(dY, "bf16"))
    torch.cuda.synchronize()
    # dX takes the gradient of every row's query through Wq, dWq sums it over the rows (TOL: bf16 storage of all stages)
    for k in ("dX", "dWq", "dWk", "dWv"):
        assert rel_err(to_np(out[k]), ref[k]) <= TOL["bf16"], (k, rel_err(to_np(out[k]), ref[k]))
    for s in range(len(b["cu"]) - 1):
        lo, hi = int(b["cu"][s]), int(b["cu"][s + 1])
        if hi > lo:
            assert rel_err(to_np(out["dX"])[lo:hi], ref["dX"][lo:hi]) <= TOL["bf16"], s


def test_responses_of_a_prompt_far_apart():
    """Responses of two prompts in turn, so that those of either lie in three windows of 64 sequences; empty ones and one that
    names no prompt between them."""
    import paper_2503_01066_amd as A
    lens = [130, 0, 70] + [(0, 3, 64, 65, 17)[i % 5] for i in range(150)]
    prefix = [-1, -1, -1] + [(0, 2)[i % 2] for i in range(150)]
    prefix[80] = -1
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    at = [lens[p] if p >= 0 else 0 for p in prefix]
    pos = np.concatenate([a + np.arange(n) for a, n in zip(at, lens)]).astype(np.int32)
    shp, prefix = synth.shape_dict("medium"), np.array(prefix, np.int32)
    osh = oracle_shape(shp)
    W = synth.layer_weights(shp, 3, "bf16", std=0.02, gain_std=0.1)
    X = synth.activations(int(cu[-1]), shp["hidden"], 4, "bf16")
    _, rec64 = layer_forward_prefix(osh, cu, prefix, X.astype(np.float64), f64(W))
    rec = {k: synth.quantize(rec64[k].astype(np.float32), "bf16") for k in REC}
    rec["LSE"] = rec64["LSE"].astype(np.float32)
    dY = synth.activations(int(cu[-1]), shp["hidden"], 5, "bf16", std=0.01)
    ref = layer_backward_reuse_prefix(osh, cu, prefix, f64(rec), f64(W), dY)
    out = A.alch_layer_backward(alch_shape(shp, "bf16"), A.Batch(cu, positions=pos, prefix=prefix), dev_record(rec, "bf16"),
                                {k: to_dev(v, "bf16") for k, v in W.items()}, to_dev(dY, "bf16"))
    torch.cuda.synchronize()
    for k in ("dX", "dWq", "dWk", "dWv"):
        assert rel_err(to_np(out[k]), ref[k]) <= TOL["bf16"], (k, rel_err(to_np(out[k]), ref[k]))


def test_many_prompts_take_the_time_of_their_tokens():
    """The attention backward of 200 prompts of 40 tokens with two responses of 20 to each, against the same sequences on their
    own.  In tiles of 64 queries by 128 keys the prompts add 400 to 600 for dK/dV and as many for dQ (1.7 times the work); found
    one after the other, the responses of a key block cost it several times that."""
    import paper_2503_01066_amd as A
    n, H, F, Hq, Hkv, D = 200, 256, 256, 32, 8, 128
    lens, prefix = [40] * n + [20] * (2 * n), [-1] * n + [k // 2 for k in range(2 * n)]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    pos = np.concatenate([np.arange(40)] * n + [40 + np.arange(20)] * (2 * n)).astype(np.int32)
    T, g = int(cu[-1]), torch.Generator(device="cuda").manual_seed(1)
    draw = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    shape = A.make_shape(H, Hq, Hkv, D, F, 1e-5, 10000.0, "bf16")
    size = dict(Wq=(Hq * D, H), Wk=(Hkv * D, H), Wv=(Hkv * D, H), Wo=(H, Hq * D), Wg=(F, H), Wu=(F, H), Wd=(H, F))
    W = {k: draw(*s) * 0.02 for k, s in size.items()}
    W["g1"], W["g2"] = draw(H), draw(H)
    rec = {k: draw(T, w) for k, w in dict(X=H, X2=H, Q=Hq * D, K=Hkv * D, V=Hkv * D, O=Hq * D, G=F, U=F).items()}
    rec["LSE"] = torch.full((T, Hq), 12.0, device="cuda")
    dY = draw(T, H) * 0.01
    ms = []
    for batch in (A.Batch(cu, positions=pos), A.Batch(cu, positions=pos, prefix=np.array(prefix, np.int32))):
        A.alch_layer_backward(shape, batch, rec, W, dY)
        A.alch_trace_enable(True)
        for _ in range(5):
            A.alch_layer_backward(shape, batch, rec, W, dY)
        A.alch_trace_enable(False)
        ms.append(min(r[3] for r in A.alch_trace_collect() if r[0] == "attn_bwd"))
    print("alone %.3f ms, on their prompts %.3f ms" % tuple(ms))
    assert ms[1] <= 2.5 * ms[0], ms

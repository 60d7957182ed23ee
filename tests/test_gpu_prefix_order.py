"""Query blocks on a shared prompt are handed out by the keys they meet: every block of every sequence has to come up once,
also where the prompt is empty, where its blocks are whole, and where one rank is reached by a single sequence.  A prompt's
key blocks meet the tiles that need a mask first: whole and ragged tiles, own and of responses, more than 64 sequences on."""
import pytest
import torch

from helpers import TOL, to_dev, to_np, f64, rel_err, alch_shape
from oracle.prefix import layer_backward_reuse_prefix
from test_gpu_prefix import dev_record, make

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

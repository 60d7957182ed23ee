"""A data gradient and the weight gradient that runs beside it in one launch (dH2 with dWd, dO with [dWg; dWu], dH1 with
dWo): tokens below, at and beyond a tile, tiles cut along the contraction beside whole ones, tiles that do not fill a
work-group, accumulation."""
import numpy as np
import pytest
import torch

import synth_inputs as synth
from helpers import to_dev, f64, alch_shape
from oracle import layer_backward_reuse, WEIGHT_KEYS
from test_gpu_layer import REC, compare, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape_name,dtype,lens", [("medium", "bf16", [1]), ("medium", "bf16", [127, 2]), ("medium", "bf16", [256, 1]),
                                                   ("medium64", "bf16", [600]), ("config1", "f32", [16]), ("config1", "f32", [48, 80]),
                                                   ("config1", "f32", [528])])
def test_products_in_one_launch(shape_name, dtype, lens):
    import paper_2503_01066_amd as A
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case(shape_name, dtype, cu, 21, "drawn", dy_std=0.01)
    ref = layer_backward_reuse(osh, cu, None, f64(rec), f64(W), dY)
    dW = {k: to_dev(v, dtype) for k, v in W.items()}
    drec = {k: to_dev(rec[k], dtype) for k in REC}
    drec["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    once = A.alch_layer_backward(alch_shape(shp, dtype), A.Batch(cu), drec, dW, to_dev(dY, dtype), want=WEIGHT_KEYS)
    once = {k: v.clone() for k, v in once.items()}
    torch.cuda.synchronize()
    compare({k: v.double().cpu().numpy() for k, v in once.items()}, ref, dtype)
    grads = {k: v.clone() for k, v in once.items() if k != "dX"}
    twice = A.alch_layer_backward(alch_shape(shp, dtype), A.Batch(cu), drec, dW, to_dev(dY, dtype), grads=grads, accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(twice["dX"], once["dX"])
    for k in grads:
        # once more of the same, one rounding of the sum on top of the one that `once` carries
        want, eps = 2 * once[k].double(), 2.0 ** (-8 if dtype == "bf16" else -23)
        assert bool(((twice[k].double() - want).abs() <= 2 * eps * want.abs() + 1e-30).all()), k


# bf16: dAct, dH2 with dWd, dO with [dWg; dWu], dH1 with dWo, d[Wq; Wk; Wv] (three launches where k and v are no whole tiles).
# fp32: dH2 has 16 wavefronts to a tile and stays alone, so does dWd.
@pytest.mark.parametrize("shape_name,dtype,lens,launches", [("medium", "bf16", [127, 2], 5), ("medium64", "bf16", [256, 1], 7),
                                                            ("medium", "bf16", [511], 5), ("config1", "f32", [48, 80], 6)])
def test_they_are_one_launch_and_keep_their_bits(shape_name, dtype, lens, launches):
    import paper_2503_01066_amd as A
    cu = synth.ragged_cu(lens)
    shp, osh, W, rec, dY = make_case(shape_name, dtype, cu, 21, "drawn", dy_std=0.01)
    dW = {k: to_dev(v, dtype) for k, v in W.items()}
    drec = {k: to_dev(rec[k], dtype) for k in REC}
    drec["LSE"] = torch.from_numpy(rec["LSE"]).cuda()
    run = lambda want: {k: v.clone() for k, v in A.alch_layer_backward(alch_shape(shp, dtype), A.Batch(cu), drec, dW,
                                                                       to_dev(dY, dtype), want=want).items()}
    A.alch_trace_enable(True)
    both = run(WEIGHT_KEYS)
    A.alch_trace_enable(False)
    kinds = [r[0] for r in A.alch_trace_collect()]
    assert kinds.count("gemm_mfma" if dtype == "bf16" else "gemm_generic") == launches, kinds
    alone = run(())  # no weight gradients: dH2, dO and dH1 by themselves
    assert torch.equal(both["dX"], alone["dX"])
    if dtype == "bf16":  # one of [dWg; dWu] runs by itself, and at fewer than 512 tokens no weight gradient is cut
        for k in ("Wg", "Wu"):
            assert torch.equal(both["d" + k], run((k,))["d" + k]), k


def test_long_tiles_do_not_wait_for_short_ones():
    """dO of 640 tiles of 8 steps and [dWg; dWu] of 224 of 160 steps, in one launch or in two.  One launch with the short ones in
    front took 1.6 times both by themselves: the long ones come two to some compute units and none to others."""
    import paper_2503_01066_amd as A
    T, H, F, Hq, Hkv, D = 5120, 256, 14336, 32, 8, 128
    g = torch.Generator(device="cuda").manual_seed(1)
    draw = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    shape = A.make_shape(H, Hq, Hkv, D, F, 1e-5, 10000.0, "bf16")
    size = dict(Wq=(Hq * D, H), Wk=(Hkv * D, H), Wv=(Hkv * D, H), Wo=(H, Hq * D), Wg=(F, H), Wu=(F, H), Wd=(H, F))
    W = {k: draw(*s) * 0.02 for k, s in size.items()}
    W["g1"], W["g2"] = draw(H), draw(H)
    rec = {k: draw(T, w) for k, w in dict(X=H, X2=H, Q=Hq * D, K=Hkv * D, V=Hkv * D, O=Hq * D, G=F, U=F).items()}
    rec["LSE"] = torch.full((T, Hq), 12.0, device="cuda")
    dY, batch = draw(T, H) * 0.01, A.Batch(np.arange(6, dtype=np.int32) * 1024)
    d_gu, h2 = draw(T, 2 * F), draw(T, H)

    f_dO, f_dW = 2.0 * T * Hq * D * H, 2.0 * T * 2 * F * H

    def time_of(call):
        call()
        ms = []
        for _ in range(5):
            A.alch_trace_enable(True)
            call()
            A.alch_trace_enable(False)
            ms.append(sum(r[3] for r in A.alch_trace_collect() if r[1] in (f_dO, f_dW, f_dO + f_dW)))
        return min(ms)
    both = time_of(lambda: A.alch_layer_backward(shape, batch, rec, W, dY, want=("Wg", "Wu")))
    without = time_of(lambda: A.alch_layer_backward(shape, batch, rec, W, dY, want=()))  # (either holds dH2 too, as many operations)
    out = torch.empty((2 * F, H), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(A.lib().alch_gemm_workspace_bytes(), dtype=torch.uint8, device="cuda")
    dW = time_of(lambda: A.alch_gemm(2 * F, H, [(d_gu, h2, T)], False, False, out=out, workspace=ws))
    print("with weight gradients %.3f ms, without %.3f, weight gradients by themselves %.3f" % (both, without, dW))
    assert both - without <= 1.35 * dW, (both, without, dW)

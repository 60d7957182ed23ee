"""alch_capture_pack marshalled by the extension and in Python: the same outputs, and the same errors for what either refuses."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def both(monkeypatch, call):
    """(result or error) of the call with the extension, and without."""
    from paper_2503_01066_amd import binding
    assert binding._marshal is not None
    out = []
    for ext in (binding._marshal, None):
        monkeypatch.setattr(binding, "_marshal", ext)
        try:
            out.append(call())
        except Exception as e:  # noqa: BLE001 (compared below)
            out.append((type(e), str(e)))
    return out


@pytest.mark.parametrize("form", ["slices", "tuple", "one", "none", "many", "empty stream", "capacity 0", "short dsts", "not contiguous",
                                  "column step", "three dims", "host mask", "no tensor", "odd width"])
def test_forms(monkeypatch, form):
    import paper_2503_01066_amd as A
    T, keep = 37, 11
    g = torch.Generator(device="cuda").manual_seed(3)
    buf = torch.randn((T, 96), generator=g, device="cuda").to(torch.bfloat16)
    mask = torch.zeros(T, dtype=torch.uint8, device="cuda")
    mask[torch.from_numpy(np.random.default_rng(1).permutation(T)[:keep]).cuda()] = 1
    streams, capacity = [buf[:, :16], buf[:, 16:64], buf[:, 64:]], keep
    if form == "tuple": streams = tuple(streams)
    if form == "one": streams = streams[1:2]
    if form == "none": streams = []
    if form == "many": streams = [buf[:, 8 * (i % 9):8 * (i % 9) + 8] for i in range(70)]
    if form == "capacity 0": capacity = 0
    if form == "column step": streams = [buf[:, ::2]]
    if form == "three dims": streams = [buf.view(T, 4, 24)]
    if form == "no tensor": streams = [buf, None]
    if form == "odd width": streams = [buf[:, :1]]
    if form == "host mask": mask = mask.cpu()
    if form == "empty stream": streams = [buf[:0]]

    def call():
        dsts = [torch.zeros((capacity, s.shape[1]) if s is not None else 1, dtype=torch.bfloat16, device="cuda") for s in streams]
        if form == "short dsts": dsts = dsts[:-1]
        if form == "not contiguous": dsts[0] = torch.zeros((16, capacity), dtype=torch.bfloat16, device="cuda").t()
        if form in ("host mask", "empty stream"):  # (what these name is not followed: only the marshalling is looked at)
            from paper_2503_01066_amd import binding
            words = binding._streams(streams, dsts).tolist()
            native = binding._marshal and binding._marshal.capture_pack(0, 0, mask, streams, dsts, capacity, 1, mask, 0)
            return native, [w for i, w in enumerate(words) if i % 4 != 1]
        index, cu, status, d = A.alch_capture_pack(A.Batch(np.array([0, 20, T])), mask, streams, capacity=capacity, dsts=dsts)
        torch.cuda.synchronize()
        return [t.tolist() for t in (index[:capacity], cu, status)], [t.float().tolist() for t in d]
    native, python = both(monkeypatch, call)
    assert native == python
    if form in ("slices", "tuple", "one", "many"):
        want = torch.nonzero(mask).flatten()
        assert native[0][0] == want.tolist() and native[0][2] == [keep, 0]
        assert native[1] == [s[want].float().tolist() for s in streams]

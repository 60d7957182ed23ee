"""The alch_stream array of a capture call, word for word what the structures hold."""
import ctypes

import pytest
import torch

from paper_2503_01066_amd import binding as B


@pytest.mark.parametrize("n_dsts", [3, 1, 0])
def test_words_are_the_structures(n_dsts):
    wide = torch.zeros((5, 24), dtype=torch.bfloat16)
    streams = [wide[:, 8:16], torch.zeros((5, 6)), torch.zeros((0, 4), dtype=torch.uint8)]
    dsts = [torch.zeros((2, 8), dtype=torch.bfloat16), torch.zeros((2, 6)), torch.zeros((0, 4), dtype=torch.uint8)][:n_dsts]
    want = (B.CStream * 3)()
    strides = [24 * 2, 6 * 4, 4]
    for i, d in enumerate(dsts):
        want[i] = B.CStream(streams[i].data_ptr(), d.data_ptr(), streams[i].shape[1] * streams[i].element_size(), strides[i])
    words = B._streams(streams, dsts)
    assert words.itemsize * len(words) == ctypes.sizeof(want) and words.tobytes() == bytes(want)


@pytest.mark.parametrize("s,d", [(torch.zeros((4, 8)).t(), torch.zeros((8, 4))), (torch.zeros((4, 8)), torch.zeros((8, 4)).t())])
def test_columns_that_are_not_contiguous_are_refused(s, d):
    with pytest.raises(AssertionError):
        B._streams([s], [d])


def test_current_stream_without_the_private_lookup(monkeypatch):
    class Stream:
        cuda_stream = 0x1234
    monkeypatch.setattr(B, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    assert B._stream_handle(None) == 0x1234 and B._stream_handle(Stream()) == 0x1234

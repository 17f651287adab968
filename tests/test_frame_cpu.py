"""Host side of the frame decode: which frames are handed to the device unseen."""
import types

import pytest
import torch


class FakeUv:
    """A CUDA tensor [n][2] as FrameDecoder looks at it, on a host without one."""
    is_cuda = True

    def __init__(self, contiguous):
        self.contiguous = contiguous

    def reshape(self, *shape):
        return self

    def is_contiguous(self):
        return self.contiguous

    def numel(self):
        return 128

    def data_ptr(self):
        return 0x1000


class Reached(Exception):
    pass


def _decoder(monkeypatch):
    from paper_2506_06040_amd import api

    def reached(*a):
        raise Reached

    monkeypatch.setattr(api, "_require_ids", lambda t: None)
    monkeypatch.setattr(api.A, "lib", lambda: types.SimpleNamespace(ntc_classify_workspace=reached))
    fd = api.FrameDecoder.__new__(api.FrameDecoder)
    fd.materials, fd.packed, fd.n_out, fd.cfg, fd.out_dtype, fd.device = [None], [None], 4, None, torch.float32, "cpu"
    fd._table = None
    return fd


def test_strided_uv_is_not_decoded_unseen(monkeypatch):
    """A uv image whose rows are not adjacent pairs (a view into a wider image,
    an expanded pixel) is left to the path that refuses it."""
    fd = _decoder(monkeypatch)
    ids = torch.zeros((8, 8), dtype=torch.int16)
    out = torch.zeros((8, 8, 4))
    with pytest.raises(Reached):
        fd._decode_on_device(ids, FakeUv(True), out)
    assert fd._decode_on_device(ids, FakeUv(False), out) is False


def test_other_output_types_are_not_decoded_unseen(monkeypatch):
    """An output type that no decode writes: left to the path that refuses it
    where there is something to decode, and only there."""
    fd = _decoder(monkeypatch)
    fd.out_dtype = torch.bfloat16
    ids = torch.zeros((8, 8), dtype=torch.int16)
    assert fd._decode_on_device(ids, FakeUv(True), torch.zeros((8, 8, 4), dtype=torch.bfloat16)) is False

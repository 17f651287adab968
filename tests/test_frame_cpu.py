"""Host side of the frame decode: which frames are handed to the device unseen."""
import gc
import types
import weakref

import numpy as np
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


def test_a_captured_frame_keeps_its_table(monkeypatch):
    """The device image of the frame table that a captured decode reads
    outlives its replacement (other materials) as long as the decoder does."""
    fd = _decoder(monkeypatch)
    from paper_2506_06040_amd import api

    class Dev:
        def record_stream(self, s):
            pass

        def data_ptr(self):
            return 0x1000

    def size(*a):
        a[-1]._obj.value = 256
        return 0

    ok = lambda *a: 0
    monkeypatch.setattr(api.A, "lib", lambda: types.SimpleNamespace(
        ntc_classify_workspace=size, ntc_classify=ok, ntc_decode_frame_workspace=size, ntc_decode_frame=ok))
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0))
    fd._frame_table = lambda: fd._table
    fd._captured = []
    ids, out = torch.zeros((8, 8), dtype=torch.int16), torch.zeros((8, 8, 4))

    def decode(capturing):
        monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing)
        fd._table = (b"", np.zeros(4, np.uint8), Dev())
        ref = weakref.ref(fd._table[2])
        assert fd._decode_on_device(ids, FakeUv(True), out)
        assert fd._decode_on_device(ids, FakeUv(True), out)
        return ref

    captured, eager = decode(True), decode(False)
    fd._table = None
    gc.collect()
    assert captured() is not None and eager() is None
    assert len(fd._captured) == 1

"""What _lib takes from torch beside tensors: the current stream's handle, and
scratch memory that a call can do without."""


from paper_2202_08614_amd import _lib


def test_stream_handle_without_the_raw_call(monkeypatch):
    """torch's raw call is not part of its interface: without it the stream's
    own handle is taken."""
    import torch

    class Stream:
        cuda_stream = 0x1234

    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 0x1000 + d, raising=False)
    assert _lib._stream().value == 0x1003
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert _lib._stream().value == 0x1234


def test_refused_scratch_is_not_asked_for_on_every_call():
    """A request that ran out of memory is left out for the next 64 calls that
    want as much; smaller ones are made all the same."""
    import torch
    tree = _lib.DeviceTree(None, 1, 3, None, None, _lib.FPO_F32, 1, 1, None, _lib.make_layout())
    asked = []

    def give(n):
        asked.append(n)
        return n

    def refuse():
        asked.append("refused")
        raise torch.OutOfMemoryError("out of memory")

    assert _lib._scratch(tree, 500, lambda: give(500)) == 500
    assert _lib._scratch(tree, 1000, refuse) is None
    for _ in range(64):
        assert _lib._scratch(tree, 1000, lambda: give(1000)) is None
        assert _lib._scratch(tree, 999, lambda: give(999)) == 999
    assert _lib._scratch(tree, 1000, lambda: give(1000)) == 1000
    assert asked.count(1000) == 1 and asked.count(999) == 64


def test_no_records_without_coefficients():
    tree = _lib.DeviceTree(None, 1, 3, None, None, _lib.FPO_F32, 1, 1, None, _lib.make_layout())
    assert _lib.spare_record_workspace(tree, _lib.make_opts(), 100, "cpu") is None

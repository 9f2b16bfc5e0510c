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

"""CPU: the handle of the current stream comes from torch's raw accessor where there is one, and from the public stream object otherwise."""
import torch


def test_current_stream_without_the_raw_accessor(monkeypatch):
    from paper_2508_18376_amd import binding

    class Stream:
        def __init__(self, handle):
            self.cuda_stream = handle

    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream(1000 + device))
    assert binding._stream(Stream(7)) == 7
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 2000 + device, raising=False)
    monkeypatch.setattr(binding, "_raw_stream", binding._raw_stream_accessor())
    assert binding._stream(None) == 2003
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    monkeypatch.setattr(binding, "_raw_stream", binding._raw_stream_accessor())
    assert binding._stream(None) == 1003

"""The stream handle that the binding passes on, with and without torch's private accessor (no GPU needed)."""
import types

from paper_2605_05888_amd import binding


def test_handle_comes_from_the_public_stream_where_torch_has_no_raw_accessor(monkeypatch):
    import torch
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4711))
    assert binding._stream() == 4711


def test_handle_is_that_of_the_current_device(monkeypatch):
    import torch
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert binding._stream() == 103

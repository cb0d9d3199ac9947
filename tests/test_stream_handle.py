"""The raw handle of the current stream that the binding passes: taken from torch's internal
query where there is one, from the public Stream object where there is not."""
import types

import pytest
import torch

cola = pytest.importorskip("paper_2302_00850_amd.cola")


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_without_the_internal_query(missing, monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda: types.SimpleNamespace(cuda_stream=4711))
    monkeypatch.delattr(torch._C, missing, raising=False)
    assert cola._stream() == 4711


def test_with_it(monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 100 + d, raising=False)
    assert cola._stream() == 103


def test_before_torch_has_initialised_the_device(monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda: types.SimpleNamespace(cuda_stream=7))
    assert cola._stream() == 7

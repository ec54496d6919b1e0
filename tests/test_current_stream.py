"""The stream a call without one goes to: by its handle where torch has the function, by the stream object where it has not, or where
nothing has been set up yet."""
from types import SimpleNamespace

import pytest

from paper_2603_09237_amd import binding

torch = pytest.importorskip("torch")


@pytest.fixture
def stream_object(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=0x51))


@pytest.mark.parametrize("missing", ("_cuda_getCurrentRawStream", "_cuda_getDevice"))
def test_a_torch_without_the_private_functions(missing, monkeypatch, stream_object):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.delattr(torch._C, missing, raising=False)
    assert binding._stream() == 0x51


def test_before_anything_is_set_up(monkeypatch, stream_object):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    assert binding._stream() == 0x51


def test_of_the_current_device(monkeypatch, stream_object):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 0x100 + d, raising=False)
    assert binding._stream() == 0x103

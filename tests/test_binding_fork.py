"""A process forked from one that used the GPU cannot use it: torch says so
when it is asked for the current device or stream, and the binding does not go
round that with the default stream."""
import pytest

from paper_1907_06696_amd import mfgmg
from tests.test_binding_checks import Stub

torch = pytest.importorskip("torch")


@pytest.fixture
def forked(monkeypatch):
    """torch.cuda as a forked child finds it: a GPU there, not initialised, any use refused."""
    def refuse(*a):
        raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    monkeypatch.setattr(torch.cuda, "current_device", refuse)
    monkeypatch.setattr(torch.cuda, "current_stream", refuse)


def test_forked_process_is_refused(forked):
    with pytest.raises(RuntimeError, match="fork"):
        mfgmg.current_stream()
    t = Stub(8)
    t.device.index = 0
    with pytest.raises(RuntimeError, match="fork"):
        mfgmg._dev_ptr(t, 8, mfgmg.FP64, "x")


def test_without_a_gpu_the_default_stream(monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_available", lambda: False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    assert not mfgmg.current_stream().value

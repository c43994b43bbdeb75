"""The wrapper's launch helper: the device is made current only when it is not,
the stream is the current one of the tensors' device, and a non-zero status
raises (the device calls are stand-ins: no GPU needed)."""
import contextlib

import pytest
import torch

from paper_2302_08381_amd import _native


@pytest.mark.parametrize("current", [0, 1])
def test_call_device_and_stream(monkeypatch, current):
    entered = []

    @contextlib.contextmanager
    def device(d):
        entered.append(d.index)
        yield

    monkeypatch.setattr(torch.cuda, "current_device", lambda: current)
    monkeypatch.setattr(torch.cuda, "device", device)
    monkeypatch.setattr(_native, "_raw_stream", lambda index: 1000 + index)
    seen = []
    _native._call(torch.device("cuda", 1), lambda *a: seen.append((a, list(entered))) or 0, 7, None)
    assert seen == [((7, None, 1001), [] if current == 1 else [1])]


def test_call_raises_on_status(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(_native, "_raw_stream", lambda index: 0)
    with pytest.raises(_native.SphError) as e:
        _native._call(torch.device("cuda", 0), lambda *a: _native.SPH_ERR_LMAX)
    assert e.value.status == _native.SPH_ERR_LMAX


def test_call_refuses_cpu_tensors():
    Y = torch.zeros(2, 4)
    with pytest.raises((ValueError, RuntimeError)):
        _native.sph_e3nn_convert(Y, None, 1)

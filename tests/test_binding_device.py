"""The binding's launch helper without a GPU: which device and stream a call is queued on, and how
its return code surfaces. The library, the tensor and torch's device state are stand-ins."""
import contextlib

import pytest
import torch

import paper_2606_07574_amd as b4


class Tensor:
    def __init__(self, device):
        self.device_index = device

    def get_device(self):
        return self.device_index


@pytest.fixture
def state(monkeypatch):
    """current device, calls made as (device at the call, arguments); stream of device d: 100 + d."""
    s = {"device": 0, "calls": [], "code": 0}

    @contextlib.contextmanager
    def device(index):
        before, s["device"] = s["device"], index
        try:
            yield
        finally:
            s["device"] = before

    class Lib:
        def call(self, *args):
            s["calls"].append((s["device"], args))
            return s["code"]

        def birkhoff4_strerror(self, code):
            return b"text"

    monkeypatch.setattr(b4, "_lib", Lib())
    monkeypatch.setattr(torch.cuda, "device", device)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: s["device"], raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 100 + index, raising=False)
    return s


@pytest.mark.parametrize("current,tensor", [(0, 0), (0, 1), (3, 2), (2, 2)])
def test_device_and_stream(state, current, tensor):
    state["device"] = current
    b4._call("call", Tensor(tensor), 7, 8)
    assert state["calls"] == [(tensor, (7, 8, 100 + tensor))]
    assert state["device"] == current  # restored


@pytest.mark.parametrize("tensor", [0, 1])
def test_error_code(state, tensor):
    state["code"] = -6
    with pytest.raises(b4.Birkhoff4Error, match="-6: text"):
        b4._call("call", Tensor(tensor))
    assert state["device"] == 0

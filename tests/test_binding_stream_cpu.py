"""The address of the caller's current stream, as the binding passes it on, with a
stand-in for torch: no GPU needed."""
import sys
import types

import pytest

from paper_2202_11288_amd import binding as B


def fake_torch(raw):
    current = types.SimpleNamespace(cuda_stream=0x1230)
    cuda = types.SimpleNamespace(current_device=lambda: 3, current_stream=lambda: current)
    lib = types.SimpleNamespace(**({"_cuda_getCurrentRawStream": lambda d: 0x4560 + d} if raw else {}))
    return types.SimpleNamespace(cuda=cuda, _C=lib)


@pytest.mark.parametrize("raw,address", [(True, 0x4563), (False, 0x1230)])
def test_current_stream_with_and_without_the_short_look_up(monkeypatch, raw, address):
    monkeypatch.setitem(sys.modules, "torch", fake_torch(raw))
    monkeypatch.setattr(B, "_torch", None)
    monkeypatch.setattr(B, "_raw_stream", None, raising=False)
    assert B._stream(None).value == address


def test_streams_that_the_caller_names():
    assert B._stream(0x70).value == 0x70
    assert B._stream(types.SimpleNamespace(cuda_stream=0x80)).value == 0x80

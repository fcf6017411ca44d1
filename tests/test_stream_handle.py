"""The current stream's handle, with and without torch's internal functions."""
import types

import pytest

import paper_2607_08006_amd as v


def _fake(initialized, **internal):
    stream = types.SimpleNamespace(cuda_stream=77)
    cuda = types.SimpleNamespace(is_initialized=lambda: initialized, current_stream=lambda: stream)
    return types.SimpleNamespace(cuda=cuda, _C=types.SimpleNamespace(**internal))


@pytest.mark.parametrize("initialized,internal,want", [
    (True, dict(_cuda_getCurrentRawStream=lambda d: 100 + d, _cuda_getDevice=lambda: 3), 103),
    (False, dict(_cuda_getCurrentRawStream=lambda d: 100 + d, _cuda_getDevice=lambda: 3), 77),
    (True, dict(_cuda_getDevice=lambda: 3), 77),
    (True, dict(_cuda_getCurrentRawStream=lambda d: 100 + d), 77),
    (True, {}, 77),
])
def test_current_stream_handle(monkeypatch, initialized, internal, want):
    monkeypatch.setattr(v, "_torch", lambda: _fake(initialized, **internal))
    assert v._stream(None) == want

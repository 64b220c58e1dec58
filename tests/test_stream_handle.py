"""CPU: the handle of the current stream comes from torch's public call where its internal one is
not there."""
import types

import pytest

torch = pytest.importorskip("torch")

from paper_1310_2041_amd import hpf  # noqa: E402


def test_current_stream_without_the_internal_call(monkeypatch):
    monkeypatch.setattr(hpf.torch, "_C", types.SimpleNamespace())
    monkeypatch.setattr(hpf.torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert hpf._stream(None) == 77
    assert hpf._stream(5) == 5

"""The binding's stream handle where torch's private shortcuts are there and
where they are not."""
import types

import pytest

from paper_1204_0334_amd import ldpc


@pytest.mark.parametrize("missing", [(), ("_current_raw_stream",), ("_current_device",)])
def test_current_stream(monkeypatch, missing):
    monkeypatch.setattr(ldpc.torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(ldpc.torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(ldpc, "_current_device", lambda: 3)
    monkeypatch.setattr(ldpc, "_current_raw_stream", lambda device: 1000 + device)
    for name in missing:
        monkeypatch.setattr(ldpc, name, None)
    assert ldpc._stream_handle(None).value == (77 if missing else 1003)
    assert ldpc._stream_handle(types.SimpleNamespace(cuda_stream=5)).value == 5

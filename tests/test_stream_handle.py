"""The binding's handle of the current stream, on builds of torch with and
without the function that gives it directly."""
import types

import pytest

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import pdd  # noqa: E402


@pytest.mark.parametrize("direct", [True, False])
def test_current_stream(monkeypatch, direct):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x7A0))
    if direct:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x500 + device, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert pdd._stream_handle(None).value == (0x503 if direct else 0x7A0)
    assert pdd._stream_handle(types.SimpleNamespace(cuda_stream=0x44)).value == 0x44

"""The handle of the current stream that every call hands to the library: torch's
raw accessor, and the public interface where a torch has none."""
import types

import pytest
import torch


@pytest.mark.parametrize("missing", ["_raw_stream", "_raw_device"])
def test_public_interface_without_raw_accessors(monkeypatch, missing):
    from paper_2505_04612_amd import api
    monkeypatch.setattr(api, missing, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    assert api._stream() == 1234


@pytest.mark.gpu
def test_raw_handle_is_the_current_stream():
    from paper_2505_04612_amd import api
    assert api._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert api._stream() == side.cuda_stream != torch.cuda.default_stream().cuda_stream
    assert api._stream() == torch.cuda.default_stream().cuda_stream

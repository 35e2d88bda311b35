"""Which stream handle the binding passes to the library."""
import types

import pytest
import torch

from paper_2605_03884_amd import binding


def test_without_torchs_raw_stream_call_the_current_stream_is_asked(monkeypatch):
    monkeypatch.setattr(binding, "_current_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1234))
    assert binding._stream(None) == 0x1234
    assert binding._stream(types.SimpleNamespace(cuda_stream=0x55)) == 0x55


@pytest.mark.gpu
def test_both_ways_name_the_same_stream(monkeypatch):
    side = torch.cuda.Stream()
    seen = []
    for raw in (binding._current_raw_stream, None):
        monkeypatch.setattr(binding, "_current_raw_stream", raw)
        with torch.cuda.stream(side):
            seen += [binding._stream(None), binding._stream(side)]
    assert set(seen) == {side.cuda_stream}

"""Host logic: the handle of torch's current stream, with and without the private function that gives it directly."""
import importlib.util
import sys
from types import SimpleNamespace

import pytest
import torch

from paper_2504_12984_amd import binding as B


@pytest.mark.parametrize("present", [True, False])
def test_handle_of_the_current_stream(present, monkeypatch):
    # device 3 is current and its current stream is number 42; either way in gives that, and nothing else is asked for
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=42))
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    if present:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", {3: 42}.__getitem__, raising=False)
        monkeypatch.setattr(torch.cuda, "current_stream", None)
    spec = importlib.util.spec_from_file_location("binding_again", B.__file__)
    again = importlib.util.module_from_spec(spec)
    monkeypatch.setitem(sys.modules, "binding_again", again)
    spec.loader.exec_module(again)
    assert again._stream() == 42

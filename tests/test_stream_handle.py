"""The handle of the current stream, by torch's internal entry or, where torch
has none, by its public one."""
import importlib.util
import types

import pytest
import torch

from paper_2510_08491_amd import render


def test_without_the_internal_entry(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=77))
    spec = importlib.util.spec_from_file_location("paper_2510_08491_amd.render_again", render.__file__)
    again = importlib.util.module_from_spec(spec)
    monkeypatch.setitem(__import__("sys").modules, spec.name, again)
    spec.loader.exec_module(again)
    assert again._stream().value == 77


@pytest.mark.gpu
def test_same_handle_both_ways(monkeypatch):
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            handle = render._stream().value
            assert (handle or 0) == stream.cuda_stream
            with monkeypatch.context() as m:
                m.setattr(render, "_raw_stream", None)
                assert render._stream().value == handle

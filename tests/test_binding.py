"""Host-only checks of the binding."""
import importlib.util
import sys

import pytest
import torch

import paper_2507_16099_amd.fp8 as fp8


def _fresh(monkeypatch):
    """The binding's module, executed anew."""
    spec = importlib.util.spec_from_file_location("fp8_fresh", fp8.__file__)
    module = importlib.util.module_from_spec(spec)
    monkeypatch.setitem(sys.modules, spec.name, module)      # (dataclasses look their module up)
    spec.loader.exec_module(module)
    return module


@pytest.mark.parametrize("missing", [("_cuda_getCurrentRawStream",), ("_cuda_getDevice",), ("_cuda_getCurrentRawStream", "_cuda_getDevice")])
def test_imports_and_finds_the_stream_without_torchs_private_functions(monkeypatch, missing):
    """A CPU build of torch has neither function, another version may have other names."""
    for name in missing:
        monkeypatch.delattr(torch._C, name, raising=False)
    module = _fresh(monkeypatch)
    assert module.fp8_version() == fp8.fp8_version()

    class Stream:
        cuda_stream = 0x1234

    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    assert module._stream() == 0x1234

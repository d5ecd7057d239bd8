"""The stream handle the binding passes: the current stream's, also where torch
lacks the private calls that give it directly; a given stream's own."""
import importlib.util
import sys
import types

import torch

from paper_1810_11066_amd import bitserial as bs


def load_without(monkeypatch, *names):
    """The binding imported anew against a torch without the given names."""
    for n in names:
        monkeypatch.delattr(torch._C, n, raising=False)
    spec = importlib.util.spec_from_file_location(
        "paper_1810_11066_amd.bitserial_again", bs.__file__)
    mod = importlib.util.module_from_spec(spec)
    monkeypatch.setitem(sys.modules, spec.name, mod)
    spec.loader.exec_module(mod)
    return mod


def test_without_the_private_calls(monkeypatch):
    mod = load_without(monkeypatch, "_cuda_getCurrentRawStream",
                       "_cuda_getDevice")
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda: types.SimpleNamespace(cuda_stream=0x1234))
    assert mod._stream() == 0x1234


def test_direct_calls(monkeypatch):
    monkeypatch.setattr(bs, "_raw_device", lambda: 3)
    monkeypatch.setattr(bs, "_raw_stream", lambda dev: 0x1000 + dev)
    assert bs._stream() == 0x1003


def test_given_stream():
    assert bs._stream(types.SimpleNamespace(cuda_stream=7)) == 7

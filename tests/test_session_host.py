"""Host side of the session layer, without a GPU."""
import importlib.util
from types import SimpleNamespace

import torch

from paper_2504_10724_amd import session as S


def test_current_stream_without_the_private_function_of_torch(monkeypatch):
    """a torch that does not have it gives the handle through its public interface"""
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=4711))
    spec = importlib.util.spec_from_file_location("paper_2504_10724_amd.session_there", S.__file__)
    there = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(there)
    assert there._stream() == 4711

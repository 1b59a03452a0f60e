"""The stream that calls are ordered on, looked up with and without torch's raw
lookup (which is not a public name), on the CPU: torch's CUDA module is stood in
for."""
import types

import pytest
import torch

from paper_1010_4639_amd import cgmi


@pytest.mark.parametrize("lacks", [None, "_cuda_getCurrentRawStream", "_cuda_getDevice"])
@pytest.mark.parametrize("initialized", [True, False])
def test_current_stream(lacks, initialized, monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: initialized)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=41))
    names = {"_cuda_getCurrentRawStream": lambda d: 100 + d, "_cuda_getDevice": lambda: 3}
    for name, f in names.items():
        monkeypatch.setattr(torch._C, name, f, raising=False)
    if lacks:
        monkeypatch.delattr(torch._C, lacks)
    assert cgmi._current_stream() == (103 if initialized and not lacks else 41)


def test_torch_has_the_raw_lookup():
    """The fast way is the one that runs here."""
    assert hasattr(torch._C, "_cuda_getCurrentRawStream") and hasattr(torch._C, "_cuda_getDevice")

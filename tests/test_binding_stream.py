"""Where the binding gets the stream from: torch's getter by device number, or its public call where a torch has no such getter."""
import types

import pytest


class Tensor:
    def __init__(self, index):
        self.index, self.device = index, f"cuda:{index}"

    def get_device(self):
        return self.index


@pytest.mark.parametrize("getter", [True, False])
def test_stream_of_a_tensor(getter, monkeypatch):
    import torch
    from paper_2605_06057_amd import binding
    monkeypatch.setattr(binding, "_raw_stream", None)
    if getter:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 1000 + index, raising=False)
        monkeypatch.setattr(torch.cuda, "current_stream", None)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
        monkeypatch.setattr(torch.cuda, "current_stream", lambda index: types.SimpleNamespace(cuda_stream=1000 + index))
    assert [binding._stream_of(Tensor(i)) for i in (0, 3, 0)] == [1000, 1003, 1000]
    with pytest.raises(ValueError, match="GPU"):
        binding._stream_of(Tensor(-1))

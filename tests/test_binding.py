"""The binding's own work, without a GPU."""
import types

import torch

from paper_1904_10509_amd import sparse_attn as sa


def test_current_stream_with_and_without_torchs_raw_handle(monkeypatch):
    """The current stream's handle comes from torch's unnamed accessor where it exists, else from the public one."""
    asked = []

    def current_stream(device):
        asked.append(device)
        return types.SimpleNamespace(cuda_stream=77)

    monkeypatch.setattr(torch.cuda, "current_stream", current_stream)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 1000 + index, raising=False)
    assert sa._stream(None, torch.device("cuda", 3)) == 1003 and not asked
    assert sa._stream(None, torch.device("cuda")) == 77  # no index: the accessor takes none
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert sa._stream(None, torch.device("cuda", 3)) == 77
    assert asked == [torch.device("cuda"), torch.device("cuda", 3)]
    # a stream that the caller names, as an object or as a handle
    assert sa._stream(types.SimpleNamespace(cuda_stream=5), torch.device("cuda", 0)) == 5
    assert sa._stream(6, torch.device("cuda", 0)) == 6

"""The current stream's handle, on the CPU (torch's binding replaced)."""
import torch

import paper_1802_05799_amd as hv


def test_current_stream_of_a_device_without_an_index(monkeypatch):
    """torch.device("cuda") means the current device; a device with an index means that one."""
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 1000 + index, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert hv.current_stream(torch.device("cuda", 1)) == 1001
    assert hv.current_stream(torch.device("cuda", 0)) == 1000
    assert hv.current_stream(torch.device("cuda")) == 1003

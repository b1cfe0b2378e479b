"""Host side of the Python binding, without a GPU."""
import torch

from paper_2512_19720_amd import binding as pd


def test_prefill_workspace_belongs_to_the_device_whose_stream_runs_the_call(monkeypatch):
    """Kernels go to the current device's current stream.  Memory from another device's pool would go back to that
    pool when the call returns and could be handed out there while the kernel still runs here."""
    seen = []

    def empty(*args, **kw):
        seen.append(torch.device(kw["device"]))
        return "workspace"

    monkeypatch.setattr(torch, "empty", empty)

    class OnAnotherDevice:
        dtype, device = torch.float16, torch.device("cuda:1")

    assert pd._prefill_workspace(1024, 4096, 4096, OnAnotherDevice) == "workspace"
    assert seen == [torch.device("cuda")]                     # no index: the current device

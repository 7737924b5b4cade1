"""The binding's scratch buffers: a device named by any form torch takes, one
buffer per device, stream and tag, and no buffer on a device that is no GPU."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_device_forms():
    from paper_2607_01844_amd import moe
    i = torch.cuda.current_device()
    ref = moe.workspace(1000, torch.device("cuda", i), "forms")
    assert ref.is_cuda and ref.numel() >= 1000
    for dev in (torch.device("cuda"), "cuda", f"cuda:{i}", i, None):
        assert moe.workspace(1000, dev, "forms").data_ptr() == ref.data_ptr(), dev
    assert moe.workspace(1000, "cuda", "other").data_ptr() != ref.data_ptr()
    with torch.cuda.stream(torch.cuda.Stream()):
        assert moe.workspace(1000, "cuda", "forms").data_ptr() != ref.data_ptr()
    for dev in ("cpu", torch.device("cpu")):
        with pytest.raises(ValueError):
            moe.workspace(1000, dev, "forms")

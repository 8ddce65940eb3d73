"""The stream that a call's work and workspace go to is torch's current one of
the tensors' device, for every form in which a device is named."""
import pytest
import torch

pytestmark = pytest.mark.gpu

nb = pytest.importorskip("paper_2112_15079_amd")
from paper_2112_15079_amd import _capi as C  # noqa: E402


@pytest.mark.parametrize("device", [None, "cuda", "cuda:0", torch.device("cuda"),
                                    torch.device("cuda", 0)])
def test_current_stream_and_its_workspace(device):
    def handle():
        return torch.cuda.current_stream(device).cuda_stream

    assert C.stream_handle(device) == handle()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert C.stream_handle(device) == handle() == side.cuda_stream
        if device is not None:
            inner = C.workspace(512, device)
    assert C.stream_handle(device) == handle() != side.cuda_stream
    if device is not None:
        assert C.workspace(512, device).data_ptr() != inner.data_ptr()


def test_workspace_bytes_refuses_what_it_refused():
    n = C.workspace_bytes(C.OP_ACCEL, 100)
    assert n > 0 and C.workspace_bytes(C.OP_ACCEL, 100) == n
    with pytest.raises(C.ctypes.ArgumentError):
        C.workspace_bytes(C.OP_ACCEL, 100.0)
    for _ in range(2):
        with pytest.raises(ValueError):
            C.workspace_bytes(C.OP_ACCEL, 0)

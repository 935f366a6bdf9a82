"""The views that Network keeps of its buffers: made once per place, a tensor
object of the caller's own each time, and ordinary tensors whatever mode the
call that made them ran in. On the CPU, with a buffer in place of the device's."""

import pytest
import torch

from paper_2107_04092_amd import snn


def holder():
    net = object.__new__(snn.Network)
    net._torch, net.device, net._views, net.ctx = torch, torch.device("cpu"), {}, None
    return net


@pytest.mark.parametrize("dtype", [torch.float32, torch.int64])
def test_a_view_made_in_inference_mode_is_an_ordinary_tensor_later(dtype):
    net, buf = holder(), torch.zeros(256, dtype=torch.uint8)
    with torch.inference_mode():
        net._view(buf, buf.data_ptr() + 64, 8, dtype)
    v = net._view(buf, buf.data_ptr() + 64, 8, dtype)
    assert not v.is_inference()
    p = torch.ones(8, requires_grad=True)
    (p * v).sum().backward()  # saved for backward: refused for inference tensors
    v += 1
    assert buf[64:64 + 8 * dtype.itemsize].any()


def test_views_are_the_callers_own_objects_over_one_buffer():
    net, buf = holder(), torch.zeros(256, dtype=torch.uint8)
    a, b = (net._view(buf, buf.data_ptr(), 4, torch.int32) for _ in range(2))
    assert a is not b and a.data_ptr() == b.data_ptr()
    a.resize_(2)
    assert net._view(buf, buf.data_ptr(), 4, torch.int32).numel() == 4
    other = torch.ones(256, dtype=torch.uint8)
    with pytest.raises(RuntimeError):
        net._view(other, other.data_ptr() + 256, 4, torch.int32)

"""Host-side plane bookkeeping against torch's own answers: the size, pitch and
contiguity of a tensor's planes, and the output views of one allocation."""
import pytest
import torch

from paper_1807_08084_amd import ops as O


@pytest.mark.parametrize("t", [
    torch.empty(9, 3, 4), torch.empty(9, 4, 3).transpose(1, 2), torch.empty(3, 4, 9).permute(2, 0, 1),
    torch.empty(9, 8, 8)[:, ::2], torch.empty(9, 8, 8)[:, :, :3], torch.empty(9, 1, 8)[:, :, ::2],
    torch.empty(9, 8, 1).expand(9, 8, 5), torch.empty(1, 8, 5).expand(9, 8, 5), torch.empty(9, 0, 3),
    torch.empty(9, 5)[:, 1:], torch.empty(9, 10)[:, ::2], torch.empty(9, 6, 1, 4)[..., :1],
    torch.empty(9, 2, 3, 4)[:, :1], torch.empty(18, 4, 4)[::2]])
def test_layout_is_what_torch_says(t):
    assert O._layout(t) == (t[0].numel(), t.stride(0), t[0].is_contiguous())


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shape", [(1,), (5,), (3, 4), (1, 7), (7, 1), (1, 1), (2, 3, 4), (2, 1, 3), (0,), (0, 4)])
def test_planes_and_one_are_slices_of_one_buffer(shape, dtype):
    out = O.empty_planes(10, shape, dtype, "cpu")
    inv, det = O._planes_and_one(9, torch.Size(shape), dtype, "cpu")
    assert inv.shape == out[:9].shape and det.shape == out[9].shape
    assert inv.untyped_storage().nbytes() == out.untyped_storage().nbytes()
    assert inv.untyped_storage().data_ptr() == det.untyped_storage().data_ptr()
    if inv.numel():
        assert inv.stride() == out[:9].stride() and det.stride() == out[9].stride()
        assert inv.storage_offset() == 0 and det.storage_offset() == out[9].storage_offset()

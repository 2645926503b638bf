"""The views of the regenerated K and V that the step returns: the same elements, sizes and strides as slices of the workspace,
also where the workspace is itself a part of a tensor, has an odd number of bytes, or holds no regenerated token."""
import pytest
import torch

from paper_2501_01792_amd import binding


@pytest.mark.parametrize("L", [0, 1, 5])
@pytest.mark.parametrize("begin,end", [(0, 4096), (0, 4095), (2, 4098), (256, 4352)])
@pytest.mark.parametrize("el", [torch.float16, torch.bfloat16])
def test_views_are_slices_of_the_workspace(el, begin, end, L):
    workspace = torch.arange(8192, dtype=torch.int32).to(torch.uint8)[begin:end]
    size, offsets = (2, 3, L, 8), (256, 1024)
    n = 2 * 2 * 3 * L * 8
    for got, o in zip(binding._regenerated(workspace, el, offsets, size), offsets):
        ref = workspace[o:o + n].view(el).view(size)
        assert got.dtype == el and got.shape == ref.shape and got.is_contiguous() and got.stride() == ref.stride()
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16))
        if L:
            assert got.data_ptr() == ref.data_ptr()

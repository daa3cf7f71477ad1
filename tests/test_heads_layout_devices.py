"""A token order that lies on another GPU than the tensor is refused before any launch (its address would mean nothing to
the kernel), as gathering with it is by torch itself.  Stand-ins for device tensors: no GPU is needed."""
import pytest
import torch


class _OnDevice:
    is_cuda = True

    def __init__(self, shape, dtype, index):
        self.shape, self.dtype, self.device = torch.Size(shape), dtype, torch.device("cuda", index)

    def is_contiguous(self):
        return True

    def dim(self):
        return len(self.shape)

    def numel(self):
        return self.shape.numel()


def test_token_order_on_another_device_is_refused():
    import paper_2509_07120_amd as B
    order = _OnDevice((8,), torch.int32, 1)
    with pytest.raises(ValueError, match="device"):
        B.bsga_split_heads(_OnDevice((8, 3 * 2 * 64), torch.bfloat16, 0), 3, 2, order)
    with pytest.raises(ValueError, match="device"):
        B.bsga_merge_heads(_OnDevice((2, 8, 64), torch.bfloat16, 0), order)

"""Weights, biases and residuals that lie on another GPU than the tensor are refused before any launch (their addresses would mean
nothing to the kernel), as torch's own linear layer and layer norm refuse them.  Stand-ins for device tensors: no GPU is needed."""
import pytest
import torch

from tests.test_heads_layout_devices import _OnDevice


class _Tensor(_OnDevice):
    def get_device(self):
        return self.device.index


def _on(shape, index):
    return _Tensor(shape, torch.bfloat16, index)


@pytest.mark.parametrize("stray", ["weight", "bias", "residual"])
def test_linear_layer(stray):
    import paper_2509_07120_amd as B
    at = {n: int(n == stray) for n in ("weight", "bias", "residual")}
    with pytest.raises(ValueError, match=f"{stray}.*device"):
        B.bsga_linear(_on((8, 128), 0), _on((64, 128), at["weight"]), _on((64,), at["bias"]), residual=_on((8, 64), at["residual"]))


@pytest.mark.parametrize("stray", ["weight", "bias"])
def test_layer_norm(stray):
    import paper_2509_07120_amd as B
    at = {n: int(n == stray) for n in ("weight", "bias")}
    with pytest.raises(ValueError, match=f"{stray}.*device"):
        B.bsga_layer_norm(_on((8, 128), 0), _on((128,), at["weight"]), _on((128,), at["bias"]))

"""Splitting a projection's output into heads and merging them back, with and without a token order: every value
bit for bit what the strided copies of torch give, at token counts around the 32 (16) rows of a workgroup."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("N,parts,heads", [(1, 1, 1), (15, 3, 2), (31, 3, 16), (32, 1, 5), (33, 2, 3), (1374, 3, 16), (4099, 3, 7)])
def test_split_and_merge(B, dtype, N, parts, heads):
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randn((N, parts * heads * 64), generator=g, device="cuda").to(dtype)
    perm = torch.randperm(N, generator=g, device="cuda").to(torch.int32)
    plain = x.view(N, parts, heads, 64).permute(1, 2, 0, 3)
    assert torch.equal(B.bsga_split_heads(x, parts, heads), plain)
    assert torch.equal(B.bsga_split_heads(x, parts, heads, perm), plain[:, :, perm.long()])
    o = plain[0].contiguous()
    back = o.permute(1, 0, 2).reshape(N, heads * 64)
    assert torch.equal(B.bsga_merge_heads(o), back)
    assert torch.equal(B.bsga_merge_heads(o, perm), back[perm.long()])
    wild = torch.full((N,), N + 5, dtype=torch.int32, device="cuda")  # clamped to the last token
    wild[0] = -3
    want = torch.full((N,), N - 1, device="cuda")
    want[0] = 0
    assert torch.equal(B.bsga_split_heads(x, parts, heads, wild), plain[:, :, want])
    assert torch.equal(B.bsga_merge_heads(o, wild), back[want])


def test_errors(B):
    x = torch.zeros((4, 64), device="cuda")
    L = B.lib
    assert L.bsga_split_heads(x.data_ptr(), 1, 4, 1, 0, 64, None, x.data_ptr(), None) == 1
    assert L.bsga_split_heads(x.data_ptr(), 1, 4, 1, 1, 32, None, x.data_ptr(), None) == 2
    assert L.bsga_split_heads(None, 1, 4, 1, 1, 64, None, x.data_ptr(), None) == 1
    assert L.bsga_merge_heads(x.data_ptr() + 4, 1, 1, 4, 64, None, x.data_ptr(), None) == 1
    assert L.bsga_merge_heads(x.data_ptr(), 1, 1, 0, 64, None, x.data_ptr(), None) == 1
    with pytest.raises(ValueError):
        B.bsga_split_heads(x, 2, 1)
    with pytest.raises(ValueError):
        B.bsga_merge_heads(x.view(1, 4, 64), torch.zeros(3, dtype=torch.int32, device="cuda"))

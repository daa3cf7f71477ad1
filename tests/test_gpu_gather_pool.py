"""Token order and pooling in one pass against the two steps it stands for, bit for bit: ragged last blocks of either part, parts of no
tokens, more and fewer tokens than the source has, indices out of range."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("H,n_src,n,n_first", [(1, 1, 1, 1), (3, 300, 300, 129), (2, 257, 257, 257), (2, 200, 200, 0), (5, 1374, 1374, 1369),
                                               (2, 100, 333, 200), (2, 500, 65, 64)])
def test_same_as_the_two_steps(B, dtype, block, H, n_src, n, n_first):
    g = torch.Generator(device="cuda").manual_seed(n_src + n)
    q, k, v = (torch.randn((H, n_src, 64), generator=g, device="cuda").to(dtype) for _ in range(3))
    index = torch.randint(0, n_src, (n,), generator=g, device="cuda").int()
    if n > 300:
        index[7], index[8] = -3, 2 ** 30
    nb = B.split_blocks(n, n_first, block)
    out = [torch.full((H, n, 64), 7.0, device="cuda").to(dtype) for _ in range(3)]
    pools = [torch.full((H, nb, 64), 7.0, dtype=torch.float64, device="cuda") for _ in range(2)]
    ptr = [x.data_ptr() for x in (q, k, v)]
    rc = B.lib.bsga_gather_pool(*ptr, int(dtype == torch.float32), H, n_src, 64, index.data_ptr(), n, n_first, block,
                                *(x.data_ptr() for x in out + pools), torch.cuda.current_stream().cuda_stream)
    assert rc == 0, B.lib.bsga_last_error()
    want = [B.bsga_gather_tokens(x, index) for x in (q, k, v)]
    for got, ref in zip(out, want):
        assert torch.equal(got, ref)
    for got, ref in zip(pools, B.bsga_pool_qk_split(want[0], want[1], block, n_first)):
        assert torch.equal(got, ref)

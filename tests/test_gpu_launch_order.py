"""The launch order of the bf16 attention rows (longest first, made by one kernel up to 8192 units and by four
above) decides only which workgroup computes which row: with and without it every row is bitwise the same,
at the sizes where the way it is made changes and for rows and pairs of rows alike."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


@pytest.mark.parametrize("b,H,nb", [(128, 16, 64), (128, 41, 25), (128, 64, 128), (128, 67, 123), (64, 32, 64), (64, 127, 129), (64, 127, 130)])
def test_order_does_not_change_results(B, b, H, nb):
    N = nb * b - 5
    g = torch.Generator(device="cuda").manual_seed(nb)
    q, k, v = (torch.randn((H, N, 64), generator=g, device="cuda").bfloat16() for _ in range(3))
    cnt = torch.randint(0, 4, (H, nb), generator=g, device="cuda", dtype=torch.int32)
    cnt[:, ::11] = nb                      # some rows much longer than the rest
    idx = torch.rand((H, nb, nb), generator=g, device="cuda").argsort(-1).int()
    idx = torch.where(torch.arange(nb, device="cuda") < cnt[..., None], idx, nb).sort(-1).values
    idx = torch.where(idx < nb, idx, 0).int().contiguous()
    out = torch.full_like(q, float("nan"))
    for _ in range(2):
        B.bsga_sparse_attn(q, k, v, b, idx, cnt, out=out)
        plain = B.bsga_sparse_attn(q, k, v, b, idx, cnt, ordered=False)
        torch.cuda.synchronize()
        assert torch.equal(out, plain)     # no NaN left: every row was computed

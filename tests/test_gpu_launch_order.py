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


@pytest.mark.parametrize("H,nb", [(16, 172), (25, 83), (16, 130), (9, 230), (40, 53)])
def test_nor_what_whole_rounds_of_pairs_leave_over(B, H, nb):
    """Pairs of blocks of 64 from 1,024 pairs on, of which 256 leave 1 to 128 over, with odd numbers of blocks in a head, empty rows, and
    long rows from a few to half of all."""
    assert 1024 < H * ((nb + 1) // 2) <= 8192 and 1 <= H * ((nb + 1) // 2) % 256 <= 128
    N = nb * 64 - 5
    g = torch.Generator(device="cuda").manual_seed(nb)
    q, k, v = (torch.randn((H, N, 64), generator=g, device="cuda").bfloat16() for _ in range(3))
    for long_every in (11, 2):
        keep = torch.rand((H, nb, nb), generator=g, device="cuda") < 0.3
        keep[:, ::long_every] |= torch.rand((H, (nb + long_every - 1) // long_every, nb), generator=g, device="cuda") < 0.9
        keep[:, 5] = False
        cnt = keep.sum(-1).int()
        idx = (~keep).to(torch.int8).argsort(dim=-1, stable=True).int().contiguous()
        got, lse = B.bsga_sparse_attn(q, k, v, 64, idx, cnt, return_lse=True)
        plain, plain_lse = B.bsga_sparse_attn(q, k, v, 64, idx, cnt, return_lse=True, ordered=False)
        torch.cuda.synchronize()
        assert torch.equal(got, plain) and torch.equal(lse, plain_lse)
        assert bool((got[:, 5 * 64:6 * 64] == 0).all())

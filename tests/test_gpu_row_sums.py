"""The row sums of bf16 attention on blocks of 64, which `lse` returns, are sums of the fp32 weights, whichever way
the launch divides its rows.  softmax_scale = ln(2) / 8 makes the factor that is multiplied into Q a power of
two, so the scores are exact products of bf16 values and lse has no error but those of fp32: 64 products of up to a
few units in a score (64 * 2^-24 relative, at most 2e-6 here), exp2 and the sum (a few 2^-24).  Weights rounded
to bf16 before they are summed would move the lse of a row that a few keys dominate by up to 2^-9."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
BAR = 2e-5


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


# how the launch divides its rows: pairs of blocks, twice; four waves to a block, more rows than the chip holds and fewer; shared by tiles; two waves
@pytest.mark.parametrize("H,N", [(140, 1000), (94, 700), (48, 1000), (16, 1374), (1, 16400), (1024, 50)])
@pytest.mark.parametrize("density", [1.0, 0.6, 0.15])
def test_lse_of_blocks_of_64(B, H, N, density):
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v = (torch.randn((H, N, 64), generator=g, device="cuda").mul(s).bfloat16() for s in (2.0, 2.0, 1.0))
    nb = -(-N // 64)
    keep = torch.rand((H, nb, nb), generator=g, device="cuda") < density
    keep[:, :, 0] = True
    cnt = keep.sum(-1).int()
    idx = (~keep).to(torch.int8).argsort(dim=-1, stable=True).int().contiguous()
    _, lse = B.bsga_sparse_attn(q, k, v, 64, idx, cnt, softmax_scale=math.log(2.0) / 8.0, return_lse=True)
    torch.cuda.synchronize()
    member = torch.arange(N, device="cuda") // 64
    some = range(0, N, 64) if N < 4000 else (0, 64, 8192, (nb - 1) * 64)
    worst = 0.0
    for s in some:
        e = min(s + 64, N)
        logits = torch.bmm(q[:, s:e].double(), k.double().transpose(1, 2).contiguous()) * (math.log(2.0) / 8.0)
        logits.masked_fill_(~keep[:, s // 64][:, member][:, None, :], -math.inf)
        worst = max(worst, (lse[:, s:e].double() - torch.logsumexp(logits, -1)).abs().max().item())
    assert worst <= BAR, worst

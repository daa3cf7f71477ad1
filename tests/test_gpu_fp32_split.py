"""fp32 attention on operands split in three bf16 parts (launches of more than 128 units of 64 rows): as near to float64 as fp32
sums are, over logits and values of all sizes, and rows with values that the parts cannot hold."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
H, N = 16, 641  # 11 blocks of 64: 176 units


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


def _qkv(seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn((H, N, 64), generator=g, device="cuda") for _ in range(3)]


def _float64(q, k, v):
    s = q.double() @ k.double().transpose(1, 2).contiguous() / 8.0
    return torch.softmax(s, -1) @ v.double(), torch.logsumexp(s, -1)


@pytest.mark.parametrize("qs,ks,vs", [(1, 1, 1), (3, 3, 1), (10, 10, 1), (1e-30, 1e28, 1), (1e18, 1e-18, 1e30), (1, 1, 1e-30)])
def test_error_against_64_bits(B, qs, ks, vs):
    q, k, v = _qkv(1)
    q, k, v = q * qs, k * ks, v * vs
    out, lse = B.bsga_dense_attn(q, k, v, return_lse=True)
    o, l = _float64(q, k, v)
    # A logit of size L carries 2^-24 L from Q's scaling and as much again from its sum, a weight that times its size; the
    # sums of 641 weights add a few 2^-24.
    size = float((q.double().norm(dim=-1).max() * k.double().norm(dim=-1).max()) / 8.0)
    bar = 2.0 ** -24 * (4.0 + 2.0 * size)
    assert ((out.double() - o).norm() / o.norm()).item() <= bar
    # ... and lse the rounding of a base-2 logarithm, of its sum with the maximum and of their product with ln 2
    assert (lse.double() - l).abs().max().item() <= bar * 2 + 2.0 ** -24 * 4.0 * float(l.abs().max())
    if qs == ks == vs == 1:
        assert ((out.double() - o).norm() / o.norm()).item() <= 3.5e-7  # on the fp32 instructions: 4.1e-7


@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("what", ["q inf", "k inf", "v inf", "v nan", "v rounds to inf", "q rounds to inf", "k -inf"])
def test_values_that_the_parts_cannot_hold(B, what, block):
    """One such value in head 3: the workgroups that meet it start over on fp32 instructions, the others are not touched."""
    q, k, v = _qkv(2)
    plain = B.bsga_dense_attn(q, k, v)
    t = {"q": q, "k": k, "v": v}[what[0]]
    x = {"inf": float("inf"), "nan": float("nan"), "-inf": -float("inf"), "rounds to inf": 3.4e38}[what[2:]]
    t[3, 100, 7] = x
    if what == "q rounds to inf":
        k[3, :, 7] = 0.0    # the logits stay what they are without it
    nb = -(-N // block)
    idx = torch.arange(nb, dtype=torch.int32, device="cuda").expand(H, nb, nb).contiguous()
    cnt = torch.full((H, nb), nb, dtype=torch.int32, device="cuda")
    out = B.bsga_sparse_attn(q, k, v, block, idx, cnt)
    assert torch.equal(B.bsga_sparse_attn(q, k, v, block, idx, cnt).nan_to_num(), out.nan_to_num())
    others = torch.arange(H, device="cuda") != 3
    assert (out[others] - plain[others]).abs().max() <= 1e-5
    want = _float64(q[3:4], k[3:4], v[3:4])[0][0] if "rounds" in what else None
    got = out[3]
    if want is not None:
        # the value itself is weighted: sizes up to 3.4e38, an fp32 rounding of each term
        assert torch.isfinite(got).all()
        assert ((got.double() - want).abs().amax(0) / want.abs().amax(0)).max() <= 1e-5
    elif what == "v inf":
        assert torch.isposinf(got[:, 7]).all() and torch.isfinite(got[:, np.arange(64) != 7]).all()
    elif what == "v nan":
        assert torch.isnan(got[:, 7]).all() and torch.isfinite(got[:, np.arange(64) != 7]).all()
    elif what == "q inf":   # logits of +-inf in this row alone
        assert torch.isnan(got[100]).all() and torch.isfinite(got[np.arange(N) != 100]).all()
    else:                   # a key of infinite logits: +inf makes a row NaN, -inf weighs nothing
        up = (q[3, :, 7] > 0) == (what == "k inf")
        assert torch.isnan(got[up]).all() and torch.isfinite(got[~up]).all()

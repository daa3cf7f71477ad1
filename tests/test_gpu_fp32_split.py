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


@pytest.mark.parametrize("room", [False, True])     # K and V split by each workgroup, or once into the workspace
@pytest.mark.parametrize("qs,ks,vs", [(1, 1, 2.0 ** -99), (1, 1, 2.0 ** -101), (1, 1, 2.0 ** -112), (1, 1, 1e-34), (1, 1, 1e-36), (1, 1, 2e-38),
                                      (1e36, 1e-37, 1), (1e-37, 1e36, 1)])
def test_operands_whose_low_parts_end_below_bf16(B, room, qs, ks, vs):
    """Values of one size, so that each counts, and keys or queries so small that only the size of the others makes them count."""
    q, k, v = _qkv(7)
    v = v.sign() * (1.0 + v.abs().clamp(max=1.0)) * vs
    q, k = q * qs, k * ks
    out = B.bsga_dense_attn(q, k, v, workspace=torch.empty(H * N * 768 if room else 16, dtype=torch.uint8, device="cuda"))
    o, _ = _float64(q, k, v)
    size = float((q.double().norm(dim=-1).max() * k.double().norm(dim=-1).max()) / 8.0)
    # as above; values of both signs cancel to a fifteenth of their size, so what fp32 sums round counts for more
    assert ((out.double() - o).norm() / o.norm()).item() <= 2.0 ** -24 * (8.0 + 2.0 * size)


def test_a_column_of_small_values(B):
    """Beside ordinary ones and one of zeros: each to its own size."""
    q, k, v = _qkv(8)
    v[:, :, 9] = (1.0 + v[:, :, 9].abs()) * 1e-37
    v[:, :, 10] = 0.0
    out, (o, _) = B.bsga_dense_attn(q, k, v).double(), _float64(q, k, v)
    size = float((q.double().norm(dim=-1).max() * k.double().norm(dim=-1).max()) / 8.0)
    for d in (9, 11):
        assert ((out - o)[..., d].norm() / o[..., d].norm()).item() <= 2.0 ** -24 * (8.0 + 2.0 * size)
    assert (out[..., 10] == 0).all()


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


@pytest.mark.parametrize("room", [False, True])
def test_a_value_that_is_not_finite_costs_what_fp32_instructions_cost(B, room):
    """A call of which one head has to start over: 1.6 times as long as one of which none has (it was 3.5 times and more)."""
    n = 2748
    g = torch.Generator(device="cuda").manual_seed(11)
    q, k, v = (torch.randn((H, n, 64), generator=g, device="cuda") for _ in range(3))
    ws = torch.empty(H * n * 768 if room else 16, dtype=torch.uint8, device="cuda")

    def time():
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(10):
            B.bsga_dense_attn(q, k, v, workspace=ws)
        end.record()
        end.synchronize()
        return start.elapsed_time(end)

    time()
    plain = min(time() for _ in range(5))
    v[3, 100, 7] = float("nan")
    assert min(time() for _ in range(5)) <= 2.5 * plain

"""Linear layers and layer norms of the transformer block against float64, at sizes that reach every tile (256 x 192, 128 x 192,
128 x 128 with two and four buffers, 128 x 64) with ragged edges in tokens and features, and one step in k.

Bounds.  The sums are fp32: at most K roundings of 2^-24 of the running sum, which |x| |w| sums bound; then one rounding to bf16 (eight
significant bits: 2^-8 of the value at most, half an ulp just above a power of two) and, with a residual, a second one of the sum.  GELU's slope is at most 1.13 and its own error 3e-5."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


def _draw(N, K, F):
    g = torch.Generator(device="cuda").manual_seed(N + K + F)
    x = torch.randn((N, K), generator=g, device="cuda").bfloat16()
    w = (torch.randn((F, K), generator=g, device="cuda") / K ** 0.5).bfloat16()
    b = torch.randn((F,), generator=g, device="cuda").bfloat16()
    res = torch.randn((N, F), generator=g, device="cuda").bfloat16()
    perm = torch.randperm(N, generator=g, device="cuda").int()
    want = x.double() @ w.double().T + b.double()
    slack = K * 2.0 ** -24 * (x.double().abs() @ w.double().abs().T + b.double().abs())
    return x, w, b, res, perm, want, slack


def _close(got, want, slack, roundings=1):
    err = (got.double() - want).abs()
    bound = 1.2 * slack + 2.0 ** -8 * 1.01 * roundings * want.abs() + 1e-30
    assert bool((err <= bound).all()), float((err - bound).max())


@pytest.mark.parametrize("N,K,F", [(1, 64, 64), (70, 192, 192), (700, 128, 3008), (1374, 1024, 3008), (2748, 1024, 3136), (5000, 64, 4032),
                                   (193, 4096, 1024), (5000, 256, 4032), (5170, 1024, 4288)])
def test_linear(B, N, K, F):
    x, w, b, res, perm, want, slack = _draw(N, K, F)
    _close(B.bsga_linear(x, w, b), want, slack)
    gelu = torch.nn.functional.gelu(want)
    # launches of more tiles than the chip holds round to bf16 before the GELU as well as after it
    _close(B.bsga_linear(x, w, b, gelu=True), gelu, slack + 3e-5 * gelu.abs() + 1.13 * 2.0 ** -8 * want.abs())
    xh = x.view(N, K // 64, 64).transpose(0, 1).contiguous()
    _close(B.bsga_linear(xh, w, b, out_heads=True), want.view(N, F // 64, 64).transpose(0, 1), slack.view(N, F // 64, 64).transpose(0, 1))
    placed, placed_slack = torch.empty_like(want), torch.empty_like(slack)
    placed[perm.long()], placed_slack[perm.long()] = want, slack
    # rounded before the residual is added: the first rounding is one of the product
    _close(B.bsga_linear(xh, w, b, residual=res, row_index=perm), placed + res.double(), placed_slack + 2.0 ** -8 * 1.01 * placed.abs())


# sizes of which the narrow tiles with three, four and five buffers take several rounds: loads of the next tile are then on their way across the
# epilogue's stores and the loads of residuals and row numbers
@pytest.mark.parametrize("N,K,F", [(13000, 4096, 1024), (13985, 512, 832), (20000, 1024, 1024), (21961, 256, 320), (1333, 256, 3072), (5440, 256, 704)])
def test_residuals_of_several_rounds(B, N, K, F):
    x, w, b, res, perm, want, slack = _draw(N, K, F)
    placed, placed_slack = torch.empty_like(want), torch.empty_like(slack)
    placed[perm.long()], placed_slack[perm.long()] = want, slack
    xh = x.view(N, K // 64, 64).transpose(0, 1).contiguous()
    y = B.bsga_linear(xh, w, b, residual=res, row_index=perm)
    _close(y, placed + res.double(), placed_slack + 2.0 ** -8 * 1.01 * placed.abs())
    for _ in range(3):
        assert torch.equal(B.bsga_linear(xh, w, b, residual=res, row_index=perm), y)
    _close(B.bsga_linear(x, w, b, residual=res), want + res.double(), slack + 2.0 ** -8 * 1.01 * want.abs())
    # the residual's place is the result's
    st = torch.cuda.current_stream().cuda_stream
    for index, ref in ((None, B.bsga_linear(x, w, b, residual=res)), (perm, y)):
        out = res.clone()
        assert B.lib.bsga_linear(x.data_ptr(), 0, w.data_ptr(), b.data_ptr(), N, K, F, 0, None if index is None else index.data_ptr(),
                                 out.data_ptr(), 0, out.data_ptr(), st) == 0
        assert torch.equal(out, ref)


def test_gelu_of_values_that_are_not_numbers(B):
    x = torch.zeros((8, 64), device="cuda").bfloat16()
    x[0, 0], x[1, 0], x[2, 0], x[3, 0] = float("inf"), -3e38, 3e38, float("nan")
    w = torch.zeros((64, 64), device="cuda").bfloat16()
    w[:, 0] = 1
    y = B.bsga_linear(x, w, torch.zeros(64, device="cuda").bfloat16(), gelu=True)
    assert bool((y[0] == float("inf")).all()) and bool((y[1] == 0).all()) and bool((y[2] == x[2, 0]).all())
    assert bool(y[3].isnan().all()) and bool((y[4:] == 0).all())


@pytest.mark.parametrize("N,K,F", [(8, 64, 64), (5170, 1024, 4288)])  # from the sums; from tiles that wait in registers
def test_gelu_of_minus_infinity(B, N, K, F):
    """NaN, as the product of x and Phi(x) and as torch's: the limit 0 would hide that a sum has overflowed."""
    x, w = torch.zeros((N, K), device="cuda").bfloat16(), torch.zeros((F, K), device="cuda").bfloat16()
    w[:, 0] = 1
    x[0, 0], x[1, 0], x[2, 0] = -float("inf"), float("inf"), -30.5
    y = B.bsga_linear(x, w, torch.zeros(F, device="cuda").bfloat16(), gelu=True)
    assert bool(torch.nn.functional.gelu(x[0, 0]).isnan())
    assert bool(y[0].isnan().all()) and bool((y[1] == float("inf")).all()) and bool((y[2:] == 0).all())


@pytest.mark.parametrize("N,D", [(1, 8), (5, 512), (33, 520), (101, 1024), (7, 1536), (9, 4096)])
def test_layer_norm(B, N, D):
    g = torch.Generator(device="cuda").manual_seed(N + D)
    x = (3.0 + 2.0 * torch.randn((N, D), generator=g, device="cuda")).bfloat16()
    w, b = (torch.randn((D,), generator=g, device="cuda").bfloat16() for _ in range(2))
    perm = torch.randperm(N, generator=g, device="cuda").int()
    want = torch.nn.functional.layer_norm(x.double(), (D,), w.double(), b.double(), 1e-5)
    terms = (want - b.double()).abs() + b.double().abs()  # fp32 throughout: a few roundings of either term, and of the mean
    slack = 2.0 ** -20 * (terms + w.double().abs() * 4)
    _close(B.bsga_layer_norm(x, w, b), want, slack)
    _close(B.bsga_layer_norm(x, w, b, 1e-5, perm), want[perm.long()], slack[perm.long()])


@pytest.mark.parametrize("D", [8, 1000, 1024, 4096])
def test_layer_norm_of_values_whose_sum_is_too_large(B, D):
    """Rows whose values, but not their sum, fit fp32: the mean is finite, the variance is not, and what is left is the bias."""
    x = torch.full((6, D), 2.0 ** 127, device="cuda").bfloat16()
    x[1] = -x[1]
    x[2, ::2] = 2.0 ** 126
    x[3] = 1.0
    x[4, 0] = float("nan")
    w, b = (torch.randn((D,), generator=torch.Generator(device="cuda").manual_seed(D), device="cuda").bfloat16() for _ in range(2))
    y = B.bsga_layer_norm(x, w, b)
    assert bool((y[[0, 1, 2, 3, 5]] == b).all()) and bool(y[4].isnan().all())


def test_block_passes_agree(B):
    """The folded pass of the transformer block against its plain one on the same weights: roundings differ, by the bf16 ones."""
    N = 3 * 300
    special = (torch.arange(N) % 300) < 5
    blk = B.GlobalAttentionBlock(256, 4, 64, 0.9, 1.0, special=special, seed=1)
    x = torch.randn((N, 256), generator=torch.Generator().manual_seed(2)).bfloat16().cuda()
    assert blk._folds(x) and not blk._folds(x.float())
    with torch.autograd.forward_ad.dual_level():
        assert not blk._folds(x)
    y = blk(x)
    seen = []
    handle = blk.ln1.register_forward_hook(lambda *a: seen.append(1))
    assert not blk._folds(x)
    plain = blk(x)
    handle.remove()
    assert seen == [1]
    # the residual stream is O(1): a few bf16 roundings of values up to about 4
    assert float((y.double() - plain.double()).abs().max()) <= 8 * 2.0 ** -8 and float((y.double() - plain.double()).abs().mean()) <= 2.0 ** -8

"""Query blocks of 128 taken two to a workgroup of eight waves: dense launches of long rows (which ones, hostglue/check_api.cpp
tells: dense bits are the same both ways), and large sparse launches whose lists are long and of nearly one length (the rest
goes row by row).  Every mix of common and own blocks in the first
pairs, an odd number of blocks in a head, ragged last blocks, split sequences, key blocks of 64, uneven pairs and
empty rows among them, lists in any order, and rows that need the second pass."""
import pytest
import torch

from tests.helpers import bf16_bars_ok

pytestmark = pytest.mark.gpu
H, NB = 18, 301  # 5,418 rows: the launch order is made by one kernel


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


def _starts(n, n_first, block):
    return [(s, min(block, e - s)) for b, e in ((0, n_first), (n_first, n)) for s in range(b, e, block)]


def _reference(q, k, v, keep, rows, spans_q, spans_k):
    """float64 softmax attention of the given (head, query block) rows: [(h, start, length, o, lse)]"""
    member = torch.empty(k.shape[1], dtype=torch.long, device=k.device)
    for j, (s, m) in enumerate(spans_k):
        member[s:s + m] = j
    for h, i in rows:
        s, m = spans_q[i]
        at = torch.ones_like(member, dtype=torch.bool) if keep is None else keep[h, i][member]
        a = q[h, s:s + m].double() @ k[h, at].double().T / 8.0
        yield h, i, s, m, torch.softmax(a, 1) @ v[h, at].double(), torch.logsumexp(a, 1)


def _check(out, lse, q, k, v, keep, rows, spans_q, spans_k, shift=0.0):
    # with a shift: Q is rounded to bf16 after scaling (2^-9), which moves a logit of 91 nats by up to 0.2 and a weight by as
    # much; the bars of the other kernels' second pass
    for h, i, s, m, o, l in _reference(q, k, v, keep, rows, spans_q, spans_k):
        got, got_l = out[h, s:s + m], lse[h, s:s + m]
        if keep is not None and not keep[h, i].any():
            assert (got == 0).all() and torch.isneginf(got_l).all()
            continue
        if shift:
            d = (got.double() - o).abs()
            assert d.max() <= 5e-2 and d.mean() <= 5e-3 and (got_l.double() - l).abs().max() <= 0.25, (h, i)
            continue
        assert bf16_bars_ok(got[None], o.cpu().numpy()[None])[0], (h, i)
        # scores: Q's bf16 rounding after scaling, 2^-9 relative of scores up to a few units; weights' sums 2^-9
        assert (got_l.double() - l).abs().max() <= 2e-2, (h, i)


def _qkv(n, seed, shift=0.0, heads=H):
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.randn((heads, n, 64), generator=g, device="cuda") for _ in range(3))
    return [x.bfloat16() for x in (q + abs(shift) / 8.0, k + shift / 8.0, v)]


def _lists(keep, seed=0):
    cnt = keep.sum(-1).int()
    g = torch.Generator(device="cuda").manual_seed(seed)
    key = torch.rand(keep.shape, generator=g, device="cuda") if seed else torch.arange(keep.shape[-1], device="cuda").expand(keep.shape).float()
    return torch.where(keep, key, 1e9).argsort(-1).int().contiguous(), cnt


@pytest.mark.parametrize("n,n_first", [(NB * 128, NB * 128), (NB * 128 - 91, NB * 128 - 91), (300 * 128 + 40, 299 * 128 + 1)])
@pytest.mark.parametrize("bk", [128, 64])
@pytest.mark.parametrize("shift", [0.0, 27.0, -27.0])   # logits of +-91 nats: beyond the range of the first pass
def test_sparse_pairs(B, n, n_first, bk, shift):
    spans_q, spans_k = _starts(n, n_first, 128), _starts(n, n_first, bk)
    nb, nbk = len(spans_q), len(spans_k)
    g = torch.Generator(device="cuda").manual_seed(n + bk)
    keep = torch.rand((H, nb, nbk), generator=g, device="cuda") < 0.88
    mixes = [(c, a, b) for c in (0, 1, 2, 5) for a in (0, 1, 2, 3) for b in (0, 1, 2)] + [(9, 60, 0), (0, 7, 90)]
    rows = []
    for p, (c, a, b) in enumerate(mixes):          # short lists, one pair of rows each, the last block among the common ones
        js = torch.randperm(nbk - 1, generator=g, device="cuda")
        for i, own in ((0, js[c:c + a]), (1, js[c + a:c + a + b])):
            keep[1, 2 * p + i] = False
            keep[1, 2 * p + i, js[:c]] = True
            keep[1, 2 * p + i, own] = True
            keep[1, 2 * p + i, nbk - 1] = c == 2
            rows.append((1, 2 * p + i))
    keep[2, 4] = False                             # a pair of an empty row and a long one
    base = torch.rand(nbk, generator=g, device="cuda") < 0.9
    for p in range(4):                             # long lists that differ in few blocks
        keep[3, 2 * p:2 * p + 2] = base
        keep[3, 2 * p, p * 7:p * 7 + p] ^= True
        keep[3, 2 * p + 1, 100:100 + 2 * p] = False
        rows += [(3, 2 * p), (3, 2 * p + 1)]
    rows += [(2, 4), (2, 5), (0, 0), (0, nb - 1), (5, nb - 1), (5, nb - 2), (15, nb - 1), (15, 100)]
    q, k, v = _qkv(n, n, shift)
    idx, cnt = _lists(keep)
    out, lse = B.bsga_sparse_attn_split(q, k, v, 128, n_first, idx, cnt, return_lse=True, block_k=bk)
    _check(out, lse, q, k, v, keep, rows, spans_q, spans_k, shift)
    assert bool(torch.isfinite(out).all())
    again = B.bsga_sparse_attn_split(q, k, v, 128, n_first, idx, cnt, block_k=bk)
    assert torch.equal(out, again)
    idx, cnt = _lists(keep, seed=7)
    mixed, mlse = B.bsga_sparse_attn_split(q, k, v, 128, n_first, idx, cnt, return_lse=True, block_k=bk)
    _check(mixed, mlse, q, k, v, keep, rows[-8:] + rows[:8], spans_q, spans_k, shift)
    if n_first == n and not shift:                 # row by row it is the same up to rounding, and not the same bits
        one = B.bsga_sparse_attn(q, k, v, 128, *_lists(keep), ordered=False, block_k=bk)
        assert not torch.equal(out, one)
        d = (out.float() - one.float()).abs()
        assert d.max() <= 1e-2 and d.mean() <= 1e-3


@pytest.mark.parametrize("heads,n", [(16, 2748), (8, 5496), (3, 11000), (12, 13740 - 77), (16, 20400), (16, 43968), (1, 100001)])
def test_dense_pairs(B, heads, n):
    spans = _starts(n, n, 128)
    nb = len(spans)
    q, k, v = _qkv(n, n, heads=heads)
    out, lse = B.bsga_dense_attn(q, k, v, return_lse=True)
    rows = [(h, i) for h in {0, heads - 1} for i in {0, 1, nb // 2, nb - 2, nb - 1}]
    _check(out, lse, q, k, v, None, rows, spans, spans)
    assert torch.equal(out, B.bsga_dense_attn(q, k, v))
    hot = _qkv(n, n + 1, 27.0, heads=heads)        # logits of 91 nats: beyond the range of the first pass
    out, lse = B.bsga_dense_attn(*hot, return_lse=True)
    _check(out, lse, *hot, None, rows, spans, spans, 27.0)
    assert bool(torch.isfinite(out).all())
    assert bool(torch.isfinite(B.bsga_dense_attn(q * 30.0, k * 30.0, v)).all())


def test_many_sparse_pairs(B):
    """More rows than one kernel puts in order."""
    heads, n = 28, NB * 128 - 70
    spans = _starts(n, n, 128)
    g = torch.Generator(device="cuda").manual_seed(5)
    keep = torch.rand((heads, NB, NB), generator=g, device="cuda") < 0.9
    keep[7, 20] = keep[7, 21] = False
    keep[7, 20, 5:40] = True
    keep[9, 100, 30:200] = False                   # a pair that is taken apart
    q, k, v = _qkv(n, 6, heads=heads)
    idx, cnt = _lists(keep)
    out, lse = B.bsga_sparse_attn(q, k, v, 128, idx, cnt, return_lse=True)
    rows = [(7, 20), (7, 21), (9, 100), (9, 101), (0, 0), (0, NB - 1), (27, NB - 1), (13, 150), (27, 0)]
    _check(out, lse, q, k, v, keep, rows, spans, spans)
    one = B.bsga_sparse_attn(q, k, v, 128, idx, cnt, ordered=False)
    assert not torch.equal(out, one) and (out.float() - one.float()).abs().max() <= 1e-2
    keep = torch.rand((heads, NB, NB), generator=g, device="cuda") < 0.8   # rows of 240 tiles: one by one, the same bits
    idx, cnt = _lists(keep)
    assert torch.equal(B.bsga_sparse_attn(q, k, v, 128, idx, cnt), B.bsga_sparse_attn(q, k, v, 128, idx, cnt, ordered=False))


@pytest.mark.parametrize("heads,n", [(5200, 100), (2600, 256), (1800, 300)])
def test_dense_many_short_heads(B, heads, n):
    """Rows too short for pairs, and heads of one block, which have none."""
    spans = _starts(n, n, 128)
    q, k, v = _qkv(n, n, heads=heads)
    out, lse = B.bsga_dense_attn(q, k, v, return_lse=True)
    rows = [(h, i) for h in {0, 1, heads // 2, heads - 1} for i in range(len(spans))]
    _check(out, lse, q, k, v, None, rows, spans, spans)

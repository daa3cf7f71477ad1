"""fp32 attention at the sizes where its kernel can go wrong: 32-row units and 32-key pieces (one short of,
exactly and one past), blocks that end before their second piece, rows with fewer pieces than the four waves
that share them, empty rows, split sequences, descending lists.  Bars: outputs are convex combinations of
unit-normal values, logits of up to a few units carry a few 2^-24 relative errors, so 1e-5 absolute covers
a weight error of 2^-24 * 64 terms; lse the same."""
import numpy as np
import pytest
import torch

from oracle import bsga_oracle as O
from tests.helpers import to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


@pytest.mark.parametrize("b", [64, 128])
@pytest.mark.parametrize("wide", [False, True])  # 32 or 64 rows to a workgroup: chosen by the number of workgroups
@pytest.mark.parametrize("N,n_first", [(1, 1), (31, 31), (32, 32), (33, 33), (63, 63), (64, 64), (65, 65), (97, 97),
                                       (128, 128), (129, 129), (161, 161), (500, 500), (500, 129), (300, 31), (641, 609)])
def test_units_and_pieces(B, b, wide, N, n_first):
    rng = np.random.default_rng(N * 1000 + b)
    H = max(3, 200 // (len(O.block_ranges(N, b, n_first)) * (b // 64))) if wide else 3
    q, k, v = (rng.standard_normal((H, N, 64)).astype(np.float32) for _ in range(3))
    nb = len(O.block_ranges(N, b, n_first))
    mask = rng.random((H, nb, nb)) < 0.6
    mask[:, np.arange(nb), rng.integers(0, nb, nb)] = True
    idx, cnt = O.mask_to_index_lists(mask)
    for r in range(nb):  # one head's lists descend
        idx[1, r, :cnt[1, r]] = idx[1, r, :cnt[1, r]][::-1].copy()
    tidx, tcnt = torch.from_numpy(np.where(idx < 0, 0, idx)).cuda(), torch.from_numpy(cnt).cuda()
    tq, tk, tv = (to_device(x, "fp32") for x in (q, k, v))
    out, lse = B.bsga_sparse_attn_split(tq, tk, tv, b, n_first, tidx, tcnt, return_lse=True)
    torch.cuda.synchronize()
    want = O.sparse_attention(q, k, v, mask, b, n_first=n_first)
    assert np.abs(out.cpu().numpy() - want).max() <= 1e-5
    dense, dlse = B.bsga_dense_attn(tq, tk, tv, return_lse=True)
    assert np.abs(dense.cpu().numpy() - O.dense_attention(q, k, v)).max() <= 1e-5
    s = np.einsum("hid,hjd->hij", q.astype(np.float64), k.astype(np.float64)) / 8.0
    top = s.max(-1, keepdims=True)
    assert np.abs(dlse.cpu().numpy() - (top[..., 0] + np.log(np.exp(s - top).sum(-1)))).max() <= 1e-5


def test_empty_row_and_large_logits(B):
    rng = np.random.default_rng(5)
    H, N, b = 2, 200, 64
    q, k, v = (rng.standard_normal((H, N, 64)).astype(np.float32) for _ in range(3))
    q *= 40.0  # logits of +-300: the reference maximum moves, weights underflow
    nb = 4
    mask = np.ones((H, nb, nb), bool)
    idx, cnt = O.mask_to_index_lists(mask)
    cnt[0, 1] = 0
    out, lse = B.bsga_sparse_attn(*(to_device(x, "fp32") for x in (q, k, v)), b, torch.from_numpy(idx).cuda(),
                                  torch.from_numpy(cnt).cuda(), return_lse=True)
    torch.cuda.synchronize()
    assert (out[0, 64:128] == 0).all() and torch.isneginf(lse[0, 64:128]).all()
    want = O.sparse_attention(q, k, v, mask, b)
    got = out.cpu().numpy()
    keep = np.ones((H, N), bool)
    keep[0, 64:128] = False
    # logits of 300 nats carry an fp32 rounding error of about 300 * 2^-24 * a few, and so do the weights
    assert np.abs(got - want)[keep].max() <= 5e-4


@pytest.mark.parametrize("b", [64, 128])
@pytest.mark.parametrize("H", [2, 200])  # 32 and 64 rows to a workgroup
@pytest.mark.parametrize("N", [33, 70, 129])
def test_infinite_value_in_the_last_key(B, b, H, N):
    """The operands of keys past a ragged block's end are weighted by zero and must themselves be finite: an infinite
    value of the last key is a weighted term like any other, and its column is infinite, not NaN."""
    rng = np.random.default_rng(N)
    q, k, v = (rng.standard_normal((H, N, 64)).astype(np.float32) for _ in range(3))
    want = O.dense_attention(q[:2], k[:2], v[:2])
    v[:, -1, 5] = np.inf
    nb = O.num_blocks(N, b)
    idx, cnt = O.mask_to_index_lists(np.ones((H, nb, nb), bool))
    out = B.bsga_sparse_attn(*(to_device(x, "fp32") for x in (q, k, v)), b, torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda())
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.isposinf(got[..., 5]).all()
    rest = np.arange(64) != 5
    assert np.isfinite(got[..., rest]).all() and np.abs(got[:2][..., rest] - want[..., rest]).max() <= 1e-5


@pytest.mark.parametrize("H", [2, 200])
def test_whole_pieces_of_zero_weight(B, H):
    """Finite operands whose score overflows to -inf have weight zero, also where all 32 keys of a piece do."""
    rng = np.random.default_rng(8)
    N = 128
    q, k, v = (rng.standard_normal((H, N, 64)).astype(np.float32) for _ in range(3))
    q[..., 0] = 1e20
    k[..., 0] = 0.0
    seen = np.ones(N, bool)
    seen[32:70] = seen[96:] = False
    k[:, ~seen, 0] = -1e20
    idx, cnt = O.mask_to_index_lists(np.ones((H, 2, 2), bool))
    out, lse = B.bsga_sparse_attn(*(to_device(x, "fp32") for x in (q, k, v)), 64, torch.from_numpy(idx).cuda(),
                                  torch.from_numpy(cnt).cuda(), return_lse=True)
    torch.cuda.synchronize()
    s = np.einsum("hid,hjd->hij", q[:2].astype(np.float64), k[:2][:, seen].astype(np.float64)) / 8.0
    p = np.exp(s - s.max(-1, keepdims=True))
    want = np.einsum("hij,hjd->hid", p, v[:2][:, seen].astype(np.float64)) / p.sum(-1, keepdims=True)
    assert np.isfinite(out.cpu().numpy()).all() and np.abs(out[:2].cpu().numpy() - want).max() <= 1e-5
    want_lse = s.max(-1) + np.log(p.sum(-1))
    assert np.abs(lse[:2].cpu().numpy() - want_lse).max() <= 1e-5

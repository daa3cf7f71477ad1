"""Launches of few rows of blocks of 64 (fewer than 1024), each shared by four independent waves that take half a key block in turn: lists
of every length at which some waves have nothing to do, more than 64 pieces to a wave, ragged blocks shorter and longer than
half a block, split sequences, lists in any order, and rows that need the second pass."""
import numpy as np
import pytest
import torch

from oracle import bsga_oracle as O
from tests.helpers import attn_errors, bf16_bars_ok, to_device
from workload import bf16_bits_to_f32, round_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


def _run(B, H, N, n_first, lengths, seed, shift=0.0, shuffle=True):
    rng = np.random.default_rng(seed)
    q, k, v = (rng.standard_normal((H, N, 64)).astype(np.float32) for _ in range(3))
    q += abs(shift) / 8.0
    k += shift / 8.0
    q, k, v = (bf16_bits_to_f32(round_to_bf16_bits(x)) for x in (q, k, v))
    nb = len(O.block_ranges(N, 64, n_first))
    mask = np.zeros((H, nb, nb), dtype=bool)
    for h in range(H):
        for r in range(nb):
            mask[h, r, rng.permutation(nb)[:min(lengths[(h * nb + r) % len(lengths)], nb)]] = True
    idx, cnt = O.mask_to_index_lists(mask)
    idx = np.where(idx < 0, 0, idx)
    if shuffle:
        for h in range(H):
            for r in range(nb):
                idx[h, r, :cnt[h, r]] = rng.permutation(idx[h, r, :cnt[h, r]])
    out, lse = B.bsga_sparse_attn_split(*(to_device(x, "bf16") for x in (q, k, v)), 64, n_first, torch.from_numpy(idx).cuda(),
                                        torch.from_numpy(cnt).cuda(), return_lse=True)
    torch.cuda.synchronize()
    empty = ~mask.any(-1)
    want, want_lse = O.sparse_attention(q, k, v, np.where(empty[..., None], True, mask), 64, n_first=n_first, return_lse=True)
    for h, I in np.argwhere(empty):
        lo, hi = O.block_ranges(N, 64, n_first)[I]
        assert (out[h, lo:hi].float() == 0).all() and torch.isneginf(lse[h, lo:hi]).all()
        want[h, lo:hi] = want_lse[h, lo:hi] = np.nan
    seen = ~np.isnan(want_lse)
    return out, want, np.abs(lse.cpu().numpy() - want_lse)[seen].max()


@pytest.mark.parametrize("H,N,n_first", [(1, 1, 1), (2, 64, 64), (3, 65, 65), (2, 97, 97), (5, 640, 640), (16, 1374, 1374), (16, 1374, 1369),
                                         (4, 700, 333), (9, 6500, 6500)])
def test_lists_of_every_length(B, H, N, n_first):
    out, want, lse_err = _run(B, H, N, n_first, [1, 0, 2, 3, 4, 5, 7, 9, 64, 1000], seed=H + N)
    assert bf16_bars_ok(out, want)[0], bf16_bars_ok(out, want)
    assert lse_err <= 2e-2


def test_more_pieces_than_lanes(B):
    # 130 blocks of one head: waves of 65 pieces, which keep their list entries 64 at a time
    out, want, lse_err = _run(B, 1, 130 * 64 - 40, 130 * 64 - 40, [130, 129, 128, 127], seed=5)
    assert max(attn_errors(out, want)) <= 1e-2 and lse_err <= 2e-2


@pytest.mark.parametrize("shift", [-27.0, 27.0])  # logits near -91 and +91 nats; bars as for the other kernels' second pass
def test_second_pass(B, shift):
    out, want, lse_err = _run(B, 2, 4500, 4500, [71, 3, 1, 0, 66], seed=3, shift=shift)
    mx, mean = attn_errors(out, want)
    assert mx <= 5e-2 and mean <= 5e-3 and lse_err <= 0.25, (mx, mean, lse_err)

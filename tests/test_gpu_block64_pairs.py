"""Query blocks of 64 taken two to a workgroup (1024 rows and more): the key blocks both lists name, those of the first alone and
those of the second alone go different ways through the kernel.  Every combination of them being empty, odd
and even, an odd number of blocks in a head, a ragged last block in each of the three, split sequences,
lists in any order, and rows that need the second, online-softmax pass."""
import numpy as np
import pytest
import torch

from oracle import bsga_oracle as O
from tests.helpers import attn_errors, bf16_bars_ok, to_device
from workload import bf16_bits_to_f32, round_to_bf16_bits

pytestmark = pytest.mark.gpu
NB = 20  # key blocks of the hand-made masks
ROWS = 1024  # launches of fewer rows are not paired


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


def _qkv(H, N, seed, shift=0.0):
    rng = np.random.default_rng(seed)
    q, k, v = (rng.standard_normal((H, N, 64)).astype(np.float32) for _ in range(3))
    q += abs(shift) / 8.0
    k += shift / 8.0
    return [bf16_bits_to_f32(round_to_bf16_bits(x)) for x in (q, k, v)]


def _run(B, q, k, v, mask, n_first, shuffle=0):
    idx, cnt = O.mask_to_index_lists(mask)
    idx = np.where(idx < 0, 0, idx)
    if shuffle:
        rng = np.random.default_rng(shuffle)
        for h in range(idx.shape[0]):
            for r in range(idx.shape[1]):
                idx[h, r, :cnt[h, r]] = rng.permutation(idx[h, r, :cnt[h, r]])
    out, lse = B.bsga_sparse_attn_split(*(to_device(x, "bf16") for x in (q, k, v)), 64, n_first, torch.from_numpy(idx).cuda(),
                                        torch.from_numpy(cnt).cuda(), return_lse=True)
    torch.cuda.synchronize()
    return out, lse


def _check(out, lse, q, k, v, mask, n_first, heads=None):
    empty = ~mask.any(-1)
    ranges = O.block_ranges(q.shape[1], 64, n_first)
    want, want_lse = O.sparse_attention(q, k, v, np.where(empty[..., None], True, mask), 64, n_first=n_first, return_lse=True, heads=heads)
    for h, I in np.argwhere(empty):
        lo, hi = ranges[I]
        assert (out[h, lo:hi].float() == 0).all() and torch.isneginf(lse[h, lo:hi]).all()
        want[h, lo:hi] = np.nan
        want_lse[h, lo:hi] = np.nan
    assert bf16_bars_ok(out, want)[0], bf16_bars_ok(out, want)
    seen = ~np.isnan(want_lse)
    assert np.abs(lse.cpu().numpy() - want_lse)[seen].max() <= 2e-2


@pytest.mark.parametrize("tail", [64, 37, 1])            # length of the last block
@pytest.mark.parametrize("last", ["none", "both", "first", "second"])  # which list names it
@pytest.mark.parametrize("extra", [0, 8])                # 8 more common blocks: lists long enough to be sorted out
def test_every_mix_of_common_and_own_blocks(B, tail, last, extra):
    """One head per (common, first alone, second alone) with counts 0, 1, 2, 3; blocks 0 and 1 are the pair."""
    mixes = [(c, a, b) for c in range(4) for a in range(4) for b in range(4)]
    N = (NB - 1) * 64 + tail
    H = max(len(mixes), -(-ROWS // NB))
    rng = np.random.default_rng(tail)
    mask = rng.random((H, NB, NB)) < 0.5
    mask[:len(mixes), :2] = False
    for h, (c, a, b) in enumerate(mixes):
        js = rng.permutation(NB - 1)
        c += extra
        mask[h, 0, js[:c + a]] = True
        mask[h, 1, js[:c]] = True
        mask[h, 1, js[c + a:c + a + b]] = True
        mask[h, 0, NB - 1] = last in ("both", "first")
        mask[h, 1, NB - 1] = last in ("both", "second")
    q, k, v = _qkv(H, N, tail)
    out, lse = _run(B, q, k, v, mask, N)
    _check(out, lse, q, k, v, mask, N)


@pytest.mark.parametrize("N,n_first", [(65, 65), (128, 128), (129, 129), (1000, 1000), (1000, 300), (1000, 64), (777, 700), (4200, 4100)])
@pytest.mark.parametrize("density", [0.1, 0.9])
def test_shapes_and_list_orders(B, N, n_first, density):
    nb = len(O.block_ranges(N, 64, n_first))
    H = -(-ROWS // nb)
    mask = np.random.default_rng(N).random((H, nb, nb)) < density
    mask[0, :, 0] = True               # at least the first of the heads compared keeps something
    q, k, v = _qkv(H, N, N)
    out, lse = _run(B, q, k, v, mask, n_first)
    _check(out, lse, q, k, v, mask, n_first, heads=sorted({0, H // 2, H - 1}))
    again, _ = _run(B, q, k, v, mask, n_first, shuffle=1)
    if density > 0.5:
        assert torch.equal(out, again)  # the kernel sorts long lists itself
    _check(again, lse, q, k, v, mask, n_first, heads=sorted({0, H // 2, H - 1}))


@pytest.mark.parametrize("N,n_first", [(1, 1), (64, 64), (65, 65), (190, 190), (1000, 300), (1700, 1700)])
def test_up_to_512_rows(B, N, n_first):
    """Four independent waves to a block, as many blocks as the chip holds at once; counts 0, 1, 2, 3, ... and all."""
    nb = len(O.block_ranges(N, 64, n_first))
    H = max(1, min(8, 512 // nb))
    rng = np.random.default_rng(N)
    mask = np.zeros((H, nb, nb), bool)
    for h in range(H):
        for I in range(nb):
            mask[h, I, rng.permutation(nb)[:(h + I) % (nb + 1)]] = True
    mask[0, 0] = True
    q, k, v = _qkv(H, N, N)
    out, lse = _run(B, q, k, v, mask, n_first)
    _check(out, lse, q, k, v, mask, n_first)
    again, lse = _run(B, q, k, v, mask, n_first, shuffle=1)
    _check(again, lse, q, k, v, mask, n_first)


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("H,N", [(94, 700), (3, 700)])  # two blocks to a workgroup; one
def test_rows_out_of_range(B, sign, H, N):
    """Logits near +-91 nats; bars as for the other kernels' fallback."""
    q, k, v = _qkv(H, N, 11, 27.0 * sign)
    nb = O.num_blocks(N, 64)
    mask = np.random.default_rng(3).random((H, nb, nb)) < 0.5
    mask[:, :, 0] = True
    out, lse = _run(B, q, k, v, mask, N)
    want, want_lse = O.sparse_attention(q, k, v, mask, 64, return_lse=True)
    assert abs(np.median(want_lse)) > 70.0
    mx, mean = attn_errors(out, want)
    assert mx <= 5e-2 and mean <= 5e-3, (mx, mean)
    assert np.abs(lse.cpu().numpy() - want_lse).max() <= 0.25


def test_longest_list_that_fits(B):
    """4096 key blocks: the lists fill the LDS beside the tiles; one block more takes the other kernel."""
    for nb, seed in ((4096, 0), (4096, 1), (4097, 1)):
        N = nb * 64
        q, k, v = _qkv(1, N, nb)
        rng = np.random.default_rng(1)
        mask = rng.random((1, nb, nb)) < 0.002
        mask[0, :2] = rng.random((2, nb)) < (0.7 if seed else 0.2)
        mask[0, :, 0] = True
        out, lse = _run(B, q, k, v, mask, N)
        blocks = [0, 1, nb - 2, nb - 1]
        want = O.sparse_attention(q, k, v, mask, 64, q_blocks=blocks)
        assert bf16_bars_ok(out, want)[0], bf16_bars_ok(out, want)


@pytest.mark.parametrize("density", [0.2, 0.9])
@pytest.mark.parametrize("N,n_first", [(1500, 1500), (1590, 700), (4200, 4100)])
def test_uneven_neighbours(B, N, n_first, density):
    """Lists of very different length side by side: rows of a pair are then taken one by one.  Every second row keeps
    `density`, its neighbour one block, none, or a sixth; in the last head the long rows come second."""
    ranges = O.block_ranges(N, 64, n_first)
    nb = len(ranges)
    H = -(-ROWS // nb)
    rng = np.random.default_rng(N)
    mask = rng.random((H, nb, nb)) < density
    for h in range(H):
        short = np.arange(0 if h == H - 1 else 1, nb, 2)
        mask[h, short] = rng.random((short.size, nb)) < (0.0, 0.0, 0.17)[h % 3]
        if h % 3 == 1:
            mask[h, short, rng.integers(0, nb, short.size)] = True
    q, k, v = _qkv(H, N, N)
    out, lse = _run(B, q, k, v, mask, n_first)
    heads = sorted({0, 1, 2, H - 1})
    if N > 4000:
        heads = [0, H - 1]
    _check(out, lse, q, k, v, mask, n_first, heads=heads)
    again, again_lse = _run(B, q, k, v, mask, n_first, shuffle=1)
    _check(again, again_lse, q, k, v, mask, n_first, heads=heads)


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_uneven_rows_out_of_range(B, sign):
    """As test_rows_out_of_range with every second list short."""
    H, N = 47, 1400
    q, k, v = _qkv(H, N, 12, 27.0 * sign)
    nb = O.num_blocks(N, 64)
    mask = np.ones((H, nb, nb), bool)
    mask[:, 1::2, 2:] = False
    out, lse = _run(B, q, k, v, mask, N)
    want, want_lse = O.sparse_attention(q, k, v, mask, 64, return_lse=True, heads=[0, 20, 46])
    mx, mean = attn_errors(out, want)
    assert mx <= 5e-2 and mean <= 5e-3, (mx, mean)
    seen = ~np.isnan(want_lse)
    assert np.abs(lse.cpu().numpy() - want_lse)[seen].max() <= 0.25


@pytest.mark.parametrize("H,N", [(16, 4096), (16, 4225), (64, 1060), (12, 6500), (9, 9200), (16, 7300)])
def test_pairs_that_go_row_by_row(B, H, N):
    """512 to 1023 pairs: none, few, many left after the first 512, the last of them taken row by row; odd numbers of
    blocks in a head."""
    nb = O.num_blocks(N, 64)
    assert 512 <= H * ((nb + 1) // 2) < 1024
    mask = np.random.default_rng(N).random((H, nb, nb)) < 0.4
    mask[:, :, 0] = True
    mask[H - 1, nb - 1] = False
    q, k, v = _qkv(H, N, N)
    out, lse = _run(B, q, k, v, mask, N)
    again, _ = _run(B, q, k, v, mask, N)
    assert torch.equal(out, again)
    _check(out, lse, q, k, v, mask, N, heads=[0, H - 1])
    assert torch.isfinite(out.float()).all()


@pytest.mark.parametrize("density", [0.1, 0.9])
@pytest.mark.parametrize("H,N,n_first", [(513, 64, 64), (300, 65, 40), (60, 700, 700), (47, 700, 333), (10, 5100, 5037), (33, 1000, 64)])
def test_513_to_1023_rows(B, H, N, n_first, density):
    """Four independent waves to a block, more blocks than the chip holds at once; empty rows, ragged and split
    sequences, any order of the list."""
    nb = len(O.block_ranges(N, 64, n_first))
    assert 512 < H * nb < 1024
    rng = np.random.default_rng(N + H)
    mask = rng.random((H, nb, nb)) < density
    mask[0, :, 0] = True
    mask[H - 1, nb - 1] = False
    q, k, v = _qkv(H, N, N)
    heads = sorted({0, H // 2, H - 1})
    out, lse = _run(B, q, k, v, mask, n_first)
    _check(out, lse, q, k, v, mask, n_first, heads=heads)
    again, again_lse = _run(B, q, k, v, mask, n_first, shuffle=1)
    _check(again, again_lse, q, k, v, mask, n_first, heads=heads)


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_513_to_1023_rows_out_of_range(B, sign):
    """As test_rows_out_of_range for the launches between."""
    H, N = 60, 700
    q, k, v = _qkv(H, N, 13, 27.0 * sign)
    nb = O.num_blocks(N, 64)
    mask = np.random.default_rng(3).random((H, nb, nb)) < 0.5
    mask[:, :, 0] = True
    out, lse = _run(B, q, k, v, mask, N)
    want, want_lse = O.sparse_attention(q, k, v, mask, 64, return_lse=True, heads=[0, 30, 59])
    mx, mean = attn_errors(out, want)
    assert mx <= 5e-2 and mean <= 5e-3, (mx, mean)
    seen = ~np.isnan(want_lse)
    assert abs(np.median(want_lse[seen])) > 70.0 and np.abs(lse.cpu().numpy() - want_lse)[seen].max() <= 0.25


def _heads_of_one_block(H, N, seed, shift=0.0):
    q, k, v = _qkv(H, N, seed, shift)
    mask = np.ones((H, 1, 1), bool)
    mask[::7] = False
    return q, k, v, mask


@pytest.mark.parametrize("H,N", [(1024, 64), (1030, 37), (1500, 1)])
def test_two_waves_to_a_block(B, H, N):
    """1024 heads of a single block and more, which has no neighbour: a workgroup of two waves each; the block kept or not."""
    q, k, v, mask = _heads_of_one_block(H, N, N)
    out, lse = _run(B, q, k, v, mask, N)
    _check(out, lse, q, k, v, mask, N, heads=None)
    again, _ = _run(B, q, k, v, mask, N)
    assert torch.equal(out, again)


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("N", [64, 37])
def test_two_waves_out_of_range(B, sign, N):
    """As test_rows_out_of_range, for two waves to a block."""
    q, k, v, mask = _heads_of_one_block(1024, N, 14, 27.0 * sign)
    out, lse = _run(B, q, k, v, mask, N)
    kept = mask[:, 0, 0]
    assert (out[torch.from_numpy(~kept)].float() == 0).all() and torch.isneginf(lse[torch.from_numpy(~kept)]).all()
    want, want_lse = O.sparse_attention(q, k, v, np.ones_like(mask), 64, return_lse=True)
    want[~kept] = np.nan
    mx, mean = attn_errors(out, want)
    assert mx <= 5e-2 and mean <= 5e-3, (mx, mean)
    assert abs(np.median(want_lse)) > 70.0 and np.abs(lse.cpu().numpy() - want_lse)[kept].max() <= 0.25


@pytest.mark.parametrize("n_first", [4097 * 64 - 20, 700])
def test_more_key_blocks_than_pairs_take(B, n_first):
    """4097 key blocks and more: two waves to a block again, with lse, empty rows, a ragged and a split sequence."""
    N = 4097 * 64 - 20
    nb = len(O.block_ranges(N, 64, n_first))
    assert nb > 4096
    q, k, v = _qkv(1, N, 5)
    rng = np.random.default_rng(2)
    mask = rng.random((1, nb, nb)) < 0.002
    mask[0, [0, 10]] = rng.random((2, nb)) < 0.3
    mask[0, :, 0] = mask[0, :, nb - 1] = True
    mask[0, 7] = False
    out, lse = _run(B, q, k, v, mask, n_first)
    blocks = [0, 1, 10, nb - 2, nb - 1]
    want, want_lse = O.sparse_attention(q, k, v, np.where(mask.any(-1, keepdims=True), mask, True), 64, q_blocks=blocks,
                                        n_first=n_first, return_lse=True)
    assert bf16_bars_ok(out, want)[0], bf16_bars_ok(out, want)
    seen = ~np.isnan(want_lse)
    assert np.abs(lse.cpu().numpy() - want_lse)[seen].max() <= 2e-2
    lo, hi = O.block_ranges(N, 64, n_first)[7]
    assert (out[0, lo:hi].float() == 0).all() and torch.isneginf(lse[0, lo:hi]).all()

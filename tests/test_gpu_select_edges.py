"""Block selection (Sec. 4.1) at the sizes where its kernels change: 16-row and 16-column product tiles,
64 blocks per register slot, the 512 key blocks up to which scores and selection share one kernel, each
register-tile size, and searches that end with more than 64, 64 and fewer candidates.  Everything is
compared with the oracle; the input is scaled so that rows keep from one block to nearly all."""
import numpy as np
import pytest
import torch

from oracle import bsga_oracle as O
from tests.helpers import bits_to_mask, lists_to_mask, unexcused_mask_mismatches

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (17, 2), (16, 15), (33, 16), (15, 17), (5, 63), (16, 64), (31, 65), (2, 255), (48, 256), (7, 257),
         (3, 511), (16, 512), (33, 513), (4, 769), (32, 1281), (3, 1793), (2, 2561), (3, 3329), (2, 4097), (1, 8192)]


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


def _check(B, qp, kp, tau, rho, scale, fq=None, fk=None):
    dev = [None if f is None else torch.from_numpy(f).cuda() for f in (fq, fk)]
    bits, idx, cnt = B.bsga_select_blocks(torch.from_numpy(qp).cuda(), torch.from_numpy(kp).cuda(), tau, rho,
                                          score_scale=scale, force_q=dev[0], force_k=dev[1])
    torch.cuda.synchronize()
    nbk = kp.shape[1]
    got = bits_to_mask(bits, nbk)
    assert (got == lists_to_mask(idx, cnt, nbk)).all()
    logits = O.block_logits(qp, kp, scale)
    if fk is not None and (fk == 2).any():
        want = O.select_blocks_unranked_columns(logits, tau, rho, fk == 2)
        want |= (fk == 1)[None, None, :]
        if fq is not None:
            want[:, fq.astype(bool), :] = True
        assert (got == want).all()
        return got
    probs = O.block_softmax(logits)
    want = O.select_blocks(probs, tau, rho, fq, fk)
    unexcused, excused = unexcused_mask_mismatches(got, want, logits, probs, tau, rho)
    assert unexcused == 0, (unexcused, excused)
    return got


@pytest.mark.parametrize("nbq,nbk", SIZES)
@pytest.mark.parametrize("tau,rho,spread", [(0.9, 1.0, 0.05), (0.5, 0.75, 3.0), (0.0, 0.6, 1.0), (0.999, 0.9, 0.3)])
def test_sizes_where_the_kernels_change(B, nbq, nbk, tau, rho, spread):
    rng = np.random.default_rng(nbq * 10007 + nbk)
    qp = rng.standard_normal((2, nbq, 64)) * spread
    kp = rng.standard_normal((2, nbk, 64))
    _check(B, qp, kp, tau, rho, 0.125)


@pytest.mark.parametrize("nbk", [100, 512, 600, 1500])
def test_ties_larger_than_a_wave(B, nbk):
    """More equal blocks than lanes: the window cannot shrink below them, and the cut lies inside the ties."""
    rng = np.random.default_rng(nbk)
    qp = rng.standard_normal((1, 5, 64))
    kp = np.repeat(rng.standard_normal((1, 3, 64)), (nbk + 2) // 3, axis=1)[:, rng.permutation(nbk)]
    for tau, rho in ((0.5, 1.0), (0.97, 1.0), (0.0, 0.7), (0.3, 0.2)):
        _check(B, qp, kp, tau, rho, 0.125)


@pytest.mark.parametrize("nbk", [130, 700, 1300, 2500, 5000, 8192])
def test_unranked_and_forced_columns(B, nbk):
    rng = np.random.default_rng(nbk)
    qp = rng.standard_normal((2, 20, 64))
    kp = rng.standard_normal((2, nbk, 64))
    fk = np.zeros(nbk, np.uint8)
    fk[[0, 5, nbk - 1]] = 2
    fk[7] = 1
    fq = np.zeros(20, np.uint8)
    fq[19] = 1
    for tau, rho in ((0.9, 1.0), (0.0, 0.8), (1.0, 1.0)):
        _check(B, qp, kp, tau, rho, 0.125, fq, fk)


@pytest.mark.parametrize("nbk", [64, 600])
def test_rows_that_keep_everything(B, nbk):
    """tau at and next to 1, a row of equal scores, and rows whose scores are NaN or infinite."""
    qp = np.zeros((1, 4, 64))
    qp[0, 1, 0], qp[0, 2, 0], qp[0, 3, 0] = 200.0, np.nan, np.inf
    kp = np.zeros((1, nbk, 64))
    kp[0, :, 0] = np.linspace(-1, 1, nbk)
    for tau in (1.0, 2.0):
        bits, idx, cnt = B.bsga_select_blocks(torch.from_numpy(qp).cuda(), torch.from_numpy(kp).cuda(), tau)
        assert (cnt.cpu().numpy() == nbk).all() and bits_to_mask(bits, nbk).all()
    bits, idx, cnt = B.bsga_select_blocks(torch.from_numpy(qp).cuda(), torch.from_numpy(kp).cuda(), 0.9)
    c = cnt.cpu().numpy()[0]
    assert c[2] == nbk and c[3] == nbk               # the mass never gets to tau
    assert c[0] == int(np.ceil(0.9 * nbk - 1e-9))    # equal scores: the shortest prefix
    assert c[1] < nbk


@pytest.mark.parametrize("nbk", [200, 500, 700, 2400, 5000])
@pytest.mark.parametrize("low", [-690.0, -725.0, -743.0])
def test_ranking_of_probabilities_near_zero(B, nbk, low):
    """One block takes the mass and a top-k floor ranks the others, whose probabilities lie around the smallest
    normal and among the subnormal values: the ranking there is that of e / z as it is rounded to float64."""
    rng = np.random.default_rng(nbk)
    logits = rng.uniform(low, low + 25.0, (1, 6, nbk))
    logits[..., nbk // 3:nbk // 3 + 5] = rng.uniform(-2.0, 0.0, (1, 6, 5))
    qp = np.zeros((1, 6, 64))
    qp[0, :, :6] = np.eye(6)
    kp = np.zeros((1, nbk, 64))
    kp[0, :, :6] = logits[0].T          # products with 1 and 0: the scores are these values themselves
    for rho in (0.25, 0.5, 0.8):
        _check(B, qp, kp, 0.0, rho, 1.0)


@pytest.mark.parametrize("H,nbq,nbk", [(1, 1, 513), (3, 64, 600), (1, 65, 640), (2, 193, 641), (5, 513, 513), (6, 500, 700), (7, 513, 513)])
def test_score_tiles(B, H, nbq, nbk):
    """Rows and columns around the tiles of the score kernel's two widths (16 and 48 query rows to a wave), and launches on
    either side of the line between them."""
    rng = np.random.default_rng(nbq)
    qp = rng.standard_normal((H, nbq, 64)) * 0.3
    kp = rng.standard_normal((H, nbk, 64))
    _check(B, qp, kp, 0.9, 0.8, 0.125)

"""bf16 attention launches of few long query-block rows, whose rows are shared between workgroups by
key tiles: the parts of a row are summed by the last workgroup to finish.  Compared with the oracle and
with the launch without a workspace (one workgroup per row); rows shorter than a part and longer than many parts, empty rows, ragged and split sequences, both block
sizes and half-size key blocks, and rows whose logits need the second, online-softmax pass."""
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


def _qkv(H, N, seed, shift=0.0):
    rng = np.random.default_rng(seed)
    q, k, v = (rng.standard_normal((H, N, 64)).astype(np.float32) for _ in range(3))
    q += abs(shift) / 8.0
    k += shift / 8.0
    return [bf16_bits_to_f32(round_to_bf16_bits(x)) for x in (q, k, v)]


def _lists(mask):
    idx, cnt = O.mask_to_index_lists(mask)
    return torch.from_numpy(np.where(idx < 0, 0, idx)).cuda(), torch.from_numpy(cnt).cuda()


CASES = [  # heads, tokens, n_first, block, key block, density
    (1, 16330, 16330, 64, 64, 1.0), (1, 16400, 16400, 64, 64, 0.01), (1, 17000, 16900, 64, 64, 0.3), (1, 25000, 25000, 64, 64, 0.1),
    (1, 43968, 43968, 128, 128, 0.9), (1, 43000, 700, 128, 64, 0.5), (2, 33000, 33000, 128, 128, 0.2),
    (5, 25000, 25000, 128, 128, 0.1), (4, 32600, 32500, 128, 64, 0.05),
]


@pytest.mark.parametrize("H,N,n_first,b,bk,density", CASES)
def test_shared_rows(B, H, N, n_first, b, bk, density):
    rng = np.random.default_rng(N + b)
    q, k, v = _qkv(H, N, N)
    nbq, nbk = len(O.block_ranges(N, b, n_first)), len(O.block_ranges(N, bk, n_first))
    assert H * nbq < 1024
    mask = rng.random((H, nbq, nbk)) < density
    mask[:, np.arange(nbq), rng.integers(0, nbk, nbq)] = True
    mask[0, nbq // 2] = True                       # a row that keeps everything
    empty = nbq // 3
    mask[0, empty] = False                         # and one that keeps nothing
    idx, cnt = _lists(mask)
    tq, tk, tv = (to_device(x, "bf16") for x in (q, k, v))
    ranges = O.block_ranges(N, b, n_first)
    outs = [B.bsga_sparse_attn_split(tq, tk, tv, b, n_first, idx, cnt, return_lse=True, block_k=bk) for _ in range(3)]
    small = torch.empty((H * (-(-N // 64) + 33) + 4) * 4, dtype=torch.uint8, device="cuda")  # the launch order alone
    plain, plse = B.bsga_sparse_attn_split(tq, tk, tv, b, n_first, idx, cnt, return_lse=True, block_k=bk, workspace=small)
    torch.cuda.synchronize()
    out, lse = outs[0]
    for o, s in outs[1:]:                          # whoever finishes last, the parts are summed in one order
        assert torch.equal(o, out) and torch.equal(s, lse)
    lo, hi = ranges[empty]
    assert (out[0, lo:hi].float() == 0).all() and torch.isneginf(lse[0, lo:hi]).all()
    finite = torch.isfinite(plse)
    # row sums are taken over bf16 weights in a part's leading full tiles and over fp32 weights from its first
    # ragged tile on, and a part starts afresh: the two sums differ by less than one rounding, 2^-9
    assert torch.equal(finite, torch.isfinite(lse)) and (lse - plse)[finite].abs().max() <= 2.0 ** -9
    # the same products over row sums that far apart, then each rounded to bf16 (2^-9 of it): under 2^-7
    a, c = out.float(), plain.float()
    assert ((a - c).abs() <= 2.0 ** -7 * torch.maximum(a.abs(), c.abs()) + 1e-6).all()
    blocks = sorted({0, nbq // 2, nbq - 1, int(rng.integers(0, nbq))} - {empty})
    want = O.sparse_attention(q, k, v, np.where(mask.any(-1, keepdims=True), mask, True), b, q_blocks=blocks, heads=[0, H - 1],
                              b_k=bk, n_first=n_first)
    assert bf16_bars_ok(out, want)[0], bf16_bars_ok(out, want)


@pytest.mark.parametrize("H,N", [(1, 20600), (2, 21999)])
def test_dense_equals_every_block_listed(B, H, N):
    q, k, v = _qkv(H, N, 9)
    tq, tk, tv = (to_device(x, "bf16") for x in (q, k, v))
    nb = O.num_blocks(N, 128)
    dense = B.bsga_dense_attn(tq, tk, tv)
    a, c = dense.float(), B.bsga_sparse_attn(tq, tk, tv, 128, *_lists(np.ones((H, nb, nb), bool))).float()
    assert ((a - c).abs() <= 2.0 ** -7 * torch.maximum(a.abs(), c.abs()) + 1e-6).all()  # not shared: another order of sums
    want = O.sparse_attention(q, k, v, np.ones((H, nb, nb), bool), 128, q_blocks=[0, nb - 1])
    assert bf16_bars_ok(dense, want)[0]


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("b,bk", [(128, 128), (64, 64), (128, 64)])
def test_rows_out_of_range_are_repeated_whole(B, sign, b, bk):
    """Logits near +-91 nats overflow or vanish in the pass without a reference maximum; only the workgroup that
    sums the parts can tell, and it repeats the whole row.  Bars as for the launch of one workgroup per row."""
    H, N = (1, 16400) if b == 64 else (1, 41000)
    q, k, v = _qkv(H, N, 11, 27.0 * sign)
    nbq, nbk = O.num_blocks(N, b), O.num_blocks(N, bk)
    mask = np.random.default_rng(3).random((H, nbq, nbk)) < 0.6
    mask[:, :, 0] = True
    idx, cnt = _lists(mask)
    out, lse = B.bsga_sparse_attn(*(to_device(x, "bf16") for x in (q, k, v)), b, idx, cnt, return_lse=True, block_k=bk)
    torch.cuda.synchronize()
    blocks = [0, 1, nbq // 2, nbq - 1]
    want, want_lse = O.sparse_attention(q, k, v, mask, b, return_lse=True, b_k=bk, q_blocks=blocks)
    seen = ~np.isnan(want_lse)
    assert abs(np.median(want_lse[seen])) > 70.0  # past 2^100 = e^69 and 2^-80 = e^-55
    mx, mean = attn_errors(out, want)
    assert mx <= 5e-2 and mean <= 5e-3, (mx, mean)
    assert np.abs(lse.cpu().numpy() - want_lse)[seen].max() <= 0.25


def test_replays_from_a_graph(B):
    H, N, b = 1, 16500, 64
    nb = O.num_blocks(N, b)
    rng = np.random.default_rng(4)
    idx, cnt = _lists((rng.random((H, nb, nb)) < 0.4) | np.eye(nb, dtype=bool))
    data = [[to_device(x, "bf16") for x in _qkv(H, N, s)] for s in (1, 2)]
    q, k, v = (x.clone() for x in data[0])
    ws = torch.empty(B.bsga_attn_workspace_bytes(q.dtype, H, N), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(q)
    want = [B.bsga_sparse_attn(*d, b, idx, cnt) for d in data]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.bsga_sparse_attn(q, k, v, b, idx, cnt, out=out, workspace=ws)
    for which in (0, 1, 1, 0):
        for dst, src in zip((q, k, v), data[which]):
            dst.copy_(src)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[which])
        B.bsga_dense_attn(q, k, v)


def _plan(ws, H, N):
    """The plan of the last launch: tiles to a piece (0: whole rows), number of pieces, parts counted in per row."""
    order = (H * (-(-N // 64) + 33) + 4) * 4
    at = (ws.data_ptr() + order + 255) // 256 * 256 - ws.data_ptr()
    words = ws[at:at + (16 + 3 * 1024) * 4].view(torch.int32).cpu().numpy()
    return words[0], words[1], words[16 + 2048:]


@pytest.mark.parametrize("H,N,n_first,b,bk,density", CASES + [(1, 16400, 16400, 64, 64, 0.6), (1, 41000, 41000, 128, 128, 0.6), (1, 41000, 41000, 128, 64, 0.6)])
def test_rows_of_these_cases_are_shared(B, H, N, n_first, b, bk, density):
    """The launches of this file do take the way that it is about."""
    nbq, nbk = len(O.block_ranges(N, b, n_first)), len(O.block_ranges(N, bk, n_first))
    mask = np.random.default_rng(N + b).random((H, nbq, nbk)) < density
    mask[:, :, 0] = True
    mask[0, nbq // 2] = True
    ws = torch.full((B.bsga_attn_workspace_bytes(torch.bfloat16, H, N),), 255, dtype=torch.uint8, device="cuda")
    q, k, v = (torch.randn((H, N, 64), device="cuda").bfloat16() for _ in range(3))
    B.bsga_sparse_attn_split(q, k, v, b, n_first, *_lists(mask), block_k=bk, workspace=ws)
    torch.cuda.synchronize()
    quota, used, arrived = _plan(ws, H, N)
    assert quota >= 4 and used > 0 and (arrived[:H * nbq] > 1).any()


@pytest.mark.parametrize("H,N", [(1, 20600), (2, 21999)])
def test_dense_rows_are_shared(B, H, N):
    ws = torch.full((B.bsga_attn_workspace_bytes(torch.bfloat16, H, N),), 255, dtype=torch.uint8, device="cuda")
    q, k, v = (torch.randn((H, N, 64), device="cuda").bfloat16() for _ in range(3))
    B.bsga_dense_attn(q, k, v, workspace=ws)
    torch.cuda.synchronize()
    quota, used, arrived = _plan(ws, H, N)
    assert quota >= 4 and used > 0 and (arrived[:H * O.num_blocks(N, 128)] > 1).any()


@pytest.mark.parametrize("H,N,bk,kept", [(1, 43900, 128, 20), (2, 43968, 128, 34), (5, 25000, 128, 90), (2, 43968, 64, 61)])
def test_lists_of_one_length_stay_whole(B, H, N, bk, kept):
    """Short lists of one length gain nothing by being shared: the plan leaves them whole, fewer and more than the
    512 workgroups of the first round, and every row is what the launch without a plan makes of it."""
    b = 128
    nb, nbk = O.num_blocks(N, b), O.num_blocks(N, bk)
    g = torch.Generator(device="cuda").manual_seed(N)
    idx = torch.rand((H, nb, nbk), generator=g, device="cuda").argsort(-1)[..., :kept].sort(-1).values
    idx = torch.nn.functional.pad(idx, (0, nbk - kept)).int().contiguous()
    cnt = torch.full((H, nb), kept, dtype=torch.int32, device="cuda")
    cnt[0, 1], cnt[H - 1, nb - 1] = 0, kept - 1
    q, k, v = (torch.randn((H, N, 64), generator=g, device="cuda").bfloat16() for _ in range(3))
    ws = torch.full((B.bsga_attn_workspace_bytes(q.dtype, H, N),), 255, dtype=torch.uint8, device="cuda")
    out = torch.full_like(q, float("nan"))
    _, lse = B.bsga_sparse_attn(q, k, v, b, idx, cnt, return_lse=True, out=out, workspace=ws, block_k=bk)
    plain, plse = B.bsga_sparse_attn(q, k, v, b, idx, cnt, return_lse=True, ordered=False, block_k=bk)
    torch.cuda.synchronize()
    assert _plan(ws, H, N)[0] == 0
    assert torch.equal(out, plain) and torch.equal(lse, plse)
    assert (out[0, b:2 * b].float() == 0).all()

"""fp32 attention with K and V split beforehand into the call's workspace: the same bits as without one, over block sizes, ragged
ends, split sequences and lists, and a workspace that it cannot use is ignored."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


def _inputs(H, N, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn((H, N, 64), generator=g, device="cuda") for _ in range(3)]


def _lists(H, nb, seed):
    """Lists of every length from one block on, in any order."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    idx = torch.rand((H, nb, nb), generator=g, device="cuda").argsort(2).int().contiguous()
    cnt = 1 + torch.randint(0, nb, (H, nb), generator=g, device="cuda", dtype=torch.int32)
    return idx, cnt


def _workspace(H, N):
    return torch.full((H * N * 768,), 255, dtype=torch.uint8, device="cuda")


# one token, one row past a tile, one short of it, whole blocks; n_first inside a block of the whole sequence
@pytest.mark.parametrize("H,N,n_first", [(129, 1, 1), (70, 65, 65), (65, 127, 100), (16, 640, 640), (16, 641, 577), (9, 1000, 1), (3, 2879, 2815)])
@pytest.mark.parametrize("block", [64, 128])
def test_same_bits_as_without(B, H, N, n_first, block):
    q, k, v = _inputs(H, N, N)
    idx, cnt = _lists(H, B.split_blocks(N, n_first, block), N)
    run = lambda ws: B.bsga_sparse_attn_split(q, k, v, block, n_first, idx, cnt, return_lse=True, workspace=ws)
    o, l = run(torch.empty(16, dtype=torch.uint8, device="cuda"))
    for ws in (_workspace(H, N), torch.cat([_workspace(H, N), _workspace(1, 1)])[8:]):  # the second is not aligned
        before = ws.clone()
        got_o, got_l = run(ws)
        assert torch.equal(got_o, o) and torch.equal(got_l, l)
        units = H * B.split_blocks(N, n_first, block) * (block // 64)
        assert torch.equal(ws, before) == (ws.data_ptr() % 16 != 0 or units <= 128)


@pytest.mark.parametrize("what", ["k inf", "v inf", "v nan"])
def test_values_that_are_not_finite(B, what):
    """In the last token of a ragged block and, in a split sequence, in the one after it."""
    H, N, n_first = 16, 900, 610
    for at in (n_first - 1, n_first, N - 1):
        q, k, v = _inputs(H, N, 3)
        {"k": k, "v": v}[what[0]][3, at, 5] = float(what[2:])
        nb = B.split_blocks(N, n_first, 64)
        idx, cnt = _lists(H, nb, 4)
        run = lambda ws: B.bsga_sparse_attn_split(q, k, v, 64, n_first, idx, cnt, workspace=ws)
        o = run(torch.empty(16, dtype=torch.uint8, device="cuda"))
        got = run(_workspace(H, N))
        # what is not finite is the same in both, sign and place
        assert torch.equal(got.isnan(), o.isnan()) and torch.equal(got.isposinf(), o.isposinf()) and torch.equal(got.isneginf(), o.isneginf())
        assert what == "k inf" or bool((~o.isfinite()).any())
        # rows that do not list the token's block but load the tokens after one that they do run on fp32 instructions: both ways
        # are as near to float64 as fp32 sums are
        finite = o.isfinite()
        assert finite.float().mean() > 0.9 and (got - o)[finite].abs().max() <= 1e-5 * max(1.0, float(o[finite].abs().max()))


def test_layer_and_graph(B):
    """The layer takes the room by itself, also under capture; each replay gives the eager bits."""
    H, N = 16, 2748
    assert B.bsga_attn_fp32_parts_bytes(H, N, 64, 0.9) == H * N * 768
    q, k, v = _inputs(H, N, 5)
    B.sparse_global_attention(q, k, v, 64, 0.9)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = B.sparse_global_attention(q, k, v, 64, 0.9)
    for seed in (6, 7, 8):
        for dst, src in zip((q, k, v), _inputs(H, N, seed)):
            dst.copy_(src)
        graph.replay()
        eager = B.sparse_global_attention(q, k, v, 64, 0.9)
        assert torch.equal(captured[0], eager[0]) and torch.equal(captured[3], eager[3])
        plain = B.bsga_sparse_attn(q, k, v, 64, eager[1], eager[2], ordered=False)
        assert torch.equal(eager[0], plain)

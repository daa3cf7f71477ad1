"""The layer's scratch: the logits of a long sequence are freed before the output is allocated, so that the peak is the
larger of the two and not their sum."""
import pytest
import torch

pytestmark = pytest.mark.gpu
MB = 1 << 20


@pytest.mark.parametrize("H,N,block", [(2, 100000, 128), (4, 21984, 64), (1, 1374, 64)])
def test_peak_memory_of_the_layer(H, N, block):
    import paper_2509_07120_amd as B
    q, k, v = (torch.randn((H, N, 64), device="cuda").bfloat16() for _ in range(3))
    nb = -(-N // block)
    B.sparse_global_attention(q, k, v, block, 0.0, 0.9)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    got = B.sparse_global_attention(q, k, v, block, 0.0, 0.9)
    torch.cuda.synchronize()
    results = sum(t.numel() * t.element_size() for t in got)
    out = got[0].numel() * got[0].element_size()
    pools = 2 * H * nb * 64 * 8
    logits = B.bsga_select_workspace_bytes(H, nb, nb)
    own = B.bsga_attn_workspace_bytes(q.dtype, H, N)
    # allocations are rounded up, at most 2 MB each above 1 MB
    assert torch.cuda.max_memory_allocated() - before <= results - out + pools + max(logits, out + own) + 8 * MB

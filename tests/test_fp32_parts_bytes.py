"""When an fp32 attention call asks for room for its split operands: the lines of the rule, and arguments that are refused."""
import pytest


@pytest.fixture(scope="module")
def B():
    import paper_2509_07120_amd as pkg
    return pkg


@pytest.mark.parametrize("heads,n_tokens,kept,asks", [
    (16, 512, 1.0, False),       # 128 rows: these go to the kernel that does not split
    (16, 2049, 1.0, True),       # 33 tiles to each of 528 rows
    (16, 2049, 0.36, False),     # 11.9 of them expected
    (16, 2049, 0.37, True),
    (8, 4096, 0.39, False),      # 512 rows: 25 tiles
    (8, 4096, 0.4, True),
    (16, 21845, 1.0, True),      # 256 MB
    (16, 21846, 1.0, False),
    (16, 2748, 0.0, False), (16, 2748, float("nan"), False),
])
def test_lines(B, heads, n_tokens, kept, asks):
    assert B.bsga_attn_fp32_parts_bytes(heads, n_tokens, 64, kept) == (heads * n_tokens * 768 if asks else 0)


@pytest.mark.parametrize("heads,n_tokens,dim", [(0, 4096, 64), (-1, 4096, 64), (65536, 4096, 64), (16, 0, 64), (16, -5, 64), (16, (1 << 24) + 1, 64), (16, 4096, 128)])
def test_invalid_arguments_ask_for_nothing(B, heads, n_tokens, dim):
    assert B.bsga_attn_fp32_parts_bytes(heads, n_tokens, dim, 1.0) == 0

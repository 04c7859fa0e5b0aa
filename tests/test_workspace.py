"""Workspace sizes, on the CPU: what the kernels write and nothing else."""
import pytest

from paper_2604_16590_amd import _binding as B
from paper_2604_16590_amd import serve


def up(n):
    return -(-n // 256) * 256


@pytest.mark.parametrize("H,d", [(1, 64), (5, 64), (1, 128), (8, 128)])
def test_fp32_rows_need_no_operand_images(H, d):
    # fp32 at d = 64 and 128: partial sums, FP64 sums and (backward) 8 bytes a
    # query token; N of one partial for every max_fp32_run tokens
    N = 1 << 20
    desc = serve.desc_for(1, H, N, d, B.LA_FP32)
    partials = up(H * (N // 4096) * (d * d + d) * 4)
    sums = up(H * d * d * 8) + up(H * d * 8)
    assert B.workspace_size(desc, 0) == partials + sums
    assert B.workspace_size(desc, 1) == partials + sums + up(H * N * 8)

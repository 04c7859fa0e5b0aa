"""The server's budget at the sizes it has always accepted, on the CPU (fake
executor): a member's kept S and z and the workspace of a partial for 2,048
(d = 128) or 512 tokens a head."""
import pytest

from paper_2604_16590_amd import _binding as B
from paper_2604_16590_amd import serve

SHAPES = [(1, 4096, 128, B.LA_FP32), (8, 4096, 128, B.LA_FP32), (1, 1000, 64, B.LA_BF16), (8, 1000, 64, B.LA_BF16),
          (8, 4096, 16, B.LA_BF16)]


def up(n):
    return -(-n // 256) * 256


def sizes(H, N, d, dtype):
    """Kept bytes and least workspace of one member."""
    partials = -(-N // (2048 if d == 128 else 512))
    keep = up(H * d * d * 8) + up(H * d * 8)
    images = B.workspace_size(serve.desc_for(1, H, N, d, dtype), 2)
    return keep, up(H * partials * (d * d + d) * 4) + keep + images


@pytest.mark.parametrize("H,N,d,dtype", SHAPES)
def test_a_member_of_the_least_size_is_accepted(H, N, d, dtype):
    keep, least = sizes(H, N, d, dtype)
    desc = serve.desc_for(1, H, N, d, dtype)
    assert least < B.workspace_size(desc, 0)
    with serve.Server(keep + least, fake_slice_ns=1000) as srv:
        assert srv.wait(srv.submit(desc), timeout_s=10).state == serve.DONE
        c = srv.stats()
        assert c.peak_bytes_in_use <= c.budget_bytes
    with serve.Server(keep + least - 256, fake_slice_ns=1000) as srv:
        with pytest.raises(B.LaError) as e:
            srv.submit(desc)
        assert e.value.status == 3  # LA_ERR_OOM


def test_a_member_runs_beside_kept_summaries():
    H, N, d, dtype = 8, 4096, 128, B.LA_FP32
    keep, least = sizes(H, N, d, dtype)
    one_head = B.workspace_size(serve.desc_for(1, 1, N, d, dtype), 0)
    with serve.Server(2 * keep + max(least, one_head), fake_slice_ns=1000) as srv:
        ids = [srv.submit(serve.desc_for(1, H, N, d, dtype)) for _ in range(2)]
        assert [srv.wait(i, timeout_s=10).state for i in ids] == [serve.DONE] * 2

"""How walk calls are planned, read out of the workspace that they ask for: host logic, no device call."""
import pytest

from paper_2403_09347_amd import binding as B


def workspace(p, rows, k_offs=None, flags=0):
    chunks = (B.BurstChunk * len(rows))()
    at = 0
    for i, c in enumerate(chunks):
        c.K, c.V, c.Nc = 4096, 8192, rows[i]        # (addresses that nothing reads)
        c.k_off = at if k_offs is None else k_offs[i]
        at += rows[i]
    return B.burst_walk_workspace_bytes(chunks, p, flags)


@pytest.mark.parametrize("H,N,ranges", [(16, 900, 2), (16, 1024, 2), (8, 2040, 4),             # 128 blocks of 128 rows
                                        (17, 1024, 1), (18, 900, 1), (20, 1000, 1),           # 136, 144, 160: two short ranges do not pay
                                        (16, 1216, 3), (15, 1130, 3), (14, 1400, 3),          # 160, 135, 154: three do
                                        (24, 1000, 1), (32, 777, 1), (16, 1500, 2)])          # 192, 224, 192
def test_key_ranges_of_the_padded_kernels(H, N, ranges):
    for d in (40, 96, 120):
        p = B.params(1, H, N, 0, d, "bf16", 0.1, causal=True)
        want = 0 if ranges == 1 else ranges * H * N * (d + 2) * 4
        assert workspace(p, [N], flags=B.BURST_WALK_NO_STATE) == want

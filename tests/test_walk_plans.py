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


@pytest.mark.parametrize("H,N,ranges", [(16, 900, 2), (16, 1024, 2), (8, 2040, 4),             # 128 blocks of 128 rows: 256 or 512 workgroups
                                        (17, 1024, 1), (18, 900, 1), (20, 1000, 1), (12, 1200, 2),   # not 272, 288, 320 or 360
                                        (1, 3840, 8), (2, 2816, 5), (8, 1536, 4),             # not 300 or 308, but 384
                                        (16, 1216, 3), (15, 1130, 3), (14, 1400, 3),          # 480, 405, 462
                                        (24, 1000, 1), (32, 777, 1), (16, 1500, 2)])          # more than 160 blocks
def test_key_ranges_of_the_padded_kernels(H, N, ranges):
    for d in (40, 96, 120):
        p = B.params(1, H, N, 0, d, "bf16", 0.1, causal=True)
        want = 0 if ranges == 1 else ranges * H * N * (d + 2) * 4
        assert workspace(p, [N], flags=B.BURST_WALK_NO_STATE) == want


@pytest.mark.parametrize("H,N,K,ranges", [(8, 958, 2268, 4), (8, 1500, 1500, 2), (130, 100, 1200, 3), (60, 128, 3000, 7)])   # 384, 384, 390, 420 workgroups
def test_key_ranges_of_walks_of_equal_length(H, N, K, ranges):
    assert workspace(B.params(1, H, N, 0, 40, "bf16", 0.1), [K], flags=B.BURST_WALK_NO_STATE) == ranges * H * N * 42 * 4


def test_fp32_walks_that_are_split():
    state = lambda s, H, N, d: 0 if s == 1 else s * H * N * (d + 2) * 4
    for H, N, K, d, s in ((8, 277, [277], 24, 1), (8, 384, [384], 36, 1), (8, 385, [385], 36, 2), (16, 256, [600], 36, 2), (8, 128, [1120], 32, 1),
                          (8, 128, [1121], 32, 8), (1, 256, [256] * 4, 32, 1), (4, 410, [410] * 4, 32, 4), (1, 128, [128] * 3, 64, 1), (1, 160, [160] * 4, 64, 5),
                          (8, 277, [277], 68, 2), (8, 700, [1400], 64, 1)):
        p = B.params(1, H, N, 0, d, "f32", 0.1)
        assert workspace(p, K, flags=B.BURST_WALK_FORWARD) == state(s, H, N, d)
    dkv = lambda H, N, K, d: form(H, N, [K], True, d=d, dtype="f32")
    assert dkv(8, 277, 277, 24) == 0 and dkv(8, 300, 300, 36) == 0 and dkv(8, 384, 384, 36) == 1 and dkv(8, 500, 500, 32) == 0 and dkv(2, 1000, 300, 24) == 1 \
        and dkv(8, 277, 277, 68) == 1


def test_partial_gradients_take_room_for_visible_keys_only():
    gradients = lambda keys, d: 2 * keys * d * 4
    # one head, 8192 rows, window of 4096 over 16 chunks of 4096: at most 8 parts of the two chunks (the first rows' window is empty
    # before key 0) that rows see
    p = B.params(1, 1, 8192, 0, 128, "bf16", 0.1, causal=True, window=4096)
    assert 0 < workspace(p, [4096] * 16) <= 8 * gradients(2 * 4096, 128)
    # 8 heads, 1024 rows that see the first of 16 chunks
    p = B.params(1, 8, 1024, 0, 64, "bf16", 0.1, causal=True)
    assert 0 < workspace(p, [1024] * 16) <= 4 * gradients(8 * 1024, 64) and workspace(p, [1024] * 16) == workspace(p, [1024])
    # hidden keys of the only chunk: 1024 rows and a window of 1000 see 2023 keys, 17 blocks of 128
    p = B.params(1, 1, 1024, 0, 64, "bf16", 0.1, causal=True, q_off=60000, window=1000)
    assert 0 < workspace(p, [65536]) <= 4 * gradients(17 * 128, 64)


def test_forward_walks_ask_for_no_partial_gradients():
    p = B.params(1, 32, 3008, 0, 128, "bf16", 0.1, causal=True, kv_heads=8)
    assert workspace(p, [3008]) > 0 and workspace(p, [3008], flags=B.BURST_WALK_FORWARD) == 0
    p = B.params(1, 1, 256, 0, 64, "f32", 0.1)                                               # split by keys: the states of the ranges
    assert workspace(p, [256] * 4, flags=B.BURST_WALK_FORWARD) == 8 * 256 * 66 * 4 <= workspace(p, [256] * 4)


def form(H, Nq, rows, workspace, d=128, dtype="bf16", **kw):
    p = B.params(1, H, Nq, 0, d, dtype, 0.1, **kw)
    chunks = (B.BurstChunk * len(rows))()
    for i, c in enumerate(chunks):
        c.K, c.V, c.Nc, c.k_off = 4096, 8192, rows[i], sum(rows[:i])
    return B.burst_walk_dkv_form(chunks, p, workspace)


def test_forms_of_dkv_launches():
    for ws in (False, True):
        assert form(32, 512, [512] * 16, ws, causal=True, q_off=15 * 512) == 2              # many short walks
        assert form(32, 4096, [4096] * 8, ws) == 0                                          # 64 tiles each: long ones
        assert form(32, 2048, [2048], ws, causal=True) == 2 and form(32, 3000, [3000], ws, causal=True) == 0   # equal shares or not
        assert form(257, 64, [128], ws) == 0 and form(8, 512, [512], ws) == 0               # one whole tile; few workgroups
        assert form(32, 512, [512] * 16, ws, q_strides=(512 * 4096, 128, 4096)) == 0        # rows of Q and K at different distances
    assert form(32, 3008, [3008], True, causal=True, kv_heads=8) == 1 and form(32, 3008, [3008], False, causal=True, kv_heads=8) == 0
    # cut where the longest walk is far above a CU's share, in tiles of 32 rows: 13 at d = 64, 21; 0, 14 on padded kernels
    cut = lambda H, N, d, rows=0, **kw: form(H, N, rows or [N], True, d=d, **kw)
    assert cut(32, 1226, 64, causal=True) == 0 and cut(16, 919, 64, causal=True) == 1
    assert cut(32, 1024, 96) == 0 and cut(32, 777, 96, causal=True) == 1
    assert cut(1, 4736, 128, [4736] * 4, causal=True, q_off=3 * 4736) == 0 and cut(2, 2609, 128, causal=True) == 1   # 148 x 2 workgroups: two rounds
    assert form(32, 0, [512], True) == 0 and form(32, 512, [0], True) == 0
    with pytest.raises(B.BurstError):
        form(32, 512, [512], True, kv_heads=5)


def test_without_the_forward_flag_the_size_is_enough_for_both_calls():
    """The forward and the dQ launches of a walk may be split differently (gradients in the inputs' type, no state)."""
    one = [(8, 2048, 128), (8, 2050, 128), (8, 2048, 64), (8, 1000, 96), (16, 1000, 128), (12, 1700, 64), (4, 2048, 80), (40, 300, 128)]
    for H, N, d in one:
        for causal in (False, True):
            p = B.params(1, H, N, 0, d, "bf16", 0.1, causal=causal)
            for rows in ([N], [N, N], [4 * N]):
                state, no_state = (workspace(p, rows, flags=f | B.BURST_WALK_FORWARD) for f in (0, B.BURST_WALK_NO_STATE))
                assert workspace(p, rows, flags=0) >= state and workspace(p, rows, flags=B.BURST_WALK_HALF_GRADS) >= state
                assert workspace(p, rows, flags=B.BURST_WALK_NO_STATE) >= no_state
                assert workspace(p, rows, flags=B.BURST_WALK_NO_STATE | B.BURST_WALK_HALF_GRADS) >= no_state
    p = B.params(1, 8, 2048, 0, 128, "bf16", 0.1, causal=True)
    state = lambda s: s * 8 * 2048 * 130 * 4
    assert workspace(p, [2048], flags=B.BURST_WALK_FORWARD) == state(4) and workspace(p, [2048], flags=B.BURST_WALK_HALF_GRADS) == state(4)
    assert workspace(p, [2048], flags=B.BURST_WALK_FORWARD | B.BURST_WALK_NO_STATE) == state(2)


@pytest.mark.parametrize("H,N,d,causal,state,no_state", [
    (8, 2048, 64, True, 4, 4), (8, 2050, 64, True, 3, 3), (8, 1500, 64, True, 3, 0), (2, 2048, 64, True, 4, 4),     # 128, 136, 96, 32 blocks of 128 rows
    (16, 2048, 64, False, 2, 2), (20, 2048, 64, False, 0, 0),                                                       # 256 and 320
    (8, 2048, 128, True, 4, 2), (8, 2050, 128, True, 3, 0), (8, 2048, 128, False, 4, 2), (2, 2048, 128, True, 4, 4)])
def test_key_ranges_of_walks_without_a_state(H, N, d, causal, state, no_state):
    """One chunk: as many ranges as workgroups of 64 rows have places for, from 32 tiles on."""
    p = B.params(1, H, N, 0, d, "bf16", 0.1, causal=causal)
    size = lambda flags: workspace(p, [N], flags=flags | B.BURST_WALK_FORWARD) / (H * N * (d + 2) * 4)
    assert size(0) == state and size(B.BURST_WALK_NO_STATE) == no_state


def test_half_gradients_in_row_groups_ask_for_no_partial_ones():
    for H, N, d in ((32, 777, 96), (16, 900, 64)):
        p = B.params(1, H, N, 0, d, "bf16", 0.1, causal=True)
        assert workspace(p, [N]) > 0 and workspace(p, [N], flags=B.BURST_WALK_HALF_GRADS) == 0
        assert form(H, N, [N], True, d=d, causal=True) == 1                        # (with fp32 gradients)

"""dK / dV launches of many short walks, d = 128, which one workgroup per CU takes in turn: every head must get the bits it gets
in a call of a few heads (a workgroup per block of keys), and the oracle's values: ragged blocks, walks of one and two tiles,
hidden chunks and blocks, chunks of different length, each memory layout, each order in which blocks are taken (one causal chunk
in alternating direction, chunks of equal length from another one for each workgroup, one after the other), accumulation,
gradients in the inputs' type.  The plan is asked for, so that every case is one."""
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    dict(H=256, Nq=128, chunk_rows=[128] * 4, causal=True, q_off=384, window=200),   # hidden chunks, each workgroup from another one
    dict(H=256, Nq=1, chunk_rows=[100, 128]),                                # one tile each, walked as two
    dict(H=256, Nq=100, chunk_rows=[30, 129, 257], causal=True, q_off=300),  # unequal chunks, ragged blocks, one and two tiles
    dict(H=256, Nq=130, chunk_rows=[100, 30], causal=True, q_off=90),
    dict(H=256, Nq=250, chunk_rows=[250], causal=True),                      # one causal chunk: alternating direction
    dict(H=512, Nq=130, chunk_rows=[130], causal=True),                      # ... with a last walk of one tile
    dict(H=128, Nq=500, chunk_rows=[500], causal=True, layout="seq"),
    dict(H=256, Nq=130, chunk_rows=[100, 100], layout="packed"),
    dict(H=256, Nq=200, chunk_rows=[200, 130, 100], causal=True, q_off=200, window=150, layout="seq"),
]


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items() if k != "chunk_rows"))
def test_every_head_as_in_a_small_call(spec):
    case = workloads.make_case(B=1, d=128, dtype="bf16", seed=223, device=DEV, **spec)

    def walk_of(a, b, form):
        part = lambda ts: [t[:, a:b] for t in ts]
        walk = RingWalk(case["Q"][:, a:b], case["scale"], case["causal"], case["q_off"], case["window"])
        args = part(case["K"]), part(case["V"]), case["k_offs"]
        O, lse = walk.forward(*args)
        dO = case["dO"][:, a:b]
        dQ, dKs, dVs = walk.backward(*args, dO)
        half = walk.backward_in_dtype(*args, dO)
        p = walk._walk_params()
        assert all(B.burst_walk_dkv_form(B.chunk_array(*args, None, p), p, ws) == form for ws in (False, True))
        twice = [[t.clone() for t in ts] for ts in (dKs, dVs)]
        B.burst_walk_bwd(walk.Q, B.chunk_array(*args, None, p, *twice, torch.float32), walk.O, walk._like_q(dO), walk.lse, walk.D,
                         torch.empty_like(dQ), p, accumulate_dq=False, accumulate_dkv=True)
        torch.cuda.synchronize()
        return [O, lse, dQ, *dKs, *dVs, half[0], *half[1], *half[2], *twice[0], *twice[1]]

    H, n = spec["H"], len(spec["chunk_rows"])
    blocks = sum((r + 127) // 128 for r in spec["chunk_rows"])
    few = max(1, 248 // blocks)                     # at most 256 workgroups
    B.burst_set_kernel_family(1)                    # (the forward and dQ kernels would otherwise depend on the number of heads)
    try:
        whole = walk_of(0, H, 2)
        parts = [walk_of(a, min(a + few, H), 0) for a in range(0, H, few)]
    finally:
        B.burst_set_kernel_family(0)
    for i, t in enumerate(whole):
        assert torch.equal(t, torch.cat([p[i] for p in parts], dim=1)), i
    for t, once in zip(whole[4 + 4 * n:], whole[3:3 + 2 * n]):
        assert torch.equal(t, 2 * once)
    some = sorted({0, H // 2, H - 1})
    compare_all_heads(case, "bf16", *whole[:3], whole[3:3 + n], whole[3 + n:3 + 2 * n], heads=some)

"""Walk calls with a query slice of no rows (Nq = 0, which the C ABI allows) and chunks that have keys: no
workspace, empty outputs, dK = dV = 0 -- with and without a GPU, for the shapes of every kernel family."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = [("bf16", 128), ("bf16", 64), ("bf16", 96), ("bf16", 20), ("f32", 64)]

# In a process of its own: a division by zero in the library ends the process that called it.
HOST = """
import sys
sys.path.insert(0, {root!r})
from paper_2403_09347_amd import binding as B
chunks = (B.BurstChunk * 2)()
for c in chunks:
    c.K, c.V, c.Nc = 4096, 8192, 1024           # (addresses that nothing reads)
for family in (0, 1, 2):
    B.burst_set_kernel_family(family)
    for causal in (False, True):
        for flags in (0, B.BURST_WALK_HALF_GRADS, B.BURST_WALK_NO_STATE):
            p = B.params(1, 4, 0, 0, {d}, {dtype!r}, 0.125, causal=causal)
            assert B.burst_walk_workspace_bytes(chunks, p, flags) == 0
"""


@pytest.mark.parametrize("dtype,d", SHAPES)
def test_workspace_of_a_walk_without_query_rows(dtype, d):
    r = subprocess.run([sys.executable, "-c", HOST.format(root=ROOT, d=d, dtype=dtype)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d", SHAPES)
def test_walk_and_differentiable_call_without_query_rows(dtype, d):
    import torch
    from paper_2403_09347_amd import workloads
    from paper_2403_09347_amd.autograd import burst_attention
    from paper_2403_09347_amd.harness import RingWalk
    case = workloads.make_case(B=1, H=4, kv_heads=2, d=d, Nq=0, chunk_rows=[70, 33], dtype=dtype, seed=2, device="cuda:0", causal=True,
                               q_off=90)
    walk = RingWalk(case["Q"], case["scale"], True, 90, kv_heads=2)
    O, lse = walk.forward(case["K"], case["V"], case["k_offs"])
    assert O.shape == (1, 4, 0, d) and lse.shape == (1, 4, 0)
    nan = lambda ts: [torch.full(t.shape, float("nan"), device=t.device) for t in ts]
    dQ, dKs, dVs = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"], None, nan(case["K"]), nan(case["V"]))
    assert dQ.shape == O.shape and all(bool((g == 0).all()) for g in dKs + dVs)
    q, ks, vs = [case["Q"].requires_grad_(True)], [k.requires_grad_(True) for k in case["K"]], [v.requires_grad_(True) for v in case["V"]]
    O, lse = burst_attention(q[0], ks, vs, causal=True, q_off=90)
    grads = torch.autograd.grad(O, q + ks + vs, case["dO"])
    assert O.shape == (1, 4, 0, d) and all(g.shape == t.shape and bool((g == 0).all()) for g, t in zip(grads, q + ks + vs))

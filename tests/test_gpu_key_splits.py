"""Walks of few query rows whose keys are split into ranges (partial states merged at the end): one row, odd
counts, ranges that see nothing under a mask, head dimensions with and without padding, against the
oracle, and against the walk without a workspace (which cannot split) for O and lse."""
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    dict(B=1, H=2, d=128, Nq=1, chunk_rows=[1280]),
    dict(B=1, H=2, d=64, Nq=40, chunk_rows=[700, 1, 800], causal=True, q_off=1461),
    dict(B=2, H=3, d=80, Nq=129, chunk_rows=[513] * 3, causal=True, q_off=1400),
    dict(B=1, H=4, kv_heads=2, d=128, Nq=33, chunk_rows=[2100], causal=True, q_off=2067, layout="seq"),
    dict(B=1, H=2, d=24, Nq=70, chunk_rows=[4000], window=1500, q_off=2000),
    dict(B=1, H=1, d=128, Nq=128, chunk_rows=[64] * 20, causal=True, q_off=-50, k_offs=[60 * i for i in range(20)]),
]


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items() if k not in ("chunk_rows", "k_offs")))
def test_split_walks(spec):
    case = workloads.make_case(dtype="bf16", seed=103, device=DEV, **spec)
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], kv_heads=case.get("kv_heads", 0))
    p = walk._walk_params()
    chunks = B.chunk_array(case["K"], case["V"], case["k_offs"], None, p)
    if not case["causal"] or case["q_off"] > 0:
        assert B.burst_walk_workspace_bytes(chunks, p) > 0          # these sizes are split
    O, lse = walk.forward(case["K"], case["V"], case["k_offs"])
    O, lse = O.clone(), lse.clone()
    dQ, dKs, dVs = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"])
    twice, _, _ = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"], dQ=dQ.clone())
    torch.cuda.synchronize()
    compare_all_heads(case, "bf16", O, lse, dQ, dKs, dVs)
    assert torch.allclose(twice, 2 * dQ, rtol=1e-6, atol=1e-6)
    B.burst_walk_fwd(case["Q"], chunks, walk.O_acc, walk.m, walk.l, walk.O, walk.lse, p)
    torch.cuda.synchronize()
    seen = torch.isfinite(lse)
    assert torch.equal(seen, torch.isfinite(walk.lse))
    # another order of fp32 sums (2^-24 each), and an O next to a rounding boundary may round the other way (2^-8)
    assert float((lse - walk.lse)[seen].abs().max()) < 1e-5
    assert torch.allclose(O.float(), walk.O.float(), rtol=2 ** -7, atol=1e-3)

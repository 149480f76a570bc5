"""fp32 walks of more than 128 row blocks whose tiles are dealt to two workgroups a block (and the nearest ones that are not), against the
oracle and against the walk without a workspace, which cannot split."""
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("spec,ranges", [
    (dict(H=4, d=128, Nq=1400, chunk_rows=[1400, 1400], causal=True, q_off=1400), 2),
    (dict(H=6, kv_heads=3, d=68, Nq=1025, chunk_rows=[4000], causal=True, q_off=2975), 2),
    (dict(H=9, d=96, Nq=1000, chunk_rows=[1500, 1500]), 2),                                   # 288 equal blocks: a round and a bit
    (dict(H=8, d=128, Nq=700, chunk_rows=[700, 700], causal=True, q_off=700), 1),
    (dict(H=8, d=128, Nq=600, chunk_rows=[600]), 1),
], ids=lambda v: str(v) if isinstance(v, int) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_two_ranges(spec, ranges):
    case = workloads.make_case(B=1, dtype="f32", seed=521, device=DEV, **spec)
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], kv_heads=case.get("kv_heads", 0))
    p = walk._walk_params()
    chunks = B.chunk_array(case["K"], case["V"], case["k_offs"], None, p)
    assert B.burst_walk_workspace_bytes(chunks, p, B.BURST_WALK_FORWARD) == (ranges > 1) * ranges * spec["H"] * spec["Nq"] * (spec["d"] + 2) * 4
    O, lse = [t.clone() for t in walk.forward(case["K"], case["V"], case["k_offs"])]
    dQ, dKs, dVs = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"])
    torch.cuda.synchronize()
    compare_all_heads(case, "f32", O, lse, dQ, dKs, dVs)
    B.burst_walk_fwd(case["Q"], chunks, walk.O_acc, walk.m, walk.l, walk.O, walk.lse, p)
    torch.cuda.synchronize()
    assert float((lse - walk.lse).abs().max()) < 1e-5 and float((O - walk.O).norm()) <= 1e-5 * float(O.norm())   # fp32 sums in another order

"""Grouped heads whose query slice is no multiple of the dK/dV kernel's 64-row tiles: every head of a
group then ends in a partial tile of its own, in front of the next head's first row.  Sizes around
one and two tiles, with each mask and memory layout, against the oracle at the usual bf16 bars."""
import pytest
import torch

from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    dict(B=1, H=2, kv_heads=1, Nq=1, chunk_rows=[130]),
    dict(B=1, H=6, kv_heads=2, Nq=63, chunk_rows=[64, 70]),
    dict(B=2, H=4, kv_heads=2, Nq=65, chunk_rows=[129], layout="seq"),
    dict(B=1, H=8, kv_heads=1, Nq=129, chunk_rows=[200], causal=True, q_off=71, layout="packed"),
    dict(B=1, H=4, kv_heads=2, Nq=300, chunk_rows=[260, 40], causal=True, q_off=0, window=90),
    dict(B=1, H=4, kv_heads=2, Nq=190, chunk_rows=[300], block=64, pattern="random", density=0.5, per_head_flags=True),
    dict(B=1, H=6, kv_heads=2, Nq=130, chunk_rows=[257], block=128, pattern="random", density=0.5),
]


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items()))
def test_grouped_heads_with_partial_last_tiles(spec):
    case = workloads.make_case(dtype="bf16", d=128, seed=91, device=DEV, **spec)
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], case.get("block", 0),
                    case["kv_heads"])
    O, lse = walk.forward(case["K"], case["V"], case["k_offs"], masks=case.get("masks"))
    dQ, dKs, dVs = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"], masks=case.get("masks"))
    torch.cuda.synchronize()
    compare_all_heads(case, "bf16", O, lse, dQ, dKs, dVs)

"""bf16 head dimensions other than 64 and 128 on the padded builds of the plainly written kernels:
the first, a middle and the last multiple of 8 of every padded width, rows and keys around the edges
of the 128-row and 64-key tiles, with each mask, grouped heads and strided tensors, against the oracle at
the usual bf16 bars."""
import pytest
import torch

from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    dict(B=1, H=2, d=8, Nq=127, chunk_rows=[65, 63]),
    dict(B=1, H=2, d=24, Nq=129, chunk_rows=[128], causal=True, q_off=10),
    dict(B=2, H=2, d=32, Nq=70, chunk_rows=[1, 190], layout="seq"),
    dict(B=1, H=2, d=40, Nq=257, chunk_rows=[255], causal=True, q_off=0, window=70),
    dict(B=1, H=4, kv_heads=2, d=56, Nq=100, chunk_rows=[64, 65], causal=True, q_off=29),
    dict(B=1, H=2, d=72, Nq=130, chunk_rows=[200], block=64, pattern="random", density=0.5),
    dict(B=1, H=3, d=80, Nq=128, chunk_rows=[129, 31], causal=True, q_off=32, layout="packed"),
    dict(B=1, H=4, kv_heads=1, d=96, Nq=161, chunk_rows=[161], causal=True, layout="seq"),
    dict(B=1, H=2, d=104, Nq=64, chunk_rows=[64]),
    dict(B=1, H=2, d=40, Nq=64, chunk_rows=[130, 65], block=64, pattern="random", density=0.5),        # one wavefront's flags a row block
    dict(B=1, H=2, d=40, Nq=65, chunk_rows=[130, 65], block=64, pattern="random", density=0.5),        # ... and two
    dict(B=1, H=43, d=40, Nq=300, chunk_rows=[130, 65], block=64, pattern="random", density=0.5),      # 129 row blocks: four
    dict(B=1, H=2, d=120, Nq=200, chunk_rows=[90, 110], block=128, pattern="band_global", causal=True, q_off=0),
]


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items()))
def test_padded_head_dimensions(spec):
    case = workloads.make_case(dtype="bf16", seed=83, device=DEV, **spec)
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], case.get("block", 0),
                    case.get("kv_heads", 0))
    O, lse = walk.forward(case["K"], case["V"], case["k_offs"], masks=case.get("masks"))
    dQ, dKs, dVs = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"], masks=case.get("masks"))
    torch.cuda.synchronize()
    compare_all_heads(case, "bf16", O, lse, dQ, dKs, dVs)

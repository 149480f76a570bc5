"""The fp32 matrix-core kernels (burst_generic.hip) where their tiling can go wrong: 32-row and 32-key
blocks with one row more and one less, every padded head dimension with and without a remainder,
rows that do not start on 16 bytes, and row counts on both sides of the line between four and eight
wavefronts per workgroup (256 row blocks), against the oracle at the usual fp32 bars."""
import pytest
import torch

from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [("f32", dict(B=1, H=2, d=d, Nq=nq, chunk_rows=rows, **kw))
         for d, nq, rows, kw in [
             (4, 31, [33], {}), (20, 32, [32, 1], dict(causal=True, q_off=20)), (33, 33, [31, 64], {}),
             (30, 65, [100], dict(causal=True, q_off=40, window=9)), (64, 257, [255, 31], dict(causal=True, q_off=29)),
             (68, 95, [97], {}), (96, 64, [63, 65], dict(window=40)), (100, 33, [161], dict(causal=True, q_off=128)),
             (128, 1, [290], {}), (128, 190, [1, 129], dict(block=64, pattern="random", density=0.5)),
             (127, 40, [70], {})]]
CASES += [("f32", dict(B=1, H=8, d=64, Nq=n, chunk_rows=[n], causal=True, q_off=0)) for n in (1024, 1025)]
CASES += [("f32", dict(B=1, H=2, d=d, Nq=70, chunk_rows=rows, **kw))            # at most four key tiles, d > 64: tiles from memory
          for d, rows, kw in [(68, [128], {}), (72, [128, 1], {}), (96, [33, 31, 5], dict(causal=True, q_off=20)), (100, [1], {}),
                              (124, [97], dict(window=30, q_off=40)), (128, [60, 64], dict(layout="seq")), (128, [128], dict(block=64, pattern="random", density=0.5))]]
CASES += [("f32", dict(B=1, H=6, kv_heads=2, d=48, Nq=70, chunk_rows=[90], causal=True, q_off=20)),
          ("bf16", dict(B=1, H=2, d=70, Nq=70, chunk_rows=[90], causal=True, q_off=20)),
          ("bf16", dict(B=1, H=4, kv_heads=2, d=7, Nq=33, chunk_rows=[65]))]


@pytest.mark.parametrize("dtype,spec", CASES, ids=lambda v: v if isinstance(v, str) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_generic_tiles(dtype, spec):
    case = workloads.make_case(dtype=dtype, seed=71, device=DEV, **spec)
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], case.get("block", 0),
                    case.get("kv_heads", 0))
    O, lse = walk.forward(case["K"], case["V"], case["k_offs"], masks=case.get("masks"))
    dQ, dKs, dVs = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"], masks=case.get("masks"))
    torch.cuda.synchronize()
    compare_all_heads(case, dtype, O, lse, dQ, dKs, dVs)

"""dK / dV launches whose walks over query tiles are cut into parts (partial gradients added by another launch): each
kernel family, blocks of keys with one part beside blocks with several or none, ragged ends, masks, chunks of different
length, blocks without rows among the partial gradients, accumulation, gradients in the inputs' type, infinities; against the oracle and against the call without a workspace
(which cannot cut): the same products summed in another order, fp32 sums of at most 2100 terms, 1e-5 of the norm."""
import numpy as np
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    dict(H=1, d=64, Nq=760, chunk_rows=[129]),                                               # 24 tiles, the fewest that are cut
    dict(H=8, kv_heads=1, d=64, Nq=100, chunk_rows=[130, 1, 200], causal=True, q_off=200),
    dict(H=3, d=64, Nq=1500, chunk_rows=[1500], causal=True, layout="seq"),
    dict(H=1, d=128, Nq=2048, chunk_rows=[127]),                                             # 32 tiles of 64 rows
    dict(H=2, d=128, Nq=2100, chunk_rows=[2100], causal=True),
    dict(H=8, kv_heads=1, d=128, Nq=256, chunk_rows=[100, 300], causal=True, q_off=130, layout="packed"),
    dict(H=16, kv_heads=2, d=128, Nq=256, chunk_rows=[300], window=150, q_off=150),
    dict(H=16, kv_heads=1, d=128, Nq=512, chunk_rows=[700, 300, 129, 300, 400], window=300, q_off=800),   # hidden blocks before and after
    dict(H=2, d=64, Nq=1500, chunk_rows=[300, 700, 900, 100, 600], window=900, q_off=700, causal=True),
    dict(H=12, kv_heads=2, d=128, Nq=161, chunk_rows=[65, 190], causal=True, q_off=90),      # partial last tiles: 24-bit P and dS
    dict(H=8, kv_heads=2, d=40, Nq=321, chunk_rows=[128, 129], window=100, q_off=-40),
    dict(H=2, d=96, Nq=900, chunk_rows=[900], causal=True),
    dict(H=4, kv_heads=1, d=8, Nq=300, chunk_rows=[33]),
    dict(H=8, kv_heads=2, d=96, Nq=321, chunk_rows=[400, 300, 129, 300], window=200, q_off=500, causal=True),
]


def walk_of(spec):
    case = workloads.make_case(B=1, dtype="bf16", seed=211, device=DEV, **spec)
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], kv_heads=case.get("kv_heads", 0))
    walk.forward(case["K"], case["V"], case["k_offs"])
    p = walk._walk_params()
    held = 0 if walk._workspace is None else walk._workspace.numel()
    assert held == B.burst_walk_workspace_bytes(B.chunk_array(case["K"], case["V"], case["k_offs"], None, p), p, B.BURST_WALK_FORWARD)
    return case, walk


def gradients(case, walk, workspace, dtype=torch.float32, into=None, accumulate=False):
    p = walk._walk_params()
    dQ = torch.zeros(walk.Q.shape, device=DEV, dtype=dtype)
    dKs, dVs = into or [[torch.full(x.shape, 5.0, device=DEV, dtype=dtype) for x in xs] for xs in (case["K"], case["V"])]
    chunks = B.chunk_array(case["K"], case["V"], case["k_offs"], None, p, dKs, dVs, dtype)
    ws = torch.empty(B.burst_walk_workspace_bytes(chunks, p, 0), device=DEV, dtype=torch.uint8).fill_(255) if workspace else None
    assert not workspace or B.burst_walk_dkv_form(chunks, p) == 1
    B.burst_walk_bwd(walk.Q, chunks, walk.O, case["dO"], walk.lse, walk.D, dQ, p, accumulate_dq=False, accumulate_dkv=accumulate,
                     workspace=ws)
    torch.cuda.synchronize()
    return dQ, dKs, dVs


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items() if k != "chunk_rows"))
def test_parts_add_up(spec):
    case, walk = walk_of(spec)
    dQ, dKs, dVs = gradients(case, walk, True)
    compare_all_heads(case, "bf16", walk.O, walk.lse, dQ, dKs, dVs)
    for a, b in zip(dKs + dVs, sum(gradients(case, walk, False)[1:], [])):
        assert float((a - b).norm()) <= 1e-5 * float(b.norm())
    half = gradients(case, walk, True, torch.bfloat16)
    for a, b in zip(half[1] + half[2], dKs + dVs):      # the same sums, rounded once
        assert torch.equal(a, b.bfloat16())
    twice = gradients(case, walk, True, into=[[x.clone() for x in xs] for xs in (dKs, dVs)], accumulate=True)
    for a, b in zip(twice[1] + twice[2], dKs + dVs):
        assert torch.allclose(a, 2 * b, rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("spec", CASES[9:], ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items() if k != "chunk_rows"))
def test_infinities_in_parts(spec):
    """Padded kernels: the same entries are infinite or NaN as without parts, the others as close as ever."""
    case, walk = walk_of(spec)
    case["dO"][:, :, spec["Nq"] // 3, 1] = float("inf")
    case["V"][0][:, :, 20:23, 3] = -float("inf")
    walk.forward(case["K"], case["V"], case["k_offs"])
    got, want = (sum(gradients(case, walk, ws)[1:], []) for ws in (True, False))
    for a, b in zip(got, want):
        a, b = f64(a), f64(b)
        for cls in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(cls(a), cls(b))
        fin = np.isfinite(b)
        assert np.linalg.norm((a - b)[fin]) <= 1e-5 * max(np.linalg.norm(b[fin]), 1e-30)

"""fp32 walks of few rows (or keys) whose tiles are dealt to several workgroups per block and merged by another launch: edges of
the 32-row blocks, ranges without a visible key, every padded head dimension, grouped heads, strided rows; against the
oracle, against the walk without a workspace (which cannot split; fp32 sums of at most 1300 terms in another order, 1e-5
of the norm), accumulation, infinities and NaN."""
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads
from test_gpu_nonfinite_inputs import check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    dict(H=1, d=64, Nq=256, chunk_rows=[256] * 4),
    dict(H=1, d=4, Nq=1, chunk_rows=[1300]),
    dict(H=2, d=128, Nq=33, chunk_rows=[500, 1, 310], causal=True, q_off=700),
    dict(H=3, d=36, Nq=520, chunk_rows=[300, 290], causal=True, q_off=-20),          # rows that see nothing
    dict(H=2, d=96, Nq=100, chunk_rows=[600], window=150, q_off=300, layout="seq"),
    dict(H=4, kv_heads=2, d=80, Nq=129, chunk_rows=[400, 33], causal=True, q_off=304, layout="packed"),
    dict(H=8, kv_heads=1, d=32, Nq=160, chunk_rows=[97]),
    dict(H=1, d=128, Nq=500, chunk_rows=[500]),
    dict(H=5, d=64, Nq=700, chunk_rows=[700], causal=True),
    dict(H=2, d=128, Nq=600, chunk_rows=[300, 330, 600, 300], window=300, q_off=500, causal=True),     # hidden blocks before and after
    dict(H=4, kv_heads=2, d=36, Nq=300, chunk_rows=[200, 330, 100, 300], window=200, q_off=500, causal=True),
]


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items() if k != "chunk_rows"))
def test_split_walks(spec):
    case = workloads.make_case(B=1, dtype="f32", seed=227, device=DEV, **spec)
    args = case["K"], case["V"], case["k_offs"]
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], kv_heads=case.get("kv_heads", 0))
    p = walk._walk_params()
    assert B.burst_walk_workspace_bytes(B.chunk_array(*args, None, p), p) > 0
    for t in (walk.O_acc, walk.m, walk.l):
        t.fill_(float("nan"))
    O, lse = walk.forward(*args)
    got = [t.clone() for t in (O, lse, walk.O_acc, walk.m, walk.l)]
    dQ, dKs, dVs = walk.backward(*args, case["dO"])
    compare_all_heads(case, "f32", O, lse, dQ, dKs, dVs)
    twice = [dQ.clone(), *[[t.clone() for t in ts] for ts in (dKs, dVs)]]
    ws = walk._workspace.fill_(255)
    B.burst_walk_bwd(walk.Q, B.chunk_array(*args, None, p, *twice[1:], torch.float32), walk.O, walk._like_q(case["dO"]), walk.lse, walk.D,
                     twice[0], p, accumulate_dq=True, accumulate_dkv=True, workspace=ws)
    torch.cuda.synchronize()
    for a, b in zip([twice[0], *twice[1], *twice[2]], [dQ, *dKs, *dVs]):
        assert torch.allclose(a, 2 * b, rtol=1e-6, atol=1e-7)
    # without a workspace
    B.burst_walk_fwd(walk.Q, B.chunk_array(*args, None, p), walk.O_acc, walk.m, walk.l, walk.O, walk.lse, p)
    one = [torch.empty_like(dQ), [torch.empty_like(t) for t in dKs], [torch.empty_like(t) for t in dVs]]
    B.burst_walk_bwd(walk.Q, B.chunk_array(*args, None, p, *one[1:], torch.float32), walk.O, walk._like_q(case["dO"]), walk.lse, walk.D, one[0], p,
                     accumulate_dq=False, accumulate_dkv=False)
    torch.cuda.synchronize()
    seen = torch.isfinite(walk.lse)
    assert torch.equal(seen, torch.isfinite(got[1])) and float((got[1] - walk.lse)[seen].abs().max() if seen.any() else 0.0) < 1e-5
    for a, b in zip([got[0], got[2], dQ, *dKs, *dVs], [walk.O, walk.O_acc, one[0], *one[1], *one[2]]):
        assert float((a - b).norm()) <= 1e-5 * float(b.norm())


@pytest.mark.parametrize("what", ["V inf", "V NaN in the last keys", "scores -inf", "scores -inf, last column", "all scores -inf", "dO inf",
                                  "dO NaN"])
@pytest.mark.parametrize("spec", [dict(H=2, d=64, Nq=100, chunk_rows=[300, 270]), dict(H=2, d=128, Nq=130, chunk_rows=[300, 270], causal=True, q_off=440),
                                  dict(H=4, kv_heads=1, d=36, Nq=70, chunk_rows=[60, 460], causal=True, q_off=450)], ids=["full", "causal", "grouped"])
def test_infinities_and_nan_in_split_walks(spec, what):
    check("f32", spec, what)

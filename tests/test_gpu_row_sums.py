"""D = rowsum(dO o O) as burst_walk_bwd leaves it, computed by its dQ launch or by one of its own, against burst_bwd_prepare: the
same bits, whichever kernel it is (an order of its own would have an error of its own); rows without a visible key, walks that
only add to dQ and walks of more rows than fp32 kernels compute D for included."""
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 8), ("bf16", 24), ("bf16", 56), ("bf16", 64), ("bf16", 72), ("bf16", 96), ("bf16", 120), ("bf16", 128),
                                     ("bf16", 20), ("f32", 4), ("f32", 12), ("f32", 20), ("f32", 32), ("f32", 36), ("f32", 64), ("f32", 68), ("f32", 96),
                                     ("f32", 128), ("f32", 34)])
@pytest.mark.parametrize("layout,k_off,Nq", [("head", 0, 131), ("seq", 60, 131), ("packed", 5000, 131), ("head", 0, 1400), ("head", 0, 5500)])
def test_row_sums_of_a_walk(dtype, d, layout, k_off, Nq):
    if layout != "head" and d * (2 if dtype == "bf16" else 4) % 16:
        pytest.skip("strided rows start on 16 bytes")
    case = workloads.make_case(B=2, H=3, d=d, Nq=Nq, chunk_rows=[70, 33], dtype=dtype, seed=229, device="cuda:0", causal=True, q_off=20,
                               k_offs=[k_off, k_off + 70], layout=layout)
    walk = RingWalk(case["Q"], case["scale"], True, 20)
    walk.forward(case["K"], case["V"], case["k_offs"])
    walk.O.copy_(torch.randn_like(walk.O))          # (rows that see nothing too)
    walk.prepare(walk._like_q(case["dO"]))
    want = walk.D.clone()
    for kept in (None, torch.full(tuple(case["Q"].shape), 2.0, device="cuda:0")):
        walk.D.fill_(float("nan"))
        dQ, _, _ = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"], dQ=kept)
        torch.cuda.synchronize()
        assert torch.equal(walk.D, want)
        if k_off == 5000:
            assert torch.all(dQ == (0.0 if kept is None else 2.0))

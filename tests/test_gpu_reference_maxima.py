"""The reference maxima of the bf16 forward kernels: the largest probability of a chunk's first tile is 1, exact in
bf16, so rows that see one key have O = V bit for bit and lse = their score, whatever the kernel family and however many
chunks one launch takes; and chunks whose scores lie far above or below the state's."""
import numpy as np
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def forward(case, step_by_step):
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], case.get("block", 0), case.get("kv_heads", 0))
    if not step_by_step:
        return walk.forward(case["K"], case["V"], case["k_offs"])
    walk.init()
    for K, V, off in zip(case["K"], case["V"], case["k_offs"]):
        walk.step(K, V, off)
    return walk.finalize()


@pytest.mark.parametrize("step_by_step", [False, True])
@pytest.mark.parametrize("spec,family", [
    (dict(d=64, Nq=200, chunk_rows=[70, 200]), 0), (dict(d=128, Nq=300, chunk_rows=[100, 200]), 1),
    (dict(d=128, Nq=300, chunk_rows=[100, 200]), 2), (dict(d=96, Nq=150, chunk_rows=[150]), 0),
], ids=["d64", "hand", "plain", "padded"])
def test_a_row_that_sees_one_key_is_exact(spec, family, step_by_step):
    """Window 1: every row sees the key at its own position only.  lse is the fp32 score: the sum of d products of two
    8-bit numbers (d x 2^-24) and m, log l in fp32 (a rounding of P would be 2^-9)."""
    B.burst_set_kernel_family(family)
    try:
        case = workloads.make_case(B=1, H=2, dtype="bf16", seed=113, device=DEV, causal=True, q_off=0, window=1, **spec)
        O, lse = forward(case, step_by_step)
        torch.cuda.synchronize()
        K, V = [torch.cat(x, dim=2)[:, :, :spec["Nq"]] for x in (case["K"], case["V"])]
        assert torch.equal(O[:, :, :K.shape[2]], V)
        want = case["scale"] * (f64(case["Q"][:, :, :K.shape[2]]) * f64(K)).sum(-1)
        assert np.abs(f64(lse)[:, :, :K.shape[2]] - want).max() < 4e-6
    finally:
        B.burst_set_kernel_family(0)


@pytest.mark.parametrize("factors", [[1, 30, 1e-3], [30, 1, 30], [1e-3, 1, 8, 60], [60, 8, 1, 1e-3]])
@pytest.mark.parametrize("d,family", [(64, 0), (128, 1), (128, 2), (40, 0)])
def test_chunks_far_above_and_below_the_state(d, family, factors):
    """Keys scaled per chunk: first maxima of some ten to some hundred powers of two above or below the reference so far."""
    B.burst_set_kernel_family(family)
    try:
        case = workloads.make_case(B=1, H=2, d=d, Nq=130, chunk_rows=[100, 70, 130, 64][:len(factors)], dtype="bf16", seed=127, device=DEV)
        for K, f in zip(case["K"], factors):
            K.mul_(f)
        O, lse = [t.clone() for t in forward(case, False)]
        compare_all_heads(case, "bf16", O, lse)
        O1, lse1 = forward(case, True)
        torch.cuda.synchronize()
        assert torch.equal(O, O1) and torch.equal(lse, lse1)
        rev = dict(case, K=case["K"][::-1], V=case["V"][::-1], k_offs=case["k_offs"][::-1])
        O2, lse2 = forward(rev, False)
        torch.cuda.synchronize()
        # the same rounding of P in another order: fp32 sums (2^-24 of |lse| up to 1000 each), O may round the other way
        assert float((lse2 - lse).abs().max()) < 5e-4
        assert torch.allclose(O.float(), O2.float(), rtol=2 ** -7, atol=1e-3)
    finally:
        B.burst_set_kernel_family(0)

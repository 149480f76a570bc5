"""Differentiable calls whose workgroups halve every tile between two groups of wavefronts (key groups in the forward and dQ
kernels, row groups in the dK/dV kernel) against the oracle and against the walk of the same chunk, which has one group: tails of one row and one key,
rows that see nothing, windows, grouped heads, every build, calls that are split by keys besides; halves of a tile whose scores lie far
apart; and infinities and NaN."""
import numpy as np
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.autograd import burst_attention
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    dict(H=2, d=64, Nq=1, chunk_rows=[1]),
    dict(H=3, d=64, Nq=65, chunk_rows=[33], causal=True),
    dict(H=3, d=64, Nq=130, chunk_rows=[161], causal=True, q_off=-40),             # 40 rows see nothing
    dict(H=40, d=64, Nq=193, chunk_rows=[190], causal=True),                       # more than 256 workgroups: mirrored
    dict(H=2, d=128, Nq=63, chunk_rows=[97], window=40, q_off=30),
    dict(H=4, kv_heads=2, d=128, Nq=700, chunk_rows=[700], causal=True, layout="seq"),
    dict(H=24, d=128, Nq=2100, chunk_rows=[2100], causal=True),                    # hand-scheduled chunk by chunk
    dict(H=2, d=96, Nq=300, chunk_rows=[300], causal=True, window=70),
    dict(H=6, kv_heads=3, d=80, Nq=257, chunk_rows=[65]),
    dict(H=2, d=40, Nq=64, chunk_rows=[130], causal=True, q_off=66),
    dict(H=2, d=8, Nq=129, chunk_rows=[31], causal=True, q_off=-3),
    dict(H=9, d=120, Nq=200, chunk_rows=[200], causal=True, layout="packed"),
    dict(H=36, d=64, Nq=1500, chunk_rows=[1100], causal=True, q_off=100),
]


def both(case):
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], kv_heads=case.get("kv_heads", 0))
    O, lse = walk.forward(case["K"], case["V"], case["k_offs"])
    dQ, dKs, dVs = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"])
    leaves = [t.detach().requires_grad_(True) for t in (case["Q"], case["K"][0], case["V"][0])]
    O1, lse1 = burst_attention(*leaves, scale=case["scale"], causal=case["causal"], q_off=case["q_off"], window=case["window"])
    grads = torch.autograd.grad(O1, leaves, case["dO"])
    torch.cuda.synchronize()
    return (O, lse, dQ, dKs[0], dVs[0]), (O1.detach(), lse1, *grads)


def compare(case, spec, lse_bar=1e-5):
    want, got = both(case)
    some = None if spec.get("kv_heads") else sorted({0, spec["H"] // 2, spec["H"] - 1})
    compare_all_heads(case, "bf16", *got[:3], [got[3]], [got[4]], heads=some, dkv_kind="rel")    # (gradients of some 10, rounded to bf16)
    seen = torch.isfinite(want[1])
    assert torch.equal(seen, torch.isfinite(got[1])) and torch.equal(want[1][~seen], got[1][~seen])
    # the same probabilities, their fp32 sums in another order (2^-24 each); O next to a rounding boundary may round the other way
    assert not seen.any() or float((want[1] - got[1])[seen].abs().max()) < lse_bar
    assert torch.allclose(want[0].float(), got[0].float(), rtol=2 ** -7, atol=1e-3)
    for a, b in zip(got[2:], want[2:]):             # rounded to bf16 (2^-9), and D comes from that O
        assert float((a.float() - b).norm()) <= 4e-3 * float(b.norm()) + 1e-6


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items()))
def test_groups_equal_the_walk_of_one_group(spec):
    compare(workloads.make_case(B=1, dtype="bf16", seed=307, device=DEV, **spec), spec)


SPLIT = [                                            # key ranges of the forward, and at least of dQ
    (dict(H=8, d=64, Nq=2048, chunk_rows=[2048], causal=True), 4, 4),
    (dict(H=8, d=64, Nq=2048, chunk_rows=[2048]), 4, 4),                           # one group
    (dict(H=8, d=64, Nq=2050, chunk_rows=[2050], causal=True, window=2000), 3, 3),
    (dict(H=8, kv_heads=2, d=64, Nq=1985, chunk_rows=[2111], causal=True, q_off=126, layout="seq"), 4, 4),
    (dict(H=8, d=128, Nq=2048, chunk_rows=[2048], causal=True), 2, 2),
    (dict(H=5, d=128, Nq=2050, chunk_rows=[2050], causal=True, window=2000), 3, 3),
    (dict(H=5, d=128, Nq=2050, chunk_rows=[2050]), 3, 3),
    (dict(H=8, d=96, Nq=2048, chunk_rows=[2048], causal=True), 4, 2),
    (dict(H=5, d=120, Nq=1601, chunk_rows=[1601], causal=True), 3, 3),
    (dict(H=6, d=40, Nq=2050, chunk_rows=[2050], causal=True, window=2000), 5, 5),
]


def ranges(case, flags, spec):
    p = B.params(1, spec["H"], spec["Nq"], 0, spec["d"], "bf16", case["scale"], case["causal"], case["q_off"], window=case["window"],
                 kv_heads=case.get("kv_heads", 0))
    n = B.burst_walk_workspace_bytes(B.chunk_array(case["K"], case["V"], case["k_offs"], None, p), p, flags)
    return n / (spec["H"] * spec["Nq"] * (spec["d"] + 2) * 4)


@pytest.mark.parametrize("spec,forward,backward", SPLIT, ids=lambda v: "-".join(f"{k}{x}" for k, x in v.items()) if isinstance(v, dict) else str(v))
def test_calls_that_are_split_besides(spec, forward, backward):
    case = workloads.make_case(B=1, dtype="bf16", seed=313, device=DEV, **spec)
    assert ranges(case, B.BURST_WALK_NO_STATE | B.BURST_WALK_FORWARD, spec) == forward and ranges(case, B.BURST_WALK_HALF_GRADS, spec) >= backward
    # Under a window the first tile of a range, and with it the reference that 8-bit probabilities are rounded against, depends on a
    # workgroup's rows: each of them is off by 2^-9 either way, and so is their sum at most.
    compare(case, spec, 2 ** -8 if case["window"] and spec["d"] in (64, 128) else 1e-5)


@pytest.mark.parametrize("d", [64, 128, 40, 96, 120])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("factors", [[1, 30], [30, 1], [1e-3, 8, 60, 1], [60, 1e-3, 1, 8]])
def test_halves_of_a_tile_far_apart(d, causal, factors):
    """Keys scaled by halves of a tile: the two groups' maxima some ten to some hundred powers of two apart, either way."""
    case = workloads.make_case(B=1, H=2, d=d, Nq=200, chunk_rows=[230], causal=causal, q_off=30, dtype="bf16", seed=317, device=DEV)
    for i in range(0, 230, 32):
        case["K"][0][:, :, i:i + 32] *= factors[i // 32 % len(factors)]
    _, got = both(case)
    compare_all_heads(case, "bf16", *got[:2])


@pytest.mark.parametrize("d,causal", [(8, True), (40, True), (96, True), (120, True), (64, False), (128, False)])
@pytest.mark.parametrize("where", ["Q", "K", "V", "dO"])
def test_infinities_and_nan_where_the_walk_has_them(d, causal, where):
    """(d = 64 and 128 multiply hidden pairs too, of which smaller workgroups have fewer: there without a mask.)"""
    case = workloads.make_case(B=1, H=2, d=d, Nq=150, chunk_rows=[150], causal=causal, dtype="bf16", seed=311, device=DEV)
    t = case[where][0] if where in "KV" else case[where]
    for i, x in enumerate((float("inf"), float("-inf"), float("nan"))):
        t[0, i % 2, 17 + 48 * i, 3 + i] = x          # rows of both halves of a tile
    want, got = both(case)
    for a, b in zip(got, want):
        a, b = f64(a), f64(b)
        for cls in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(cls(a), cls(b))

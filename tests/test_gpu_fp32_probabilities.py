"""bf16 calls whose probabilities and dS keep their 24 bits (head dimensions other than 64 and 128; dK and dV of
grouped heads whose slice is no multiple of 64 rows): lse, O and the fp32 gradients of a walk against 64 bits, at
a bar that 8-bit probabilities miss a hundred times over.

The bar: with |x| = |scale s - lse| up to about 20 in log2 units, an fp32 exponent is off by 20 x 2^-24 = 1.2e-6 at
worst, sums of n terms add about sqrt(n) x 2^-24 (n = 1000: 2e-6), so 4e-6 of the result's norm; 8-bit probabilities
give 1.6e-3.  The gradients are compared with those of the D that the call computed from its own bf16 O."""
import numpy as np
import pytest
import torch

from paper_2403_09347_amd import binding as B
from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import f64, head_inputs, pattern_of

pytestmark = pytest.mark.gpu
BAR = 4e-6

CASES = [
    dict(B=1, H=2, d=8, Nq=127, chunk_rows=[65, 63]),
    dict(B=1, H=2, d=40, Nq=257, chunk_rows=[255, 190], causal=True, q_off=188),
    dict(B=1, H=4, kv_heads=2, d=72, Nq=130, chunk_rows=[200], block=64, pattern="random", density=0.5),
    dict(B=1, H=3, d=80, Nq=129, chunk_rows=[129, 31], causal=True, q_off=32, window=90, layout="packed"),
    dict(B=1, H=4, kv_heads=1, d=96, Nq=161, chunk_rows=[161], causal=True, layout="seq"),
    dict(B=1, H=2, d=96, Nq=33, chunk_rows=[1000, 1100]),          # split keys
    dict(B=1, H=2, d=120, Nq=200, chunk_rows=[90, 110]),
]

GROUPED = [
    dict(B=1, H=2, kv_heads=1, Nq=1, chunk_rows=[130]),
    dict(B=1, H=6, kv_heads=2, Nq=63, chunk_rows=[64, 70]),
    dict(B=2, H=4, kv_heads=2, Nq=65, chunk_rows=[129], layout="seq"),
    dict(B=1, H=8, kv_heads=1, Nq=129, chunk_rows=[200], causal=True, q_off=71, layout="packed"),
    dict(B=1, H=4, kv_heads=2, Nq=300, chunk_rows=[260, 40], causal=True, q_off=0, window=90),
    dict(B=1, H=4, kv_heads=2, Nq=190, chunk_rows=[300], block=64, pattern="random", density=0.5, per_head_flags=True),
    dict(B=1, H=6, kv_heads=2, Nq=130, chunk_rows=[257], block=128, pattern="random", density=0.5),
]


def references(case, walk, b, h, own_lse=False):
    """lse, O, dQ, dK, dV of one query head in 64 bits, with D from the walk's O (own_lse: and the walk's lse)."""
    Q, K, V, dO, qp, kp = head_inputs(case, b, h)
    seen = np.ones((len(qp), len(kp)), bool)
    if case["causal"]:
        seen &= kp[None] <= qp[:, None]
    if case.get("window"):
        seen &= kp[None] > qp[:, None] - case["window"]
    pat = pattern_of(case, b=b, h=h)
    if pat is not None:
        seen &= pat
    S = np.where(seen, case["scale"] * (Q @ K.T), -np.inf)
    top = np.where(seen.any(1), S.max(1), 0.0)
    l = np.exp(S - top[:, None]).sum(1)
    with np.errstate(divide="ignore"):
        lse = f64(walk.lse[b, h]) if own_lse else top + np.log(l)
    P = np.exp(S - np.where(np.isfinite(lse), lse, 0.0)[:, None]) * seen
    dS = P * (dO @ V.T - (dO * f64(walk.O[b, h])).sum(1)[:, None])
    return lse, P @ V, case["scale"] * (dS @ K), case["scale"] * (dS.T @ Q), P.T @ dO


def off(got, want):
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


def check_gradients(case, walk, grads, own_lse=False):
    dQ, dKs, dVs = grads
    H, hk = case["Q"].shape[1], case["K"][0].shape[1]
    for b in range(case["Q"].shape[0]):
        for k in range(hk):
            refs = [references(case, walk, b, h, own_lse) for h in range(k * (H // hk), (k + 1) * (H // hk))]
            dK, dV = [np.concatenate([f64(g[b, k]) for g in gs]) for gs in (dKs, dVs)]
            if not own_lse:
                assert off(np.concatenate([f64(dQ[b, k * (H // hk) + i]) for i in range(len(refs))]), np.concatenate([r[2] for r in refs])) < BAR
            assert off(dK, sum(r[3] for r in refs)) < BAR
            assert off(dV, sum(r[4] for r in refs)) < BAR


def walk_of(case):
    walk = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"], case["window"], case.get("block", 0), case.get("kv_heads", 0))
    O, lse = walk.forward(case["K"], case["V"], case["k_offs"], masks=case.get("masks"))
    grads = walk.backward(case["K"], case["V"], case["k_offs"], case["dO"], masks=case.get("masks"))
    torch.cuda.synchronize()
    return walk, O, lse, grads


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items() if k != "chunk_rows"))
def test_padded_head_dimensions_keep_fp32_probabilities(spec):
    case = workloads.make_case(dtype="bf16", seed=107, device="cuda:0", **spec)
    walk, O, lse, grads = walk_of(case)
    for b in range(spec["B"]):
        for h in range(spec["H"]):
            lse_ref, O_ref = references(case, walk, b, h)[:2]
            seen = np.isfinite(lse_ref)
            assert np.array_equal(f64(lse[b, h])[~seen], lse_ref[~seen])
            assert np.abs(f64(lse[b, h]) - lse_ref)[seen].max() < 4e-6
            # O is the 64-bit result rounded once to bf16 (8 bits: 2^-8 of a value at most), and as far off as that in the norm
            assert np.all(np.abs(f64(O[b, h]) - O_ref) <= np.abs(O_ref) * 2.0 ** -8 + 1e-5)
            assert off(f64(O[b, h]), O_ref) < 1.02 * off(f64(torch.from_numpy(O_ref).bfloat16()), O_ref) + BAR
    check_gradients(case, walk, grads)


@pytest.mark.parametrize("family", [0, 1])
@pytest.mark.parametrize("spec", GROUPED, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items() if k != "chunk_rows"))
def test_grouped_heads_with_partial_last_tiles_keep_fp32_probabilities_in_dkv(spec, family):
    """(O and lse come from the kernels with 8-bit probabilities: the references take lse and D from them.)"""
    B.burst_set_kernel_family(family)
    try:
        case = workloads.make_case(dtype="bf16", d=128, seed=109, device="cuda:0", **spec)
        walk, _, _, grads = walk_of(case)
        check_gradients(case, walk, grads, own_lse=True)
    finally:
        B.burst_set_kernel_family(0)


@pytest.mark.parametrize("d", [40, 96, 120])
def test_gradients_of_tiny_values(d):
    """dO times 2^-60 and 2^-100: the same digits.  Smaller, dS and the two remainders it is split into leave the range of
    normal numbers, where each counts as nothing: 2^-126 a pair for each at most, and as much for dP before."""
    case = workloads.make_case(B=1, H=2, d=d, Nq=192, chunk_rows=[192], dtype="bf16", seed=113, device="cuda:0")
    dO = case["dO"].float()
    for e in (60, 100, 112, 118):
        case["dO"] = (dO * 2.0 ** -e).bfloat16()
        walk, _, _, grads = walk_of(case)
        if e <= 100:
            check_gradients(case, walk, grads)
            continue
        for h in range(2):
            Q, K = f64(case["Q"][0, h]), f64(case["K"][0][0, h])
            _, _, dQ, dK, dV = references(case, walk, 0, h)
            lost = case["scale"] * 4 * 2.0 ** -126
            assert np.all(np.abs(f64(grads[0][0, h]) - dQ) <= lost * np.abs(K).sum(0) + BAR * np.abs(dQ).max())
            assert np.all(np.abs(f64(grads[1][0][0, h]) - dK) <= lost * np.abs(Q).sum(0) + BAR * np.abs(dK).max())
            assert off(f64(grads[2][0][0, h]), dV) < BAR

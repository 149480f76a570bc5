"""Scores far beyond the ordinary, from finite inputs, in the calls whose probabilities have 24 bits (fp32, bf16 head
dimensions other than 64 and 128): a row's largest key has the exponent 0 exactly in every kernel, however large its
score, so that a key of 1e30 takes or loses its rows whole; and keys pushed out by the lowest value of the type in
one column, alone in a tile, a chunk or the whole walk."""
import numpy as np
import pytest
import torch

from paper_2403_09347_amd import workloads
from paper_2403_09347_amd.harness import RingWalk
from gpu_util import compare_all_heads, f64, head_inputs, positions

pytestmark = pytest.mark.gpu

SPECS = [
    ("bf16", dict(H=2, d=96, Nq=130, chunk_rows=[100, 70])),
    ("bf16", dict(H=2, d=40, Nq=130, chunk_rows=[100, 70], causal=True, q_off=40)),
    ("bf16", dict(H=2, d=80, Nq=33, chunk_rows=[1000, 1100])),            # split keys
    ("bf16", dict(H=2, d=20, Nq=70, chunk_rows=[40, 33], causal=True, q_off=3)),
    ("f32", dict(H=2, d=64, Nq=100, chunk_rows=[90, 70])),
    ("f32", dict(H=2, d=128, Nq=130, chunk_rows=[100, 70], causal=True, q_off=40)),
    ("f32", dict(H=2, d=34, Nq=70, chunk_rows=[40, 33], causal=True, q_off=3)),
]
IDS = lambda v: v if isinstance(v, str) else "-".join(f"{k}{x}" for k, x in v.items() if k != "chunk_rows")


def walk(case):
    w = RingWalk(case["Q"], case["scale"], case["causal"], case["q_off"])
    O, lse = w.forward(case["K"], case["V"], case["k_offs"])
    grads = w.backward(case["K"], case["V"], case["k_offs"], case["dO"])
    torch.cuda.synchronize()
    return O, lse, grads


@pytest.mark.parametrize("dtype,spec", SPECS, ids=IDS)
def test_keys_at_the_lowest_value_of_the_type(dtype, spec):
    """Column 0 of Q is positive; keys with the lowest value there have scores of -1e37 to -inf."""
    for where in ("in a tile", "a whole tile", "a whole chunk"):
        case = workloads.make_case(B=1, dtype=dtype, seed=131, device="cuda:0", **spec)
        case["Q"][..., 0] = case["Q"][..., 0].abs() + 1.1
        low = torch.finfo(case["Q"].dtype).min
        rows = {"in a tile": slice(5, 20), "a whole tile": slice(1, 35), "a whole chunk": slice(0, None)}[where]
        case["K"][1 if where == "a whole chunk" else 0][:, :, rows, 0] = low
        O, lse, (dQ, dKs, dVs) = walk(case)
        compare_all_heads(case, dtype, O, lse, dQ, dKs, dVs)


@pytest.mark.parametrize("dtype,spec", SPECS, ids=IDS)
def test_a_key_of_1e30(dtype, spec):
    """Rows with a positive product see nothing but that key: O = V and dV = the sum of their dO; the others do
    not see it.  (dQ of the former is a rounding error times 1e30.)"""
    case = workloads.make_case(B=1, dtype=dtype, seed=137, device="cuda:0", **spec)
    case["K"][0][:, :, 5] *= 1e30
    O, lse, (dQ, dKs, dVs) = walk(case)
    rounding, rel = (2.0 ** -8, 1e-2) if dtype == "bf16" else (2.0 ** -20, 1e-5)
    for h in range(spec["H"]):
        Q, K, V, dO, qp, kp = head_inputs(case, 0, h)
        vis = (kp[None] <= qp[:, None]) if case["causal"] else np.ones((len(qp), len(kp)), bool)
        S = np.where(vis, case["scale"] * (Q @ K.T), -np.inf)
        top = S.max(1)
        P = np.exp(S - top[:, None])
        l = P.sum(1)
        P /= l[:, None]
        won = S[:, 5] > 1e20
        assert won.any() and not won.all()
        # the score is a sum of d products of 1e30 in 32 bits: its terms are some 10 times the sum at worst
        assert np.all(np.abs(f64(lse[0, h]) - top - np.log(l)) <= np.where(won, 1e-4 * np.abs(top), 1e-4))
        assert np.all(np.abs(f64(O[0, h]) - P @ V) <= rounding * np.abs(P @ V) + 1e-4)
        dV, want = np.concatenate([f64(g[0, h]) for g in dVs]), P.T @ dO
        assert np.abs(dV - want).max() <= rel * np.abs(want).max()
        assert all(bool(torch.isfinite(g).all()) for g in [dQ, *dKs])
        dQ_ref = case["scale"] * ((P * (dO @ V.T - (dO * (P @ V)).sum(1)[:, None])) @ K)
        assert np.abs(f64(dQ[0, h]) - dQ_ref)[~won].max() <= rel * np.abs(dQ_ref[~won]).max()
